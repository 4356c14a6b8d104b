"""Program order within one engine of the interpreter: an engine's load has
landed before its next instruction reads the slot, whether or not anything
waits for the load (an instruction that nothing waits for has no counter), and an
add has written its slot before the next load goes there.
Loads, stores and sums of one engine without dependencies between them, as an
instruction before an inner loop and as sibling inner loops, with loads and
stores of the same and of different widths (one buffer aligned, the other not)."""
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import core  # noqa: E402
from paper_2608_13757_amd import ALLOC_PER_INSTR, ALLOC_PER_LOOP, MODE_BARRIER, MODE_BARRIER_FREE, Plan, bfs  # noqa: E402
from tests.gpu_util import dev, trip_tensors  # noqa: E402
from workloads import (OP_ADDC, OP_LOAD, OP_SCALE_ACC, OP_STORE_ACC, OP_STORE_RING, ProgramBuilder, TripTables,  # noqa: E402
                       draw_trips, tile_args, tile_bases)

PER, GEN = 3, 2


def order_program(form, tile, dep):
    """One engine over A{ LOAD | B{ LOAD }; C{ STORE | ACC } }, slots by r_A (and
    the position in B and C)."""
    b = ProgramBuilder("interp", n_engines=1)
    read = OP_SCALE_ACC if form.endswith("acc") else OP_STORE_RING
    with b.loop("A") as A:
        slot = dict(gen_loop=A, n_gen=GEN)
        if form.startswith("direct"):
            b.instr(0, OP_LOAD, tile_args(src=1, dst=0, idx_loop=A, **slot), name="LOAD")
            n = GEN
        else:
            with b.loop("B") as B:
                b.instr(0, OP_LOAD, tile_args(src=1, dst=0, idx_loop=B, pos_loop=B, per_gen=PER, **slot), name="LOAD")
            n = GEN * PER
        with b.loop("C") as C:
            at = dict(slot) if form.startswith("direct") else dict(slot, pos_loop=C, per_gen=PER)
            b.instr(0, read, tile_args(src=0, dst=0 if read == OP_SCALE_ACC else 2, idx_loop=C, const=0.5, **at), name="READ")
    if read == OP_SCALE_ACC:
        b.instr(0, OP_STORE_ACC, tile_args(src=0, dst=2), name="SUM")
    if dep:
        b.dep("LOAD", "READ", 0)
    p = b.build()
    p.tile_elems, p.ring_slots, p.n_accs = tile, [n], 1
    return p


def overwrite_program(inner, tile):
    """One engine over A{ LOAD r0; ADD r0 -> r1 (alone or in a loop C); LOAD r1;
    STORE r1 }: the second load replaces what the add wrote."""
    b = ProgramBuilder("interp", n_engines=1)
    with b.loop("A") as A:
        slot = dict(gen_loop=A, n_gen=GEN)
        b.instr(0, OP_LOAD, tile_args(src=1, dst=0, idx_loop=A, **slot), name="LOAD0")
        if inner:
            with b.loop("C"):
                b.instr(0, OP_ADDC, tile_args(src=0, dst=1, const=1.0, **slot), name="ADD")
        else:
            b.instr(0, OP_ADDC, tile_args(src=0, dst=1, const=1.0, **slot), name="ADD")
        b.instr(0, OP_LOAD, tile_args(src=1, dst=1, idx_loop=A, **slot), name="LOAD1")
        b.instr(0, OP_STORE_RING, tile_args(src=1, dst=2, idx_loop=A, **slot), name="STORE")
    p = b.build()
    p.tile_elems, p.ring_slots = tile, [GEN, GEN]
    return p


@pytest.mark.gpu
@pytest.mark.parametrize("inner", [False, True])
@pytest.mark.parametrize("tile", [64, 256])
def test_interp_load_after_add(tile, inner):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    bfs.lib()
    n_wg, n_a = 64, 40
    prog = overwrite_program(inner, tile)
    tt = TripTables([draw_trips(prog, lambda l, n: np.full(n, n_a) if l == 1 else np.arange(n) % 3)] * n_wg)
    base = n_a * np.arange(n_wg, dtype=np.int64)
    x = torch.randn(n_wg * n_a * tile, generator=torch.Generator(device="cuda").manual_seed(tile), device="cuda")
    out = torch.zeros_like(x)
    t_dev, o_dev = trip_tensors(tt)
    print(f"[interp order] overwrite tile={tile} inner={inner}", file=sys.stderr, flush=True)
    plan = Plan(prog)
    plan.run([dev(base), x, out], t_dev, o_dev, n_wg, watchdog_polls=20_000_000)
    plan.status()
    assert torch.equal(out, x)


def order_trips(prog, form, n_wg, n_a):
    """B as many loads as C reads; C 0 to 3 of them."""
    rng = np.random.default_rng(n_a)
    reads = {}

    def draw(loop, n):
        if loop == prog.loop_id("A"):
            return np.full(n, n_a)
        return reads.setdefault("n", rng.integers(0, PER + 1, size=n))

    tables = []
    for _ in range(n_wg):
        reads.clear()
        tables.append(draw_trips(prog, draw))
    return TripTables(tables)


CASES = [(form, tile, sx, so, dep) for form in ("direct", "direct_acc", "sibling", "sibling_acc")
         for tile, sx, so in ((64, 0, 0), (192, 0, 0), (256, 0, 0), (256, 1, 1), (256, 1, 0), (256, 0, 1))
         for dep in (False, True)]


def test_order_programs_have_no_counters():
    """Without the declared dependency nothing has a counter, and the plan is accepted."""
    for form, tile, _, _, dep in CASES:
        for alloc in (ALLOC_PER_LOOP, ALLOC_PER_INSTR):
            assert Plan(order_program(form, tile, dep), MODE_BARRIER_FREE, alloc).stats()["n_counters"] == (1 if dep else 0)


@pytest.mark.gpu
@pytest.mark.parametrize("alloc", [ALLOC_PER_LOOP, ALLOC_PER_INSTR])
@pytest.mark.parametrize("form,tile,shift_x,shift_out,dep", CASES)
def test_interp_program_order(form, tile, shift_x, shift_out, dep, alloc):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    bfs.lib()
    n_wg, n_a = 5, 70
    prog = order_program(form, tile, dep)
    tt = order_trips(prog, form, n_wg, n_a)
    _, counts = tile_bases(tt, prog.loop_id("C"))
    per_wg = max(n_a, int(counts.max()))
    base = n_wg + per_wg * np.arange(n_wg, dtype=np.int64)     # output tiles 0 .. n_wg - 1 hold the sums
    n_tiles = n_wg + per_wg * n_wg
    x = np.random.default_rng(tile).uniform(-1, 1, size=(n_tiles, tile)).astype(np.float32)
    trips, off = tt.flat()
    ref = core.values(prog, trips, off, base, x, n_tiles * tile)
    xd = torch.zeros(n_tiles * tile + shift_x, dtype=torch.float32, device="cuda")[shift_x:]
    xd.copy_(torch.from_numpy(x.reshape(-1)))
    t_dev, o_dev = trip_tensors(tt)
    print(f"[interp order] {form} tile={tile} shifts={shift_x},{shift_out} dep={dep} alloc={alloc}", file=sys.stderr, flush=True)
    outs = []
    for mode in (MODE_BARRIER_FREE, MODE_BARRIER):
        od = torch.zeros(n_tiles * tile + shift_out, dtype=torch.float32, device="cuda")[shift_out:]
        plan = Plan(prog, mode, alloc)
        plan.run([dev(base), xd, od], t_dev, o_dev, n_wg, watchdog_polls=20_000_000)
        plan.status()
        outs.append(od.cpu().numpy())
    assert np.array_equal(outs[0], outs[1])
    if form.endswith("acc"):
        # sums of at most n terms of magnitude <= 1/2: each addition rounds a partial sum of at most n / 2
        n = int(counts.max())
        assert np.abs(outs[0].astype(np.float64) - ref).max() <= n * (n / 2) * 2.0 ** -24
    else:
        assert np.array_equal(outs[0], ref.astype(np.float32))
