"""GPU parity of the interpreter's tile paths: every tile size, buffers at
16-byte and at 4-byte alignment (one wide access or one per 64 elements), the
program held in registers and programs too long for that (more than 64 code
words or waits per engine, read with scalar loads), in both modes."""
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import core  # noqa: E402
from paper_2608_13757_amd import ALLOC_PER_ENGINE, ALLOC_PER_LOOP, MODE_BARRIER, MODE_BARRIER_FREE, Plan, bfs  # noqa: E402
from tests.gpu_util import dev, trip_tensors  # noqa: E402
from workloads import (OP_ADDC, OP_LOAD, OP_NOP, OP_SCALE_ACC, OP_STORE_ACC, OP_STORE_RING, ProgramBuilder,  # noqa: E402
                       TripTables, draw_trips, tile_args, tile_bases)

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    bfs.lib()


def _program(tile, ring, nops, waits):
    """Load / add 1 / store over A{ B{ } } through two rings, an accumulator
    over the loaded tiles, ``nops`` no-ops per engine and iteration of A, and
    ``waits`` more (redundant) waits on the add."""
    b = ProgramBuilder("interp", n_engines=3)
    with b.loop("A"):
        b.instr(0, OP_NOP, name="ACQ")
        for i in range(nops):
            for e in range(3):
                b.instr(e, OP_NOP, name=f"N{i}_{e}")
        with b.loop("B") as B:
            slot = dict(gen_loop=B, n_gen=ring)
            b.instr(0, OP_LOAD, tile_args(src=1, dst=0, idx_loop=B, **slot), name="LOAD")
            b.instr(1, OP_ADDC, tile_args(src=0, dst=1, const=1.0, **slot), name="ADD")
            b.instr(1, OP_SCALE_ACC, tile_args(src=0, dst=0, const=0.5, **slot), name="ACC")
            b.instr(2, OP_STORE_RING, tile_args(src=1, dst=2, idx_loop=B, **slot), name="STORE")
    b.instr(1, OP_STORE_ACC, tile_args(src=0, dst=2), name="SUM")
    b.dep("LOAD", "ADD", 0)
    b.dep("ADD", "STORE", 0)
    b.dep("ACC", "LOAD", ring)
    b.dep("STORE", "ADD", ring)
    b.dep("ACC", "ACQ", 1)                  # slots follow r_B across trips of B
    b.dep("STORE", "SUM", 0)
    b.dep("STORE", "ACQ", 1)
    for k in range(waits):
        b.dep("LOAD", "ADD", 1 + k)
    p = b.build()
    p.tile_elems, p.ring_slots, p.n_accs = tile, [ring, ring], 1
    return p


@pytest.mark.parametrize("mode", [MODE_BARRIER_FREE, MODE_BARRIER])
@pytest.mark.parametrize("tile,ring,shift,nops,waits,alloc", [
    (64, 1, 0, 0, 0, ALLOC_PER_LOOP), (128, 3, 0, 0, 0, ALLOC_PER_LOOP), (192, 9, 0, 0, 0, ALLOC_PER_LOOP),
    (256, 4, 0, 0, 0, ALLOC_PER_LOOP), (256, 12, 1, 0, 0, ALLOC_PER_LOOP), (128, 5, 3, 0, 0, ALLOC_PER_ENGINE),
    (256, 12, 0, 70, 0, ALLOC_PER_LOOP), (192, 2, 1, 70, 0, ALLOC_PER_ENGINE), (256, 4, 0, 0, 80, ALLOC_PER_LOOP)])
def test_interp_tile_paths(tile, ring, shift, nops, waits, alloc, mode):
    n_wg = 3
    if mode == MODE_BARRIER and alloc == ALLOC_PER_ENGINE:
        alloc = ALLOC_PER_LOOP
    prog = _program(tile, ring, nops, waits)
    rng = np.random.default_rng([tile, ring])
    tt = TripTables([draw_trips(prog, lambda l, n: np.full(n, 5) if l == 1 else rng.integers(0, 9, size=n))
                     for _ in range(n_wg)])
    base, counts = tile_bases(tt, prog.loop_id("B"))
    base = base + n_wg                       # output tiles 0 .. n_wg - 1 hold the sums
    n_tiles = n_wg + int(counts.sum())
    x = rng.uniform(-1, 1, size=(n_tiles, tile)).astype(np.float32)
    trips, off = tt.flat()
    ref = core.values(prog, trips, off, base, x, n_tiles * tile)
    xd = torch.zeros(n_tiles * tile + shift, dtype=torch.float32, device="cuda")[shift:]
    xd.copy_(torch.from_numpy(x.reshape(-1)))
    od = torch.zeros(n_tiles * tile + shift, dtype=torch.float32, device="cuda")[shift:]
    print(f"[interp] tile={tile} ring={ring} shift={shift} nops={nops} waits={waits} alloc={alloc} mode={mode}",
          file=sys.stderr, flush=True)
    plan = Plan(prog, mode, alloc)
    t_dev, o_dev = trip_tensors(tt)
    plan.run([dev(base), xd, od], t_dev, o_dev, n_wg)
    plan.status()
    got = od.cpu().numpy()
    cut = n_wg * tile
    assert np.array_equal(got[cut:], x.reshape(-1)[cut:] + np.float32(1.0))
    # sums of at most n terms of magnitude <= 1/2: each addition rounds a partial sum of at most n / 2
    n = int(counts.max())
    assert np.abs(got[:cut].astype(np.float64) - ref[:cut]).max() <= n * (n / 2) * 2.0 ** -24
