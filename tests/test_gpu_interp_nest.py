"""The interpreter's inner loops of one instruction (decoded once, run without
dispatch, over the trips of the loop around them where it holds nothing else):
every datapath, tile size and form of ring slot, two- and three-level nests
with empty trips, more trips than are read at a time.  The output tiles are x +
1 exactly; the accumulated sums are those of barrier mode bit for bit, which
runs every instruction on the general path in the same order."""
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2608_13757_amd import ALLOC_PER_INSTR, ALLOC_PER_LOOP, MODE_BARRIER, MODE_BARRIER_FREE, Plan, bfs  # noqa: E402
from tests.gpu_util import dev, trip_tensors  # noqa: E402
from workloads import (OP_ADDC, OP_LOAD, OP_NOP, OP_SCALE_ACC, OP_STORE_ACC, OP_STORE_RING, ProgramBuilder,  # noqa: E402
                       TripTables, draw_trips, tile_args, tile_bases)

pytestmark = pytest.mark.gpu


def _program(tile, slots, depth, acquire):
    """Four engines over [O{] [ACQO] A{ [ACQ] B{ LOAD | ADD | ACC | STORE } } [}].
    Slots by the position in B start over at each iteration of O too, where ACQ's
    offset, counted per trip of A, does not reach back: ACQO drains them there."""
    b = ProgramBuilder("interp", n_engines=4)

    def nest():
        with b.loop("A") as A:
            if acquire:
                b.instr(0, OP_NOP, name="ACQ")
            with b.loop("B") as B:
                if slots == "gen":                       # slots follow r_B, reused after 4
                    slot, n = dict(gen_loop=B, n_gen=4), 4
                elif slots == "pos":                     # slots follow rhat_B, drained by ACQ
                    slot, n = dict(pos_loop=B, per_gen=7), 7
                else:                                    # slots follow r_A and rhat_B, never reused
                    slot, n = dict(gen_loop=A, n_gen=12, pos_loop=B, per_gen=7), 84
                b.instr(0, OP_LOAD, tile_args(src=1, dst=0, idx_loop=B, **slot), name="LOAD")
                b.instr(1, OP_ADDC, tile_args(src=0, dst=1, const=1.0, **slot), name="ADD")
                b.instr(3, OP_SCALE_ACC, tile_args(src=0, dst=0, const=0.5, **slot), name="ACC")
                b.instr(2, OP_STORE_RING, tile_args(src=1, dst=2, idx_loop=B, **slot), name="STORE")
        return n

    if depth == 3:
        with b.loop("O"):
            if acquire and slots == "pos":
                b.instr(0, OP_NOP, name="ACQO")
            n = nest()
    else:
        n = nest()
    b.instr(3, OP_STORE_ACC, tile_args(src=0, dst=2), name="SUM")
    b.dep("LOAD", "ADD", 0)
    b.dep("LOAD", "ACC", 0)
    b.dep("ADD", "STORE", 0)
    if slots != "both":
        linear = slots == "gen" and not acquire
        b.dep("ADD", "LOAD", n, linear=linear)
        b.dep("ACC", "LOAD", n, linear=linear)
        b.dep("STORE", "ADD", n, linear=linear)
    if acquire:
        if slots == "gen":                               # (three waits; STORE's implies it)
            b.dep("ADD", "ACQ", 1)
        b.dep("ACC", "ACQ", 1)
        b.dep("STORE", "ACQ", 1)
        if depth == 3 and slots == "pos":
            b.dep("ACC", "ACQO", 1)
            b.dep("STORE", "ACQO", 1)
    p = b.build()
    p.tile_elems, p.ring_slots, p.n_accs = tile, [n, n], 1
    return p


@pytest.mark.parametrize("alloc", [ALLOC_PER_LOOP, ALLOC_PER_INSTR])
@pytest.mark.parametrize("slots,depth,acquire,n_a,tile,shift",
                         [(*c, *t) for c in [("gen", 2, False, 150), ("gen", 2, True, 70), ("gen", 3, False, 9),
                                             ("pos", 2, True, 66), ("pos", 3, True, 3)]
                          for t in [(64, 0), (192, 0), (256, 0), (256, 1)]] +
                         [("both", 2, False, 12, 64, 0), ("both", 3, False, 4, 64, 0)])
def test_interp_inner_loops(slots, depth, acquire, n_a, tile, shift, alloc):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    bfs.lib()
    n_wg = 3
    prog = _program(tile, slots, depth, acquire)
    rng = np.random.default_rng([tile, depth, n_a])
    A, B = prog.loop_id("A"), prog.loop_id("B")

    def draw(loop, n):
        if loop == B:
            return rng.integers(0, 8, size=n)
        return np.full(n, n_a if loop == A else 3)

    tt = TripTables([draw_trips(prog, draw) for _ in range(n_wg)])
    base, counts = tile_bases(tt, B)
    base = base + n_wg                       # output tiles 0 .. n_wg - 1 hold the sums
    n_tiles = n_wg + int(counts.sum())
    x = rng.uniform(-1, 1, size=n_tiles * tile).astype(np.float32)
    xd = torch.zeros(n_tiles * tile + shift, dtype=torch.float32, device="cuda")[shift:]
    xd.copy_(torch.from_numpy(x))
    t_dev, o_dev = trip_tensors(tt)
    print(f"[interp nest] {slots} depth={depth} acquire={acquire} tile={tile} shift={shift} alloc={alloc}",
          file=sys.stderr, flush=True)
    outs = []
    for mode in (MODE_BARRIER_FREE, MODE_BARRIER):
        od = torch.zeros(n_tiles * tile + shift, dtype=torch.float32, device="cuda")[shift:]
        plan = Plan(prog, mode, alloc)
        plan.run([dev(base), xd, od], t_dev, o_dev, n_wg, watchdog_polls=20_000_000)
        plan.status()
        outs.append(od.cpu().numpy())
    assert np.array_equal(outs[0], outs[1])
    assert np.array_equal(outs[0][n_wg * tile:], x[n_wg * tile:] + np.float32(1.0))
