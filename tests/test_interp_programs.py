"""The programs by which the interpreter's GPU tests compare its paths order
every conflicting pair of accesses (otherwise equal outputs would be luck)."""
import numpy as np
import pytest

pytest.importorskip("torch")

from oracle import core, hazard  # noqa: E402
from tests import test_gpu_interp, test_gpu_interp_nest, test_gpu_interp_order  # noqa: E402
from workloads import TripTables, draw_trips, tile_bases  # noqa: E402


def _races(prog, trips_of):
    tt = TripTables([draw_trips(prog, trips_of)])
    trips, off = tt.flat()
    n = 1 + max(tt.total_iters(0, l) for l in range(prog.n_loops))
    base = np.array([1], np.int64)
    res = core.run(prog, trips, off[0], 0, base, np.zeros((n, prog.tile_elems), np.float32), n * prog.tile_elems)
    thr = res.recs["sem_thr"].copy()
    for d, linear in enumerate(prog.dep_linear):
        if linear:
            thr[res.recs["dep"] == d] = core.linearized_records(prog, res, d)["sem_thr"]
    # (the check's tiles start at 0; the launches' behind those that hold the sums)
    return [r for r in hazard.check(prog, res, thresholds=thr) if r[0] != ("buf", 2, 0)]


@pytest.mark.parametrize("slots,depth,acquire,n_a", [("gen", 2, False, 20), ("gen", 2, True, 20), ("gen", 3, False, 6),
                                                     ("pos", 2, True, 20), ("pos", 3, True, 3), ("both", 2, False, 12),
                                                     ("both", 3, False, 4)])
def test_nest_programs_are_race_free(slots, depth, acquire, n_a):
    prog = test_gpu_interp_nest._program(64, slots, depth, acquire)
    rng = np.random.default_rng(1)
    A, B = prog.loop_id("A"), prog.loop_id("B")

    def trips_of(l, n):
        return rng.integers(0, 8, size=n) if l == B else np.full(n, n_a if l == A else 3)
    assert _races(prog, trips_of) == []


@pytest.mark.parametrize("ring,nops,waits", [(1, 0, 0), (4, 0, 0), (3, 2, 0), (4, 0, 4)])
def test_tile_programs_are_race_free(ring, nops, waits):
    prog = test_gpu_interp._program(64, ring, nops, waits)
    rng = np.random.default_rng(ring)
    assert _races(prog, lambda l, n: np.full(n, 5) if l == 1 else rng.integers(0, 9, size=n)) == []


@pytest.mark.parametrize("form", ["direct", "direct_acc", "sibling", "sibling_acc"])
def test_order_programs_are_race_free(form):
    prog = test_gpu_interp_order.order_program(form, 64, False)
    tt = test_gpu_interp_order.order_trips(prog, form, 1, 9)
    tables = iter(tt.per_wg[0][1:])
    assert tile_bases(tt, prog.loop_id("C"))[1][0] > 0
    assert _races(prog, lambda l, n: next(tables)) == []
