"""GPU parity of the chain kernel's uninstrumented barrier-free engines (tiles
staged ahead of the waits, several tiles per hand-off): ring depths from one
slot, trips longer than the ring, empty trips, more than 64 iterations of A
(the trips are held 64 at a time) and fewer tiles than the staging ring."""
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import core  # noqa: E402
from paper_2608_13757_amd import ALLOC_PER_INSTR, ALLOC_PER_LOOP, MODE_BARRIER, MODE_BARRIER_FREE, Plan, bfs  # noqa: E402
from tests.gpu_util import dev, trip_tensors  # noqa: E402
from workloads import TripTables, chain_program, draw_trips, tile_bases  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    bfs.lib()


@pytest.mark.parametrize("ring,outer,lo,hi,n_wg,alloc", [
    (1, 3, 0, 2, 2, ALLOC_PER_LOOP), (2, 1, 1, 1, 1, ALLOC_PER_LOOP), (3, 5, 0, 1, 3, ALLOC_PER_INSTR),
    (4, 64, 0, 12, 5, ALLOC_PER_LOOP), (5, 65, 0, 9, 2, ALLOC_PER_INSTR), (8, 130, 1, 20, 3, ALLOC_PER_LOOP),
    (4, 4, 0, 0, 2, ALLOC_PER_LOOP), (7, 0, 1, 1, 2, ALLOC_PER_LOOP)])
def test_chain_uninstrumented_values(ring, outer, lo, hi, n_wg, alloc):
    prog = chain_program(ring_slots=ring)
    rng = np.random.default_rng([ring, outer])
    tt = TripTables([draw_trips(prog, lambda l, n: np.full(n, outer) if l == 1 else rng.integers(lo, hi + 1, size=n))
                     for _ in range(n_wg)])
    base, counts = tile_bases(tt, prog.loop_id("B"))
    n_tiles = int(counts.sum())
    x = rng.uniform(-1, 1, size=(max(1, n_tiles), 256)).astype(np.float32)
    trips, off = tt.flat()
    ref = core.values(prog, trips, off, base, x, n_wg * 256)
    t_dev, o_dev = trip_tensors(tt)
    outs = []
    for mode in (MODE_BARRIER_FREE, MODE_BARRIER):
        print(f"[chain] ring={ring} outer={outer} trips={lo}..{hi} n_wg={n_wg} alloc={alloc} mode={mode}",
              file=sys.stderr, flush=True)
        plan = Plan(prog, mode, alloc if mode == MODE_BARRIER_FREE else ALLOC_PER_LOOP)
        out = torch.full((n_wg * 256,), float("nan"), dtype=torch.float32, device="cuda")
        plan.run([dev(base), dev(x), out], t_dev, o_dev, n_wg)
        plan.status()
        outs.append(out.cpu().numpy())
    # sums of at most n terms of magnitude <= 1/2: each addition rounds a partial sum of at most n / 2
    n = int(counts.max()) if n_tiles else 0
    assert np.abs(outs[0].astype(np.float64) - ref).max() <= n * (n / 2) * 2.0 ** -24
    assert np.array_equal(outs[0].view(np.uint32), outs[1].view(np.uint32))
