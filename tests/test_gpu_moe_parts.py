"""MoE grouped GEMM in units of work items (barrier-free, uninstrumented)
against the same program instrumented, which runs whole items one step at a
time: every element has the same order of K in both, so the outputs are equal
bit for bit.  (The instrumented run against the fp64 oracle is
test_gpu_moe.py's.)"""
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2608_13757_amd import ALLOC_PER_INSTR, ALLOC_PER_LOOP, MODE_BARRIER_FREE, BfsError, Plan, bfs  # noqa: E402
from tests.gpu_util import trip_tensors  # noqa: E402
from workloads import moe_program, moe_worklist  # noqa: E402
from workloads.configs import moe_chunks  # noqa: E402

pytestmark = pytest.mark.gpu

RAGGED = [300, 0, 129, 1, 530, 33, 256, 31]
# (counts, K, N, bm, mchunk, options); N is a multiple of both phases' tiles.
# Quarters where 2 sum ceil(rows / 128) N-tiles <= 256, units on several
# workgroups of their item up to 128 items (phase 2: 512), in turn beyond; K
# steps: one, odd, even.
CASES = {
    "quarters": (RAGGED, 256, 256, 256, None, {}),
    "quarters_one_step": (RAGGED, 32, 256, 256, None, {}),
    "quarters_odd_k": (RAGGED, 352, 256, 256, None, {"ring": 2, "e_ring": 1}),
    "quarters_128_linear": (RAGGED, 320, 256, 128, 2, {"linear": True}),
    "quarters_one_row": ([1], 96, 256, 256, None, {}),
    "split": ([1100, 900, 255, 257, 64, 1, 0, 700], 224, 1280, 256, None, {}),
    "split_two_slots": ([1100, 900, 255, 257, 64, 1, 0, 700], 128, 1280, 256, 3, {"ring": 2, "e_ring": 2}),
    "split_odd_ring": ([1100, 900, 255, 257, 64, 1, 0, 700], 96, 1280, 256, 9, {"ring": 3, "e_ring": 1}),
    "split_one_step": ([1100, 900, 255, 257, 64, 1, 0, 700], 32, 1280, 256, None, {"linear": False}),
    "split_128": ([1100, 900, 255, 257, 64, 1, 0, 700], 288, 1280, 128, None, {}),
    "split_128_ring": ([1100, 900, 255, 257, 64, 1, 0, 700], 160, 1280, 128, 3, {"ring": 4, "e_ring": 0}),
    "split_linear": ([1100, 900, 255, 257, 64, 1, 0, 700], 192, 1280, 256, None, {"linear": True}),
    "items": ([40, 300, 0, 1, 257, 96, 31, 510, 32, 33], 160, 16384, 256, 1, {}),
    "items_128_linear": ([40, 300, 0, 1, 257, 96, 31, 510, 32, 33], 192, 16384, 128, 2, {"linear": True, "e_ring": 1}),
    "items_long_runs": ([1100, 900, 255, 257, 64, 1, 0, 700], 96, 20480, 256, 9, {}),
    "items_phases": ([1100, 900, 255, 257, 64, 1, 0, 700], 224, 6144, 256, None, {}),
    "quarters_128_odd_k": (RAGGED, 352, 256, 128, None, {}),
    "quarters_padded": ([40, 0, 0, 129, 0, 7, 300, 1], 160, 512, 128, 1, {"ring": 3, "e_ring": 1}),
    "quarters_all_cus": ([128, 127, 1, 65] * 8, 96, 1024, 128, None, {"linear": False}),
    "split_128_linear_odd_ring": ([1100, 900, 255, 257, 64, 1, 0, 700], 192, 1280, 128, None, {"linear": True}),
    "items_128_odd_ring": ([40, 300, 0, 1, 257, 96, 31, 510, 32, 33], 224, 16384, 128, 2, {}),
    "items_128_odd_ring_odd_k": ([40, 300, 0, 1, 257, 96, 31, 510, 32, 33], 160, 16384, 128, 3, {"ring": 3, "e_ring": 2}),
    "items_128_long_k": ([40, 300, 0, 1, 257, 96, 31, 510, 32, 33], 576, 8192, 128, 2, {}),
    "items_128_long_odd_k": ([40, 300, 0, 1, 257, 96, 31, 510, 32, 33], 544, 16384, 128, 3, {}),
    "whole_128_short_k": ([40, 300, 0, 1, 257, 96, 31, 510, 32, 33], 256, 8192, 128, 2, {}),
    "whole_odd_ring": ([1100, 900, 255, 257, 64, 1, 0, 700], 96, 6144, 256, 2, {"ring": 3, "e_ring": 1}),
    "linear_odd_k": (RAGGED, 96, 256, 256, None, {"linear": True}),      # stays whole
}


@pytest.mark.parametrize("alloc", [ALLOC_PER_LOOP, ALLOC_PER_INSTR])
@pytest.mark.parametrize("phase", [1, 2])
@pytest.mark.parametrize("case", sorted(CASES))
def test_moe_units_equal_items(case, phase, alloc):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    bfs.lib()
    counts, k, n, bm, mchunk, opt = CASES[case]
    tokens = sum(counts)
    g = torch.Generator(device="cuda").manual_seed(7)

    def rand(*shape):
        return torch.randn(*shape, generator=g, device="cuda").to(torch.bfloat16)

    hidden, ffn = (k, n) if phase == 1 else (n, k)
    perm = torch.randperm(tokens, generator=g, device="cuda").to(torch.int32)
    eoff = torch.tensor(np.concatenate([[0], np.cumsum(counts)]).astype(np.int32), device="cuda")
    wl = moe_worklist(counts, phase, hidden, ffn, mchunk=mchunk, bm=bm)
    trips, toff = trip_tensors(wl.trips)
    plan = Plan(moe_program(phase, hidden, ffn, bm=bm, **opt), MODE_BARRIER_FREE, alloc)
    weights = [rand(len(counts), n, k) for _ in range(2 if phase == 1 else 1)]
    ins = [torch.from_numpy(wl.work.reshape(-1)).cuda(), perm, eoff, rand(tokens, k), *weights]
    outs = []
    for cap in (0, 4):
        out = torch.full((tokens, n), -1, dtype=torch.int16, device="cuda")
        log = torch.zeros(plan.debug_log_words(wl.trips.n_wg, cap), dtype=torch.int32, device="cuda") if cap else None
        plan.run(ins + [out], trips, toff, wl.trips.n_wg, debug_log=log, debug_capacity=cap)
        plan.status()
        outs.append(out)
    assert torch.isfinite(outs[1].view(torch.bfloat16).float()).all()
    assert torch.equal(outs[0], outs[1])


@pytest.mark.parametrize("instrumented", [False, True])
@pytest.mark.parametrize("phase", [1, 2])
@pytest.mark.parametrize("case", ["quarters", "split", "items", "items_128_odd_ring", "items_phases"])
@pytest.mark.parametrize("expert_rows", ["none", "some"])
def test_moe_trip_beyond_rows_is_reported(case, phase, instrumented, expert_rows):
    """An item whose M loop runs beyond its expert's M-tiles, without rows (no
    unit of it runs) or with some, is reported by every kernel, at the ends of
    the item list and inside."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    bfs.lib()
    counts, k, n, bm, mchunk, opt = CASES[case]
    tokens = sum(counts)
    hidden, ffn = (k, n) if phase == 1 else (n, k)
    perm = torch.arange(tokens, dtype=torch.int32, device="cuda")
    eoff = torch.tensor(np.concatenate([[0], np.cumsum(counts)]).astype(np.int32), device="cuda")
    wl = moe_worklist(counts, phase, hidden, ffn, mchunk=mchunk, bm=bm)
    trips, toff = wl.trips.flat()
    plan = Plan(moe_program(phase, hidden, ffn, bm=bm, **opt))
    ins = [perm, eoff] + [torch.zeros(s, dtype=torch.bfloat16, device="cuda")
                          for s in [(tokens, k)] + [(len(counts), n, k)] * (2 if phase == 1 else 1)]
    out = torch.zeros((tokens, n), dtype=torch.bfloat16, device="cuda")
    n_wg = wl.trips.n_wg
    stats = torch.zeros(n_wg * plan.n_waves * 8, dtype=torch.int64, device="cuda") if instrumented else None
    expert = counts.index(0) if expert_rows == "none" else counts.index(max(counts))
    limit = -(-counts[expert] // bm)
    for at in (0, n_wg // 2 + 3, n_wg - 1):
        work, t = wl.work.copy(), trips.copy()
        work[at] = (expert, 0, 0, limit + 1)
        # an own table behind the others: M beyond the rows, K and C for these M-tiles
        tables = np.r_[[limit + 1], np.full(limit + 1, k // 32), np.full(limit + 1, moe_chunks(phase, bm))]
        off = toff.copy()
        off[at, 1:] = len(t) + np.array([0, 1, 1 + limit + 1])
        args = [torch.from_numpy(work.reshape(-1)).cuda()] + ins + [out]
        dev = [torch.from_numpy(a).cuda() for a in (np.r_[t, tables.astype(np.int32)], off)]
        print(f"[moe trips] {case} phase={phase} rows={expert_rows} instrumented={instrumented} item {at} of {n_wg}",
              file=sys.stderr, flush=True)
        plan.run(args, dev[0], dev[1], n_wg, stats=stats)
        with pytest.raises(BfsError) as e:
            plan.status()
        assert e.value.status == bfs.E_INVALID
        plan.status()                          # reported once
