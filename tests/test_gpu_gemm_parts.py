"""GPU parity of the GEMM's uninstrumented barrier-free kernels (K steps in
pairs; whole tiles, halves, quarters or a mix by the grid's size) with the
instrumented kernel, which runs one K step at a time on whole tiles: every
element sums K in the same order, so the outputs are bit-identical."""
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import mathref  # noqa: E402
from paper_2608_13757_amd import Plan, bfs  # noqa: E402
from tests.gpu_util import trip_tensors  # noqa: E402
from workloads import gemm_program, gemm_trips  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    bfs.lib()


def _program(m, n, k, ring, e_ring, offset=None):
    """offset: of MMA->LOAD in place of the ring's depth."""
    p = gemm_program(m, n, k, ring=ring, e_ring=e_ring)
    reuse = (p.instr_id("MMA"), p.instr_id("LOAD"))
    p.deps = [(a, c, offset if offset and (a, c) == reuse else o) for a, c, o in p.deps]
    return p


def _run(m, n, k, ring, e_ring, steps, chunks, offset=None):
    g = torch.Generator(device="cuda").manual_seed(m + n + k)
    a = torch.randn((m, k), generator=g, device="cuda").bfloat16()
    bt = torch.randn((n, k), generator=g, device="cuda").bfloat16()
    bias = torch.randn((n,), generator=g, device="cuda")
    plan = Plan(_program(m, n, k, ring, e_ring, offset))
    trips, off = trip_tensors(gemm_trips(m, n, k))
    if steps is not None:
        trips[off[:, 1]] = steps
    if chunks is not None:
        trips[off[:, 2]] = chunks
    n_wg = (m // 256) * (n // 256)
    outs = []
    for stats in (None, torch.zeros(n_wg * plan.n_waves * 8, dtype=torch.int64, device="cuda")):
        print(f"[gemm-parts] {m}x{n}x{k} ring={ring} e_ring={e_ring} steps={steps} chunks={chunks} offset={offset} "
              f"stats={stats is not None}", file=sys.stderr, flush=True)
        c = torch.full((m, n), -1.0, dtype=torch.bfloat16, device="cuda")
        plan.run([a, bt, bias, c], trips, off, n_wg, stats=stats, watchdog_polls=20_000_000)
        plan.status()
        outs.append(c)
    assert torch.equal(outs[0].view(torch.int16), outs[1].view(torch.int16))
    return a, bt, bias, outs[0]


# tiles (rows x columns): 1, 8 (XCD map), 64, 65, 128, 129, 256, 257, 330, 385, 513
@pytest.mark.parametrize("tm,tn,k", [
    (1, 1, 32), (1, 1, 64), (4, 2, 96), (8, 8, 160), (5, 13, 32), (13, 5, 224), (8, 16, 96), (1, 128, 64), (3, 43, 96),
    (16, 16, 32), (16, 16, 352), (1, 257, 96), (10, 33, 64), (5, 77, 160), (27, 19, 96)])
def test_gemm_grids(tm, tn, k):
    a, bt, bias, c = _run(256 * tm, 256 * tn, k, 4, 4, None, None)
    # rows of the first and last tile against fp64
    rows = np.r_[0:3, 256 * tm - 3:256 * tm]
    ref = mathref.gelu((a[rows].double() @ bt.double().t() + bias.double()).cpu().numpy())
    # bf16 output: half an ulp (2^-9 relative); the fp32 sum of K <= 352 products of N(0, 1) pairs is
    # off by less than K 2^-24 of its partial sums (below 100)
    err = np.abs(c[rows].double().cpu().numpy() - ref)
    assert (err <= 2.0 ** -8 * np.abs(ref) + 1e-3).all()


@pytest.mark.parametrize("ring,e_ring", [(2, 1), (2, 4), (3, 2), (4, 1), (4, 8)])
@pytest.mark.parametrize("tm,tn", [(2, 3), (9, 11), (2, 150)])
def test_gemm_rings(tm, tn, ring, e_ring):
    _run(256 * tm, 256 * tn, 288, ring, e_ring, None, None)


@pytest.mark.parametrize("e_ring", [1, 4])
@pytest.mark.parametrize("tm,tn,k", [(2, 3, 544), (9, 11, 512), (9, 11, 544), (12, 12, 512), (12, 12, 544), (5, 53, 544)])
def test_gemm_ring_of_two(tm, tn, k, e_ring):
    """One pair of slots: whole tiles in pairs up to K = 512, step by step beyond;
    parts in pairs."""
    _run(256 * tm, 256 * tn, k, 2, e_ring, None, None)


@pytest.mark.parametrize("ring,offset", [(2, 1), (3, 1), (3, 2), (4, 1), (4, 2), (4, 3)])
@pytest.mark.parametrize("tm,tn,k", [(2, 3, 32), (2, 3, 288), (9, 11, 320), (2, 150, 160)])
def test_gemm_smaller_offsets(tm, tn, k, ring, offset):
    """Programs that reuse a ring slot later than they could: LOAD waits for the
    MMA 1, 2 or 3 steps back.  (With 1 a load waits for the MMA before it, so
    steps cannot go in pairs.)"""
    _run(256 * tm, 256 * tn, k, ring, 1, None, None, offset)


@pytest.mark.parametrize("steps,chunks", [(0, 8), (1, 8), (4, 3), (5, 0), (7, 5)])
@pytest.mark.parametrize("tm,tn", [(2, 3), (9, 11), (2, 150)])
def test_gemm_shorter_trips(tm, tn, steps, chunks):
    """Trip tables below K / 32 steps or 8 chunks: partial sums, and chunks
    beyond the trip left as they were."""
    _run(256 * tm, 256 * tn, 224, 4, 4, steps, chunks)


def test_gelu_special_values():
    """GELU at +-0, tiny and large values, infinities and NaN (through K = 32
    with a zero product: the bias is the argument).  Finite values within the
    bf16 rounding (2^-8 of the result) and 4e-7, what the fp32 evaluation is
    off by at most; -inf times a tail of zero is NaN, as in torch."""
    vals = np.array([0.0, -0.0, 1e-30, -1e-30, 5.0, -5.0, 20.0, -20.0, 1e30, -1e30, np.inf, -np.inf, np.nan], np.float32)
    m = n = 256
    a = torch.zeros((m, 32), dtype=torch.bfloat16, device="cuda")
    bias = torch.zeros(n, device="cuda")
    bias[:len(vals)] = torch.from_numpy(vals).cuda()
    trips, off = trip_tensors(gemm_trips(m, n, 32))
    c = torch.zeros((m, n), dtype=torch.bfloat16, device="cuda")
    plan = Plan(gemm_program(m, n, 32))
    print("[gemm-parts] gelu values", file=sys.stderr, flush=True)
    plan.run([a, a, bias, c], trips, off, 1)
    plan.status()
    got = c[17, :len(vals)].double().cpu().numpy()
    ref = torch.nn.functional.gelu(torch.from_numpy(vals).double()).numpy()
    finite = np.isfinite(vals)
    assert (np.abs(got - ref)[finite] <= 2.0 ** -8 * np.abs(ref[finite]) + 4e-7).all()
    assert got[-3] == np.inf and np.isnan(ref[-2]) and np.isnan(got[-2]) and np.isnan(got[-1])
    assert got[9] == 0.0
