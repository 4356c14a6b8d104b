"""The cases by which the performance of this library is measured.

Every case plans a program with ``Plan`` and launches it with ``Plan.run``,
the way a program that uses the library does: the plan, the trip tables and
the device buffers exist before the call, and a pass enqueues the launches on
the current stream.  All kernel families are covered, in barrier-free mode
(the mode that is used in earnest; the barrier mode is the scheme it is
compared with), from one workgroup to launches that fill the GPU.
"""
import math

import numpy as np
import torch

from paper_2608_13757_amd import ALLOC_PER_ENGINE, ALLOC_PER_INSTR, ALLOC_PER_LOOP, MODE_BARRIER_FREE, Plan
from workloads import (ADAM_HP, TripTables, adamw_default_wg, adamw_program, adamw_worklist, attn_program,
                       attn_worklist, chain_program, draw_trips, gemm_program, gemm_trips, moe_program,
                       moe_worklist, ring_program, rmsnorm_program, rmsnorm_worklist, stream_program, tile_bases)
from workloads.tensors import zipf_counts

ALLOCS = {"per_loop": ALLOC_PER_LOOP, "per_instr": ALLOC_PER_INSTR, "per_engine": ALLOC_PER_ENGINE}
RMS_EPS = 1e-6
RMS_MAX_WG = 768        # three workgroups on each compute unit


def listed():
    return [
        # The smallest call: a two-engine chain in one workgroup, a dependent
        # sequence of 1 KiB tile hand-offs.  Latency and launch cost only.
        dict(name="chain_one_wg", kind="chain", n_wg=1, outer=16, inner_max=8, ring=4),
        # A program that no dedicated kernel serves, on the generic interpreter
        # over a grid that fills the GPU: what a new program runs on first.
        dict(name="interp_ring_1024wg", kind="interp", program="ring", linear=True, alloc="per_loop", n_wg=1024,
             outer=64, inner_max=8, ring=4),
        # The synchronization-bound load / add / store stream over a dynamically
        # bounded three-level nest, at the benchmark's size.
        dict(name="stream_1024wg", kind="stream", n_wg=1024, outer=256, mid_max=16, inner_max=4, layout="inplace"),
        # A fused linear layer (GEMM + bias + GELU) of a few hundred tokens with
        # odd sizes: three output tiles and a K of three steps.
        dict(name="gemm_256x768x96", kind="gemm", m=256, n=768, k=96),
        # The same layer at 2048 tokens and features: fewer output tiles than
        # the GPU has compute units.
        dict(name="gemm_2048", kind="gemm", m=2048, n=2048, k=2048),
        # ... and with one output tile for each compute unit.
        dict(name="gemm_4096", kind="gemm", m=4096, n=4096, k=4096),
        # Attention forward of a batch of short ragged prompts.
        dict(name="attn_short_prompts", kind="attn", batch=8, heads=8, lmin=1, lmax=512, linear=False),
        # Attention forward of a large batch of ragged sequences (prefill).
        dict(name="attn_varlen_32x4096", kind="attn", batch=32, heads=16, lmin=128, lmax=4096, linear=False),
        # A dropless mixture-of-experts layer of a small batch: few tokens per
        # expert, every expert with a ragged last tile.
        dict(name="moe_2048tok_8e", kind="moe", tokens=2048, experts=8, hidden=1024, ffn=1408, zipf=0.5, bm=256,
             linear=False),
        # The layer at prefill size with skewed routing (Zipf 1.1 over 64 experts).
        dict(name="moe_32768tok_64e", kind="moe", tokens=32768, experts=64, hidden=4096, ffn=1408, zipf=1.1, bm=256,
             linear=False),
        # RMSNorm + per-row FP8 quantization of a prefill's activations.
        dict(name="rmsnorm_32768x8192", kind="rmsnorm", t=32768, h=8192),
        # One optimizer step over a million parameters (updates p, m and v).
        dict(name="adamw_1m", kind="adamw", n=1 << 20, chunk=1024),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: the families in turn by chance, sizes spread over the
    logarithm of their ranges, options as users set them."""
    kind = rng.choice(["chain", "interp", "stream", "gemm", "gemm", "attn", "attn", "moe", "moe", "rmsnorm", "adamw"])
    if kind == "chain":
        return dict(kind=kind, n_wg=_log_int(rng, 1, 512), outer=_log_int(rng, 2, 64), inner_max=rng.randint(1, 12),
                    ring=rng.randint(2, 8))
    if kind == "interp":
        return dict(kind=kind, program=rng.choice(["ring", "chain"]), linear=rng.random() < 0.5,
                    alloc=rng.choice(["per_loop", "per_loop", "per_instr", "per_engine"]),
                    n_wg=_log_int(rng, 1, 1024), outer=_log_int(rng, 2, 64), inner_max=rng.randint(1, 8),
                    ring=rng.randint(2, 8))
    if kind == "stream":
        return dict(kind=kind, n_wg=_log_int(rng, 1, 1024), outer=_log_int(rng, 1, 256), mid_max=rng.randint(1, 16),
                    inner_max=rng.randint(1, 4), layout=rng.choice(["inplace", "inplace", "two_rings"]))
    if kind == "gemm":
        return dict(kind=kind, m=256 * _log_int(rng, 1, 24), n=256 * _log_int(rng, 1, 24), k=32 * _log_int(rng, 1, 256))
    if kind == "attn":
        lmax = _log_int(rng, 32, 4096)
        return dict(kind=kind, batch=_log_int(rng, 1, 32), heads=rng.randint(1, 16), lmin=rng.randint(1, lmax),
                    lmax=lmax, linear=rng.random() < 0.3)
    if kind == "moe":
        return dict(kind=kind, tokens=_log_int(rng, 16, 32768), experts=rng.choice([4, 8, 16, 32, 64]),
                    hidden=256 * _log_int(rng, 1, 16), ffn=128 * _log_int(rng, 1, 11), zipf=round(rng.uniform(0, 1.2), 2),
                    bm=rng.choice([256, 256, 128]), linear=rng.random() < 0.3)
    if kind == "rmsnorm":
        return dict(kind=kind, t=_log_int(rng, 1, 32768), h=rng.choice([1024, 2048, 4096, 8192]))
    return dict(kind=kind, n=4 * _log_int(rng, 1, 1 << 25), chunk=rng.choice([512, 1024, 1024]))


# ---------------------------------------------------------------------------
# what a program has in hand before the call
# ---------------------------------------------------------------------------
def _gen(seed, stream=0):
    return torch.Generator(device="cuda").manual_seed(1000003 * (seed + 1) + stream)


def _normal(seed, stream, shape, scale=1.0, dtype=torch.bfloat16):
    x = torch.empty(shape, dtype=dtype, device="cuda")
    x.normal_(0.0, scale, generator=_gen(seed, stream))
    return x


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _launch(program, trips, bufs, alloc=ALLOC_PER_LOOP):
    t, off = trips.flat()
    return dict(plan=Plan(program, MODE_BARRIER_FREE, alloc), bufs=bufs, trips=_dev(t), off=_dev(off), n_wg=trips.n_wg)


def _nest(case, seed, program, outer, mid_max, inner_max):
    """Trip tables of a nest: the outermost loop runs ``outer`` times, the
    loops below a count that is known only at run time.  The case fixes the
    workgroups' tables and the seed their order, so that the number of tiles
    does not depend on the seed."""
    rng = np.random.default_rng([case["n_wg"], outer, inner_max])

    def trips_of(l, n):
        if l == 1:
            return np.full(n, outer)
        return rng.integers(1, (mid_max if l == 2 and program.n_loops == 4 else inner_max) + 1, size=n)
    tables = [draw_trips(program, trips_of) for _ in range(case["n_wg"])]
    return TripTables([tables[w] for w in np.random.default_rng(seed).permutation(case["n_wg"])])


def _tiles(case, seed):
    """Program, trip tables, tile bases and tile counts of a tile workload."""
    if case["kind"] == "stream":
        two = case["layout"] == "two_rings"
        program = stream_program(n_gen=8 if two else 32, per_gen=case["inner_max"], layout=case["layout"])
        trips = _nest(case, seed, program, case["outer"], case["mid_max"], case["inner_max"])
    else:
        if case["kind"] == "chain":
            program = chain_program(ring_slots=case["ring"])
        elif case["program"] == "chain":
            program = chain_program(ring_slots=case["ring"], kernel="interp")
        else:
            program = ring_program(case["ring"], linear=case["linear"])
        trips = _nest(case, seed, program, case["outer"], 0, case["inner_max"])
    base, counts = tile_bases(trips, program.n_loops - 1)
    return program, trips, base, counts


def _tile_data(case, seed, counts):
    elems = 64 if case["kind"] == "stream" else 256
    x = torch.empty((int(counts.sum()), elems), dtype=torch.float32, device="cuda")
    return x.uniform_(-1.0, 1.0, generator=_gen(seed))


def _lengths(case, seed):
    """Sequence lengths: the case fixes which, the seed their order."""
    rng = np.random.default_rng([case["batch"], case["lmin"], case["lmax"]])
    lengths = rng.integers(case["lmin"], case["lmax"] + 1, size=case["batch"])
    return np.random.default_rng(seed).permutation(lengths)


def _qkv(case, seed, tokens):
    return [_normal(seed, 1 + i, (tokens, case["heads"], 128)) for i in range(3)]


def _routing(case, seed):
    """Tokens per expert, token ids grouped by expert and group offsets."""
    rng = np.random.default_rng(seed)
    counts = zipf_counts(case["tokens"], case["experts"], case["zipf"])[rng.permutation(case["experts"])]
    assign = rng.permutation(np.repeat(np.arange(case["experts"]), counts))
    perm = np.argsort(assign, kind="stable").astype(np.int32)
    return counts, perm, np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)


def _moe_data(case, seed):
    e, h, f = case["experts"], case["hidden"], case["ffn"]
    return (_normal(seed, 1, (case["tokens"], h)), _normal(seed, 2, (e, f, h), 0.02), _normal(seed, 3, (e, f, h), 0.02),
            _normal(seed, 4, (e, h, f), 0.02))


def _rms_data(case, seed):
    """Activations with a few outlier channels, and a gain near one."""
    t, h = case["t"], case["h"]
    x = _normal(seed, 1, (t, h))
    channels = np.random.default_rng(seed).choice(h, size=max(1, h // 200), replace=False)
    x[:, _dev(channels)] *= 20.0
    return x, 1.0 + _normal(seed, 2, (h,), 0.1)


def _adam_data(case, seed):
    n, f32 = case["n"], torch.float32
    p, g = _normal(seed, 1, (n,), 0.02, f32), _normal(seed, 2, (n,), 0.01, f32)
    g = torch.where(torch.rand(n, device="cuda", generator=_gen(seed, 3)) < 0.01, 30.0 * g, g)
    return p, g, _normal(seed, 4, (n,), 0.003, f32), _normal(seed, 5, (n,), 0.01, f32).square_()


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("chain", "interp", "stream"):
        program, trips, base, counts = _tiles(case, seed)
        x = _tile_data(case, seed, counts)
        out = torch.empty_like(x) if kind == "stream" else x.new_empty((case["n_wg"], 256))
        alloc = ALLOCS[case.get("alloc", "per_loop")]
        return dict(launches=[_launch(program, trips, [_dev(base), x, out], alloc)], out=[out])
    if kind == "gemm":
        m, n, k = case["m"], case["n"], case["k"]
        out = torch.empty((m, n), dtype=torch.bfloat16, device="cuda")
        bufs = [_normal(seed, 1, (m, k), 1 / 64), _normal(seed, 2, (n, k), 1 / 64),
                _normal(seed, 3, (n,), 1.0, torch.float32), out]
        return dict(launches=[_launch(gemm_program(m, n, k), gemm_trips(m, n, k), bufs)], out=[out])
    if kind == "attn":
        lengths = _lengths(case, seed)
        work = attn_worklist(lengths, case["heads"])
        q, k, v = _qkv(case, seed, int(lengths.sum()))
        out = torch.empty_like(q)
        program = attn_program(case["heads"], linear=case["linear"])
        return dict(launches=[_launch(program, work.trips, [_dev(work.work), q, k, v, out])], out=[out])
    if kind == "moe":
        counts, perm, offsets = _routing(case, seed)
        x, w_gate, w_up, w_down = _moe_data(case, seed)
        perm, offsets = _dev(perm), _dev(offsets)
        h = x.new_empty((case["tokens"], case["ffn"]))
        y = torch.empty_like(x)
        launches = []
        for phase, data in ((1, [x, w_gate, w_up, h]), (2, [h, w_down, y])):
            work = moe_worklist(counts, phase, case["hidden"], case["ffn"], bm=case["bm"])
            program = moe_program(phase, case["hidden"], case["ffn"], bm=case["bm"], linear=case["linear"])
            launches.append(_launch(program, work.trips, [_dev(work.work), perm, offsets] + data))
        return dict(launches=launches, out=[h, y])
    if kind == "rmsnorm":
        t, h = case["t"], case["h"]
        base, trips = rmsnorm_worklist(t, min(RMS_MAX_WG, t))
        x, gamma = _rms_data(case, seed)
        codes = torch.empty((t, h), dtype=torch.uint8, device="cuda")
        scales = torch.empty((t,), dtype=torch.float32, device="cuda")
        program = rmsnorm_program(t, h, waves=2 if h == 1024 else 4, eps=RMS_EPS)
        return dict(launches=[_launch(program, trips, [_dev(base), x, gamma, codes, scales])], out=[codes, scales])
    n, chunk = case["n"], case["chunk"]
    base, trips = adamw_worklist(n, chunk, adamw_default_wg(n, chunk))
    p, g, m, v = _adam_data(case, seed)
    program = adamw_program(n, chunk, **ADAM_HP)
    return dict(launches=[_launch(program, trips, [_dev(base), p, g, m, v])], out=[p, m, v])


def run(state):
    for x in state["launches"]:
        x["plan"].run(x["bufs"], x["trips"], x["off"], x["n_wg"])
    return state["out"]


# ---------------------------------------------------------------------------
# what a pass cannot do without, and how exact it is
# ---------------------------------------------------------------------------
def work(case):
    kind = case["kind"]
    if kind in ("chain", "interp", "stream"):
        tiles = case["n_wg"] * case["outer"] * (1 + case["inner_max"]) / 2
        if kind == "stream":
            tiles *= (1 + case["mid_max"]) / 2
            return dict(bytes=tiles * 512, flops=tiles * 64)
        return dict(bytes=tiles * 1024 + case["n_wg"] * 1024, flops=tiles * 512)
    if kind == "gemm":
        m, n, k = case["m"], case["n"], case["k"]
        return dict(bytes=2 * (m * k + n * k + m * n) + 4 * n, flops=2.0 * m * n * k)
    if kind == "attn":
        lengths, h = _lengths(case, 0).astype(np.float64), case["heads"]
        return dict(bytes=float(lengths.sum()) * h * 128 * 2 * 4, flops=4.0 * 128 * h * float((lengths * lengths).sum()))
    if kind == "moe":
        t, h, f = case["tokens"], case["hidden"], case["ffn"]
        used = int(np.count_nonzero(zipf_counts(t, case["experts"], case["zipf"])))
        return dict(bytes=2.0 * (2 * t * h + 2 * t * f + 3 * used * h * f), flops=6.0 * t * h * f)
    if kind == "rmsnorm":
        return dict(bytes=case["t"] * (3 * case["h"] + 4) + 2 * case["h"], flops=6.0 * case["t"] * case["h"])
    return dict(bytes=28.0 * case["n"], flops=20.0 * case["n"])


def tolerance(case):
    kind = case["kind"]
    if kind == "stream":
        return "exact"                              # one fp32 addition per element
    if kind in ("chain", "interp"):
        return dict(rel=1.5e-6)                     # fp32 sums of some hundred tiles
    if kind == "gemm":
        return dict(rel=7e-3, max=0.03)             # fp32 accumulation, output rounded to bf16
    if kind == "attn":
        return dict(rel=1.2e-2, max=0.1)            # ... with probabilities rounded to bf16
    if kind == "moe":
        return dict(rel=1.2e-2, max=0.1)            # ... with h rounded to bf16 between the two products
    if kind == "rmsnorm":
        return dict(rel=5e-7, differ=1e-4)          # scales; codes next to a rounding midpoint
    return dict(rel=2e-7, max=1e-5)                 # fp32 element-wise


def exact(case, seed):
    """The outputs in 64-bit arithmetic (FP8 codes have no such value)."""
    kind, f64 = case["kind"], torch.float64
    if kind in ("chain", "interp", "stream"):
        _, _, _, counts = _tiles(case, seed)
        x = _tile_data(case, seed, counts)
        if kind == "stream":
            return [x.to(f64) + 1.0]
        out = torch.zeros((case["n_wg"], 256), dtype=f64, device="cuda")
        owner = torch.repeat_interleave(torch.arange(case["n_wg"], device="cuda"), _dev(counts))
        return [out.index_add_(0, owner, 0.5 * x.to(f64))]
    if kind == "gemm":
        m, n, k = case["m"], case["n"], case["k"]
        a, bt = _normal(seed, 1, (m, k), 1 / 64), _normal(seed, 2, (n, k), 1 / 64)
        z = a.to(f64) @ bt.to(f64).t() + _normal(seed, 3, (n,), 1.0, torch.float32).to(f64)
        return [0.5 * z * (1.0 + torch.erf(z / math.sqrt(2.0)))]
    if kind == "attn":
        lengths = _lengths(case, seed)
        q, k, v = _qkv(case, seed, int(lengths.sum()))
        out, lo = torch.empty(q.shape, dtype=f64, device="cuda"), 0
        for n in lengths.tolist():
            for h in range(case["heads"]):
                qs, ks, vs = (t[lo:lo + n, h].to(f64) for t in (q, k, v))
                out[lo:lo + n, h] = torch.softmax(qs @ ks.t() / math.sqrt(128.0), dim=-1) @ vs
            lo += n
        return [out]
    if kind == "moe":
        counts, perm, offsets = _routing(case, seed)
        x, w_gate, w_up, w_down = _moe_data(case, seed)
        h = torch.empty((case["tokens"], case["ffn"]), dtype=f64, device="cuda")
        y = torch.empty((case["tokens"], case["hidden"]), dtype=f64, device="cuda")
        for e in range(case["experts"]):
            rows = _dev(perm[offsets[e]:offsets[e + 1]].astype(np.int64))
            if len(rows):
                xe = x[rows].to(f64)
                he = torch.nn.functional.silu(xe @ w_gate[e].to(f64).t()) * (xe @ w_up[e].to(f64).t())
                h[offsets[e]:offsets[e + 1]] = he
                y[rows] = he @ w_down[e].to(f64).t()
        return [h, y]
    if kind == "rmsnorm":
        x, gamma = _rms_data(case, seed)
        scales = torch.empty((case["t"],), dtype=f64, device="cuda")
        for lo in range(0, case["t"], 4096):
            r = x[lo:lo + 4096].to(f64)
            y = r * torch.rsqrt(r.square().mean(dim=1, keepdim=True) + RMS_EPS) * gamma.to(f64)
            top = y.abs().amax(dim=1)
            scales[lo:lo + 4096] = torch.where(top > 0, top / 448.0, torch.ones_like(top))
        return [None, scales]
    p, g, m, v = (t.to(f64) for t in _adam_data(case, seed))
    lr, b1, b2, eps, wd = (float(np.float32(ADAM_HP[k])) for k in ("lr", "b1", "b2", "eps", "wd"))
    m = b1 * m + (1 - b1) * g
    v = b2 * v + (1 - b2) * g * g
    t = ADAM_HP["t"]
    step = (m / (1 - b1 ** t)) / (torch.sqrt(v / (1 - b2 ** t)) + eps) + wd * p
    return [p - lr * step, m, v]
