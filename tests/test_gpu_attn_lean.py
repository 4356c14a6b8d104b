"""Attention, barrier-free and uninstrumented (joined and split waits, stores
of S under the MFMAs), against the same program instrumented (every wait of an
instruction before its effects): the arithmetic is the same, so the outputs are
equal bit for bit.  (The instrumented run against the fp64 oracle is
test_gpu_attn.py's.)"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2608_13757_amd import ALLOC_PER_INSTR, ALLOC_PER_LOOP, MODE_BARRIER_FREE, Plan, bfs  # noqa: E402
from tests.gpu_util import trip_tensors  # noqa: E402
from workloads import attn_program, attn_worklist  # noqa: E402

pytestmark = pytest.mark.gpu

# one key, the edges of 64-key blocks and 128-query tiles, one to many steps
RAGGED = [1, 63, 64, 65, 127, 128, 129, 200, 321, 777]


def _compare(program, lengths, heads, n_wg, alloc):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    bfs.lib()
    g = torch.Generator(device="cuda").manual_seed(3)
    tokens = sum(lengths)
    q, k, v = (torch.randn(tokens, heads, 128, generator=g, device="cuda").to(torch.bfloat16) for _ in range(3))
    wl = attn_worklist(np.array(lengths), heads, n_wg=n_wg)
    trips, toff = trip_tensors(wl.trips)
    work = torch.from_numpy(wl.work.reshape(-1)).cuda()
    plan = Plan(program, MODE_BARRIER_FREE, alloc)
    outs = []
    for cap in (0, 4):
        out = torch.full((tokens, heads, 128), -1, dtype=torch.int16, device="cuda")
        log = torch.zeros(plan.debug_log_words(wl.trips.n_wg, cap), dtype=torch.int32, device="cuda") if cap else None
        plan.run([work, q, k, v, out], trips, toff, wl.trips.n_wg, debug_log=log, debug_capacity=cap,
                 watchdog_polls=20_000_000)
        plan.status()
        outs.append(out)
    assert torch.isfinite(outs[1].view(torch.bfloat16).float()).all()
    assert torch.equal(outs[0], outs[1])
    return outs[0]


@pytest.mark.parametrize("alloc", [ALLOC_PER_LOOP, ALLOC_PER_INSTR])
@pytest.mark.parametrize("linear", [False, True])
@pytest.mark.parametrize("rings", [(2, 2), (2, 3), (3, 2)])
@pytest.mark.parametrize("lengths,heads,n_wg", [(RAGGED, 2, 256), (RAGGED, 3, 5), ([1], 1, 8), ([2000], 1, 1)])
def test_attn_lean_equals_instrumented(lengths, heads, n_wg, rings, linear, alloc):
    _compare(attn_program(heads, nk=rings[0], nv=rings[1], linear=linear), lengths, heads, n_wg, alloc)


@pytest.mark.parametrize("alloc", [ALLOC_PER_LOOP, ALLOC_PER_INSTR])
@pytest.mark.parametrize("linear", [False, True])
@pytest.mark.parametrize("lengths,heads,n_wg", [(RAGGED, 3, 5), ([1], 1, 8)])
def test_attn_v_load_after_pread(lengths, heads, n_wg, linear, alloc):
    """A program whose V load waits for the step's PREAD, so that PREAD cannot
    wait with PV: the same bits as the program without that wait."""
    p = attn_program(heads, linear=linear)
    kv = next(b for b in p.blocks if p.instr_id("LOADV") in b)
    kv.insert(kv.index(p.instr_id("PREAD")), kv.pop(kv.index(p.instr_id("LOADV"))))
    order = [i for b in p.blocks for i in b]
    new = {old: i for i, old in enumerate(order)}
    p.instrs = [p.instrs[i] for i in order]
    p.blocks = [[new[i] for i in b] for b in p.blocks]
    p.deps = [(new[a], new[c], k) for a, c, k in p.deps] + [(p.instr_id("PREAD"), p.instr_id("LOADV"), 0)]
    p.dep_linear = p.dep_linear + [0]
    out = _compare(p, lengths, heads, n_wg, alloc)
    assert torch.equal(out, _compare(attn_program(heads, linear=linear), lengths, heads, n_wg, alloc))
