"""AdamW whose first chunk is loaded before the workgroup's trip is known
(barrier-free, uninstrumented) against the same program instrumented, which
loads it after its waits: equal bit for bit, also where workgroups have no
chunk, the last chunk is partial or the first chunk lies outside the vector."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2608_13757_amd import MODE_BARRIER_FREE, Plan, bfs  # noqa: E402
from tests.gpu_util import trip_tensors  # noqa: E402
from workloads import adamw_default_wg, adamw_program, adamw_worklist  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,chunk,n_wg", [(4, 256, 1), (4, 1024, 3), (1020, 512, 5), (4096, 1024, 4), (5000, 256, 7),
                                          (70000, 1024, 9)])
@pytest.mark.parametrize("ring", [1, 2, 4])
def test_adamw_ahead_equals_instrumented(n, chunk, n_wg, ring):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    bfs.lib()
    base, trips = adamw_worklist(n, chunk, n_wg)
    base = np.where(np.array([len(t[1]) and t[1][0] for t in trips.per_wg]) > 0, base, base + (1 << 40))
    t, off = trip_tensors(trips)
    plan = Plan(adamw_program(n, chunk, ring=ring), MODE_BARRIER_FREE)
    base = torch.from_numpy(base.astype(np.int64)).cuda()
    outs = []
    for cap in (0, 4):
        g = torch.Generator(device="cuda").manual_seed(n)
        p, grad, m = (torch.randn(n, generator=g, device="cuda") for _ in range(3))
        v = torch.rand(n, generator=g, device="cuda")
        log = torch.zeros(plan.debug_log_words(n_wg, cap), dtype=torch.int32, device="cuda") if cap else None
        plan.run([base, p, grad, m, v], t, off, n_wg, debug_log=log, debug_capacity=cap)
        plan.status()
        outs.append((p, m, v))
    for a, b in zip(*outs):
        assert torch.isfinite(a).all() and torch.equal(a, b)


@pytest.mark.parametrize("n", [(40 << 16) + 4, 1 << 24, (40 << 16), (1 << 24) + 4])
def test_adamw_store_kinds_equal_instrumented(n):
    """Vectors just inside and just outside the sizes whose results are stored
    through the caches: the same bits as the instrumented launch."""
    test_adamw_ahead_equals_instrumented(n, 1024, adamw_default_wg(n, 1024), 2)
