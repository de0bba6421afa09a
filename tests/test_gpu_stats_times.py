"""GPU: the device times that a routing call reports."""
import time

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("assignment", ["exact", "iter"])
@pytest.mark.parametrize("T,E,k", [(64, 8, 2), (700, 16, 2), (5000, 64, 8), (44032, 64, 2), (3000, 32, 20)])
def test_gates_and_dispatch_have_a_time(T, E, k, assignment):
    import paper_2508_12801_amd as ms
    print(f"times T={T} E={E} k={k} {assignment}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(T)
    L = torch.randn(T, E, generator=gen, device="cuda") + torch.randn(E, generator=gen, device="cuda")
    for _ in range(4):
        torch.cuda.synchronize()
        t = time.perf_counter()
        stats = ms.route_logits(L, k, -(-T * k // E), assignment=assignment, allow_not_converged=True)["stats"]
        took = (time.perf_counter() - t) * 1e3
        assert 0 < stats["gates_dispatch_ms"] < took
