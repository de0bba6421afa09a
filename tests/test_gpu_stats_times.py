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


@pytest.mark.parametrize("T,E,k,C", [(64, 8, 2, 16), (500, 64, 8, 80), (700, 16, 2, 88), (4096, 16, 2, 512), (4096, 64, 8, 4096)])
def test_time_between_the_two_calls_is_no_time_of_the_solve(T, E, k, C):
    """Passes begun ahead of a call that comes much later: the device time of the solve is that of its kernels."""
    import ctypes

    import paper_2508_12801_amd as ms
    from paper_2508_12801_amd import binding as b
    print(f"pause T={T} E={E} k={k} C={C}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(T)
    scores, q = ms.softtopk(torch.randn(T, E, generator=gen, device="cuda") + 0.5 * torch.randn(E, generator=gen, device="cuda"), k, 1.0)
    ws, need = b._workspace(T, E, k, C, q.device)
    lib, opts, begun, stats = b.load_library(), b._opts(), ctypes.c_int32(), b.Stats()
    o = b._route_outputs(T, E, k, q.device, dict(scores=scores, q=q))
    for pause in (0.0, 0.05):
        opts.flags = 0
        assert lib.maxscore_route_begin(b._ptr(q), T, E, k, C, ctypes.byref(opts), ctypes.byref(begun), b._ptr(ws), need, b._stream()) == 0 and begun.value
        torch.cuda.synchronize()
        time.sleep(pause)
        opts.flags |= b.FLAG_PASSES_BEGUN
        t = time.perf_counter()
        assert lib.maxscore_route_rewards(
            b._ptr(scores), b._ptr(q), T, E, k, C, ctypes.byref(opts), b._ptr(o["assign"]), b._ptr(o["gates"]), b._ptr(o["expert_offsets"]),
            b._ptr(o["disp_token"]), b._ptr(o["disp_gate"]), b._ptr(o["token_pos"]), b._ptr(o["prices"]), ctypes.byref(stats), b._ptr(ws), need, b._stream()) == 0
        took = (time.perf_counter() - t) * 1e3
        assert ms.solve_account()["begun"] == 1
        print(stats.solver_ms, took, flush=True)
        assert 0 < stats.solver_ms < 1.0          # (with the pause in it 50)
