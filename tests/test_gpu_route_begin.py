"""GPU: price passes begun ahead of the call that solves the batch.  They are used by that call alone: with other rewards, behind another
solve or behind rerouting, the call solves the batch as if nothing had been begun, and passes that are given up disturb neither."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("between", ["nothing", "other rewards", "another solve", "rerouting", "other sizes"])
@pytest.mark.parametrize("T,E,k,C", [(64, 8, 2, 16), (512, 128, 8, 40), (512, 64, 8, 48), (513, 64, 8, 80), (300, 16, 9, 200), (5000, 64, 8, 625),
                                     (140000, 8, 2, 35000)])
def test_begun_passes(T, E, k, C, between):
    import paper_2508_12801_amd as ms
    from paper_2508_12801_amd import binding as b
    print(f"route begin T={T} E={E} k={k} C={C} {between}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(T + E)
    scores, q = ms.softtopk(torch.randn(T, E, generator=gen, device="cuda") + 0.5 * torch.randn(E, generator=gen, device="cuda"), k, 1.0)
    other = ms.softtopk(torch.randn(T, E, generator=gen, device="cuda"), k, 1.0)[1]
    want, want_other = ms.assign_i32(q, k, C), ms.assign_i32(other, k, C)
    ws, need = b._workspace(T, E, k, C, q.device)
    opts, begun, stats = b._opts(), ctypes.c_int32(7), b.Stats()
    lib = b.load_library()
    assert lib.maxscore_route_begin(b._ptr(q), T, E, k, C, ctypes.byref(opts), ctypes.byref(begun), b._ptr(ws), need, b._stream()) == 0
    assert begun.value == 1
    opts.flags |= b.FLAG_PASSES_BEGUN
    if between == "another solve":
        assert torch.equal(ms.assign_i32(other, k, C)["assign"], want_other["assign"])
    if between == "rerouting":
        first, again = (ms.assign_iter_i32(other, k, C, allow_not_converged=True) for _ in range(2))
        assert torch.equal(first["assign"], again["assign"]) and first["total"] == again["total"]
    use, C_use = (other, C) if between == "other rewards" else (q, C + 1) if between == "other sizes" else (q, C)
    if between == "other rewards":
        want = want_other
    elif between == "other sizes":
        want = ms.assign_i32(q, k, C_use)
    o = b._route_outputs(T, E, k, q.device, dict(scores=scores, q=use))
    for run in range(2):                 # (the second time there is nothing begun)
        rc = lib.maxscore_route_rewards(
            b._ptr(scores), b._ptr(use), T, E, k, C_use, ctypes.byref(opts), b._ptr(o["assign"]), b._ptr(o["gates"]), b._ptr(o["expert_offsets"]),
            b._ptr(o["disp_token"]), b._ptr(o["disp_gate"]), b._ptr(o["token_pos"]), b._ptr(o["prices"]), ctypes.byref(stats), b._ptr(ws), need, b._stream())
        assert ms.solve_account()["begun"] == (run == 0 and between == "nothing")
        assert rc == 0 and stats.total_score_q == want["stats"]["total_score_q"] and stats.rounds == want["stats"]["rounds"]
        assert torch.equal(o["assign"], want["assign"]) and torch.equal(o["prices"], want["prices"])
        held = o["assign"].long()
        assert torch.equal(o["gates"], torch.where(held >= 0, scores.gather(1, held.clamp(min=0)), torch.zeros(1, device="cuda")))


def test_nothing_is_begun_without_a_price_solve():
    import paper_2508_12801_amd as ms
    from paper_2508_12801_amd import binding as b
    q = torch.randint(0, 1 << 20, (64, 8), dtype=torch.int32, device="cuda")
    ws, need = b._workspace(64, 8, 2, 16, q.device)
    lib, begun = b.load_library(), ctypes.c_int32(7)

    def begin(opts, k=2, rc=0, size=need):
        assert lib.maxscore_route_begin(b._ptr(q), 64, 8, k, 16, ctypes.byref(opts), ctypes.byref(begun), b._ptr(ws), size, b._stream()) == rc
        return begun.value

    assert begin(b._opts(finisher=False)) == 0 and begin(b._opts(max_rounds=10)) == 0 and begin(b._opts(assignment="iter")) == 0
    assert begin(b._opts(), k=9, rc=-2) == 0 and begin(b._opts(), size=16, rc=-3) == 0
    ms.set_kernel_timing(True)
    try:
        assert begin(b._opts()) == 0
    finally:
        ms.set_kernel_timing(False)
    assert begin(b._opts()) == 1
    torch.cuda.synchronize()


def test_given_up_in_another_stream():
    """Passes that are given up run beside the thread's next solve, in a stream and a workspace of their own, and tell of themselves meanwhile."""
    import paper_2508_12801_amd as ms
    from paper_2508_12801_amd import binding as b
    shapes = [(3000, 64, 8, 375), (5000, 64, 8, 800), (4096, 16, 2, 512), (700, 16, 2, 100)]
    a, c, keep = torch.cuda.Stream(), torch.cuda.Stream(), []
    lib = b.load_library()
    for round_, (T, E, k, C) in enumerate(shapes * 3):
        print(f"two streams {round_} T={T} E={E} k={k} C={C}", flush=True)
        gen = torch.Generator(device="cuda").manual_seed(round_)
        q, other = (ms.softtopk(torch.randn(T, E, generator=gen, device="cuda") + torch.randn(E, generator=gen, device="cuda"), k, 1.0)[1] for _ in range(2))
        want = ms.assign_i32(other, k, C)
        torch.cuda.synchronize()
        for given_up in range(1 + round_ % 3):
            with torch.cuda.stream(a):
                ws, need = b._workspace(T, E, k, C, q.device)
                opts, begun = b._opts(), ctypes.c_int32()
                assert lib.maxscore_route_begin(b._ptr(q), T, E, k, C, ctypes.byref(opts), ctypes.byref(begun), b._ptr(ws), need, b._stream()) == 0
                assert begun.value == 1
                keep += [q, ws]
        with torch.cuda.stream(c):
            got = ms.assign_i32(other, k, C)
        torch.cuda.synchronize()
        assert got["stats"]["total_score_q"] == want["stats"]["total_score_q"] and got["stats"]["rounds"] == want["stats"]["rounds"]
        assert torch.equal(got["assign"], want["assign"]) and torch.equal(got["prices"], want["prices"])
