"""GPU: small calls whose last kernel tells the host that it is done, on both sides of that rule (16 workgroups): what the call has written is there for
another stream that nothing orders behind it, and the report is that of the call."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("T,E,k", [(1, 8, 2), (64, 8, 2), (512, 64, 8), (513, 64, 8), (256, 32, 9), (257, 32, 9), (500, 8, 1), (128, 128, 4), (1024, 64, 4), (1025, 64, 4)])
@pytest.mark.parametrize("assignment", ["exact", "iter"])
def test_outputs_are_there(T, E, k, assignment):
    import paper_2508_12801_amd as ms
    print(f"told ends T={T} E={E} k={k} {assignment}", flush=True)
    C = -(-5 * T * k // (4 * E))
    batches = []
    for seed in range(4):
        gen = torch.Generator(device="cuda").manual_seed(seed)
        scores = ms.softtopk(torch.randn(T, E, generator=gen, device="cuda") + torch.randn(E, generator=gen, device="cuda"), k, 1.0)[0]
        want = ms.route_scores(scores, k, C, assignment=assignment, allow_not_converged=True)
        torch.cuda.synchronize()
        a = want["assign"].long()
        assert torch.equal(want["gates"], scores.gather(1, a.clamp(min=0)) * (a >= 0))
        assert torch.equal(want["expert_offsets"].long().diff(), torch.bincount(a[a >= 0], minlength=E))
        batches.append((scores, want))
    names = ("assign", "gates", "expert_offsets", "disp_token", "disp_gate", "token_pos")
    other, keep = torch.cuda.Stream(), []
    for run in range(60):
        scores, want = batches[run % 4]
        got = ms.route_scores(scores, k, C, assignment=assignment, allow_not_converged=True)
        with torch.cuda.stream(other):               # (the call has waited: nothing else has to)
            seen = [got[n].clone() for n in names]
        keep.append((got, seen, want))
        assert got["stats"]["total_score_q"] == want["stats"]["total_score_q"] and got["stats"]["flow_value"] == want["stats"]["flow_value"]
        assert got["stats"]["rounds"] == want["stats"]["rounds"] and 0 < got["stats"]["gates_dispatch_ms"] < 1
    torch.cuda.synchronize()
    for got, seen, want in keep:
        n = int(want["expert_offsets"][-1])
        for name, x in zip(names, seen):
            y = want[name]
            assert torch.equal(x[:n], y[:n]) if name in ("disp_token", "disp_gate") else torch.equal(x, y)
