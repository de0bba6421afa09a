"""GPU: the last pass of small batches, made by the workgroup that searches.  Sizes on both sides of its rule (8192 rewards, eight slots, 128
experts), rows that end in the middle of a block or a wavefront, columns beside whole loads, every relation of demand and capacity, and rows that are
all alike (every exchange is listed, or too many are).  Totals are the auction's, and with more demand than capacity the CPU checker's; the lists and
positions, which come from its counts, fit the assignment."""
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("room", [0.75, 1.0, 1.3])
@pytest.mark.parametrize("T,E,k", [(3, 2, 1), (33, 7, 2), (64, 8, 2), (64, 128, 8), (65, 127, 8), (128, 64, 5), (129, 63, 8), (129, 64, 8), (512, 16, 1), (482, 17, 3),
                                   (511, 8, 8), (1280, 8, 2), (100, 16, 9), (64, 129, 4)])
def test_small_last_pass(T, E, k, room):
    import paper_2508_12801_amd as ms
    print(f"last pass T={T} E={E} k={k} room={room}", flush=True)
    if k == E and room < 1:
        pytest.skip("every token takes every expert")
    C = min(T, max(1, -int(-room * T * k // E)))
    for seed, alike in enumerate((0.0, 0.0, 0.3, 1.0)):
        gen = torch.Generator(device="cuda").manual_seed(100 * T + seed)
        L = torch.randn(T, E, generator=gen, device="cuda") + 0.7 * torch.randn(E, generator=gen, device="cuda")
        n = int(T * alike)
        if n:
            L[:n] = L[0] + 1e-3 * torch.randn(n, E, generator=gen, device="cuda")
        scores, q = ms.softtopk(L, k, 1.0)
        over = T * k > E * C
        want = oracle.assign_literal_graph(q.cpu().numpy(), k, C)["total"] if over else ms.assign_i32(q, k, C, finisher=False)["stats"]["total_score_q"]
        r, again = ms.route_scores(scores, k, C), ms.route_scores(scores, k, C)
        tries = ms.solve_account()["tries"]
        # by prices, not by the auction: what the price solve takes, of rows that are not alike
        assert alike or tries > 0 or (E > 64 and T * k < 3 * E)
        a, off = r["assign"].long(), r["expert_offsets"].long()
        held = torch.where(a >= 0, q.long().gather(1, a.clamp(min=0)), torch.zeros_like(a))
        assert r["stats"]["total_score_q"] == int(held.sum()) and r["stats"]["flow_value"] == int((a >= 0).sum()) == min(T * k, E * C)
        assert r["stats"]["total_score_q"] == again["stats"]["total_score_q"] == want
        assert alike or torch.equal(r["assign"], again["assign"])          # (rows alike may come to the auction, which takes any of the best)
        counts = torch.bincount(a[a >= 0], minlength=E)
        assert int(counts.max()) <= C and torch.equal(off[1:] - off[:-1], counts)
        for e in range(E):
            mine = r["disp_token"][off[e]:off[e + 1]].long()
            assert torch.equal(mine.sort().values, (a == e).any(1).nonzero().flatten())
