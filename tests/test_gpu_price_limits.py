"""GPU: batches whose price solves end in their first try, or at all, by the limits of their class: more than 256 experts, few experts with a price
among many with room, few places per expert, rows that are nearly alike.  (With one limit and one number of exchanges for all of them the first went into a second try or to
the auction, 1.5 to 12 times as long.)  Totals of the smaller ones are the auction's."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _logits(T, E, kind, alike, noise, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    L = torch.randn(T, E, generator=gen, device="cuda")
    if kind == "normal":
        L += 0.7 * torch.randn(E, generator=gen, device="cuda")
    elif kind == "zipf":
        w = torch.arange(1, E + 1, device="cuda", dtype=torch.float64) ** -1.2
        L += (2 * (w - w[-1]) / (w[0] - w[-1]))[torch.randperm(E, generator=gen, device="cuda")].float()
    n = int(T * alike)
    if n:
        L[:n] = L[0] + noise * torch.randn(n, E, generator=gen, device="cuda")
    return L


@pytest.mark.parametrize("T,E,k,room,kind,alike,noise,seed,most", [
    (4096, 512, 8, 0.75, "zipf", 0, 0, 2512, 1), (10007, 512, 8, 1.1, "none", 0, 0, 512, 1), (16384, 512, 8, 1.1, "none", 0, 0, 512, 1),
    (16384, 512, 2, 1.1, "zipf", 0, 0, 2512, 1),
    (10007, 128, 2, 1.5, "zipf", 0, 0, 2128, 1), (32768, 128, 2, 1.5, "zipf", 0, 0, 2128, 1), (16384, 160, 2, 1.1, "zipf", 0, 0, 2160, 1),
    (65536, 256, 2, 1.1, "zipf", 0, 0, 2256, 1),
    (64, 128, 8, 0.75, "none", 0, 0, 0, 1), (64, 128, 8, 0.75, "normal", 0, 0, 1, 1), (64, 128, 8, 1.0, "none", 0, 0, 5, 1),
    (4096, 64, 4, 1.0, "normal", 0.1, 0.03, 1064, 3), (4096, 256, 4, 1.2, "none", 0.1, 0.03, 256, 3), (16384, 64, 4, 0.8, "normal", 0.5, 0.1, 1064, 3),
    (16384, 128, 4, 1.0, "none", 0.05, 0.03, 128, 3),
])
def test_price_solves_stand(T, E, k, room, kind, alike, noise, seed, most):
    import paper_2508_12801_amd as ms
    print(f"price limits T={T} E={E} k={k} room={room} {kind} alike={alike}", flush=True)
    C = min(T, -int(-room * T * k // E))
    q = ms.softtopk(_logits(T, E, kind, alike, noise, seed), k, 1.0)[1]
    a = ms.assign_i32(q, k, C)
    tries = ms.solve_account()["tries"]
    print(tries, a["stats"], flush=True)
    assert 1 <= tries <= most
    if T <= 4096:
        assert a["stats"]["total_score_q"] == ms.assign_i32(q, k, C, finisher=False)["stats"]["total_score_q"]
