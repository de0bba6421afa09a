"""GPU parity of the price solve at the edges of its launch shapes: lanes per row and columns per lane change at powers of
two of E and k, small batches run in one workgroup, large ones start on a sample of their rows; capacity tight, nearly
tight, spare and short, and as many slots as experts.  Optimality is the checker's certificate, or for a short capacity
the checker's optimum (small sizes) or the padded auction's total; dispatch comes from the checker's lists."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SHAPES = [  # T, E, k, C
    (1, 2, 1, 1), (65, 2, 2, 65), (64, 8, 8, 64), (9, 17, 3, 2), (129, 63, 8, 17), (512, 64, 8, 64), (513, 65, 9, 72),
    (300, 65, 1, 5), (257, 128, 33, 67), (31, 129, 2, 1), (255, 255, 4, 4), (256, 257, 16, 20), (2049, 512, 2, 9),
    (100, 48, 1, 3), (600, 16, 4, 150), (600, 16, 4, 188), (600, 16, 4, 113), (40, 20, 4, 6), (2048, 96, 6, 96),
    (16383, 32, 2, 1024), (16384, 32, 2, 1024), (16385, 33, 1, 500), (16390, 33, 1, 620), (16400, 31, 2, 800),
]


@pytest.fixture(scope="module")
def ms():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2508_12801_amd as m
    m.load_library()
    return m


@pytest.mark.parametrize("T,E,k,C", SHAPES)
def test_edges(ms, T, E, k, C):
    print(f"price edges T={T} E={E} k={k} C={C}", flush=True)
    rng = np.random.default_rng(T + E)
    L = (rng.standard_normal((T, E)) + 0.5 * rng.standard_normal(E)).astype(np.float32)
    out = ms.route_logits(torch.from_numpy(L).cuda(), k, C)
    q = out["q"].cpu().numpy().astype(np.int64)
    a = out["assign"].cpu().numpy()
    filled = a >= 0
    total = int(np.take_along_axis(q, np.where(filled, a, 0).astype(np.int64), axis=1)[filled].sum())
    assert total == out["stats"]["total_score_q"] and int(filled.sum()) == out["stats"]["flow_value"]
    assert np.bincount(a[filled], minlength=E).max() <= min(C, T)
    if T * k <= E * C:
        P = oracle.assignment_matrix(a, E)
        assert (P.sum(axis=1) == k).all() and oracle.verify_optimal(q, P, k, C)["optimal"]
    elif T <= 100:
        assert total == oracle.assign_literal_graph(q, k, C)["total"]
    else:
        plain = ms.assign_i32(out["q"], k, C, finisher=False)["stats"]
        assert (total, int(filled.sum())) == (plain["total_score_q"], plain["flow_value"])
    want = oracle.dispatch(a, out["gates"].cpu().numpy(), E)
    n = int(filled.sum())
    assert np.array_equal(out["expert_offsets"].cpu().numpy(), want["expert_offsets"])
    assert np.array_equal(out["disp_token"].cpu().numpy()[:n], want["disp_token"][:n])
    assert np.array_equal(out["token_pos"].cpu().numpy(), want["token_pos"])


@pytest.mark.parametrize("T,E,k,room,uneven", [(300, 2, 1, 1.3, 3.0), (500, 8, 2, 1.01, 1.5), (64, 64, 8, 1.1, 1.0), (2000, 65, 3, 1.002, 1.0),
                                               (1500, 96, 6, 1.1, 2.0), (1200, 256, 4, 2.0, 1.0), (1100, 257, 2, 1.25, 1.0), (900, 512, 1, 1.5, 0.7),
                                               (4099, 16, 2, 1.25, 0.0)])
def test_spare_room(ms, T, E, k, room, uneven):
    """The level of the prices with next to no, some and much spare capacity, experts as popular as each other and not: the optimum, and
    started from the prices it ended with the same one."""
    C = min(T, -int(-room * T * k // E))
    print(f"spare room T={T} E={E} k={k} C={C} uneven={uneven}", flush=True)
    rng = np.random.default_rng(T + E + k)
    L = (rng.standard_normal((T, E)) + uneven * rng.standard_normal(E)).astype(np.float32)
    out = ms.route_logits(torch.from_numpy(L).cuda(), k, C)
    q = out["q"].cpu().numpy().astype(np.int64)
    a = out["assign"].cpu().numpy()
    P = oracle.assignment_matrix(a, E)
    assert (P.sum(axis=1) == k).all() and P.sum(axis=0).max() <= C and oracle.verify_optimal(q, P, k, C)["optimal"]
    if E < 512:
        assert (out["stats"]["phases"], out["stats"]["finish_passes"]) == (1, 1)         # not by the auction
    again = ms.assign_i32(out["q"], k, C, prices_in=out["prices"])
    assert again["stats"]["total_score_q"] == out["stats"]["total_score_q"]


@pytest.mark.parametrize("T", [131071, 131072, 131080])
@pytest.mark.parametrize("C", [32768, 36000, 25000])
def test_first_sampled_batches(ms, T, C):
    """Where the first two passes begin to look at a sample of the rows: the auction's totals."""
    print(f"sampled passes T={T} C={C}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(T + C)
    L = torch.randn(T, 8, generator=gen, device="cuda") + torch.randn(8, generator=gen, device="cuda")
    q = ms.softtopk(L, 2, 1.0)[1]
    got, plain = ms.assign_i32(q, 2, C)["stats"], ms.assign_i32(q, 2, C, finisher=False)["stats"]
    assert (got["total_score_q"], got["flow_value"]) == (plain["total_score_q"], plain["flow_value"])


@pytest.mark.parametrize("seed", [0, 1, 2, 3])
def test_near_copies_with_spare_room(ms, seed):
    """A quarter of the rows alike but for a little noise, a quarter more room than demand: the price solve has to get there itself (the
    auction takes some 50 rounds), at the optimum that the auction finds."""
    print(f"near copies with spare room seed={seed}", flush=True)
    from workloads import CONFIGS, make_logits
    c = CONFIGS["cfg4b_near"]
    q = ms.softtopk(torch.from_numpy(make_logits("cfg4b_near", seed)).cuda(), c["k"], c["t"])[1]
    st = ms.assign_i32(q, c["k"], c["C"])["stats"]
    auction = ms.assign_i32(q, c["k"], c["C"], finisher=False)["stats"]
    assert st["total_score_q"] == auction["total_score_q"] and st["rounds"] <= 14
    assert (st["phases"], st["finish_passes"]) == (1, 1)               # not by the auction


@pytest.mark.parametrize("k,noise,passes", [(4, 0.1, 14), (8, 0.1, 12), (2, 0.1, 15)])
def test_few_near_copies_with_spare_room(ms, k, noise, passes):
    """A tenth of the rows alike, many experts: the steps of both kinds, at the auction's optimum."""
    print(f"few near copies k={k} noise={noise}", flush=True)
    T, E = 16384, 256
    gen = torch.Generator(device="cuda").manual_seed(7)
    logits = torch.randn(T, E, generator=gen, device="cuda")
    n = T // 10
    logits[:n] = logits[0] + noise * torch.randn(n, E, generator=gen, device="cuda")
    q = ms.softtopk(logits, k, 1.0)[1]
    C = -(-5 * T * k // (4 * E))
    st = ms.assign_i32(q, k, C)["stats"]
    auction = ms.assign_i32(q, k, C, finisher=False)["stats"]
    assert st["total_score_q"] == auction["total_score_q"]
    assert (st["phases"], st["finish_passes"]) == (1, 1) and st["rounds"] <= passes


@pytest.mark.parametrize("T,E,k,C", [(64, 8, 2, 20), (96, 6, 1, 18), (500, 8, 3, 200), (900, 33, 2, 60), (2000, 257, 1, 9), (131080, 8, 2, 36000)])
def test_copies_on_the_edges(ms, T, E, k, C):
    """Half the rows alike up to 3e-2 where the steps' tables are at their edges: passes of one workgroup, column counts off the pieces, bins
    of one an octave, sampled passes."""
    print(f"copies on the edges T={T} E={E} k={k} C={C}", flush=True)
    rng = np.random.default_rng(T + E)
    L = rng.standard_normal((T, E)).astype(np.float32)
    L[: T // 2] = L[0] + 0.03 * rng.standard_normal((T // 2, E)).astype(np.float32)
    q = ms.softtopk(torch.from_numpy(L).cuda(), k, 1.0)[1]
    out, plain = ms.assign_i32(q, k, C), ms.assign_i32(q, k, C, finisher=False)
    assert out["stats"]["total_score_q"] == plain["stats"]["total_score_q"]
    a = out["assign"].cpu().numpy()
    assert (a >= 0).all() and np.bincount(a.ravel(), minlength=E).max() <= C and (np.diff(np.sort(a, axis=1), axis=1) > 0).all()


@pytest.mark.parametrize("T,E,k,room,part,noise", [(16384, 64, 8, 1.0, 0.5, 0.1), (16384, 64, 8, 1.0, 0.1, 0.03), (16384, 64, 8, 0.75, 0.25, 0.03),
                                                   (16384, 256, 8, 1.0, 0.5, 0.1), (4096, 16, 2, 1.0, 0.25, 0.03)])
def test_near_copies_without_spare_room(ms, T, E, k, room, part, noise):
    """Rows that are nearly alike where capacity is tight or short: the passes that follow the usual six bring the prices near enough for
    the search, and the optimum is the auction's."""
    print(f"near copies T={T} E={E} k={k} room={room} part={part} noise={noise}", flush=True)
    rng = np.random.default_rng(7)
    logits = rng.standard_normal((T, E)).astype(np.float32)
    n = int(T * part)
    logits[:n] = logits[0] + noise * rng.standard_normal((n, E)).astype(np.float32)
    q = ms.softtopk(torch.from_numpy(logits).cuda(), k, 1.0)[1]
    C = int(T * k / E * room)
    st = ms.assign_i32(q, k, C)["stats"]
    auction = ms.assign_i32(q, k, C, finisher=False)["stats"]
    assert st["total_score_q"] == auction["total_score_q"] and st["rounds"] < 24
    assert (st["phases"], st["finish_passes"]) == (1, 1)


@pytest.mark.parametrize("T,E,k,C,part,noise,scale,seed", [(2945, 4, 2, 1915, 0.5, 0.1, 3.0, 244), (3510, 4, 2, 2282, 0.8, 0.1, 3.0, 60),
                                                           (2240, 8, 1, 283, 0.8, 0.1, 3.0, 400), (12875, 4, 1, 3251, 0.1, 0.1, 3.0, 423),
                                                           (2346, 6, 3, 1525, 0.8, 0.1, 1.0, 330)])
def test_few_experts_with_a_price(ms, T, E, k, C, part, noise, scale, seed):
    """Near copies to few experts, of which one or two have a price: a step of these together by their own mean demand alone finds nothing to
    do while they have room, and the auction had to solve these."""
    print(f"few experts T={T} E={E} k={k} C={C} part={part} noise={noise}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    L = torch.randn(T, E, generator=gen, device="cuda") * scale
    n = int(T * part)
    L[:n] = L[0] + noise * torch.randn(n, E, generator=gen, device="cuda")
    q = ms.softtopk(L, k, 1.0)[1]
    st, auction = ms.assign_i32(q, k, C)["stats"], ms.assign_i32(q, k, C, finisher=False)["stats"]
    assert st["total_score_q"] == auction["total_score_q"]
    assert (st["phases"], st["finish_passes"]) == (1, 1)               # not by the auction


@pytest.mark.parametrize("T,E,k,C,seed,passes", [(150000, 96, 6, 10313, 9, 12), (524288, 64, 2, 20480, 8, 13)])
def test_samples_before_all_rows(ms, T, E, k, C, seed, passes):
    """Spare room beyond 131071 tokens: what the passes over samples leave the first pass over all rows finds, which must not be taken for
    rows that are nearly alike."""
    print(f"samples before all rows T={T} E={E} k={k}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    L = torch.randn(T, E, generator=gen, device="cuda") + 0.7 * torch.randn(E, generator=gen, device="cuda")
    q = ms.softtopk(L, k, 1.0)[1]
    st, auction = ms.assign_i32(q, k, C)["stats"], ms.assign_i32(q, k, C, finisher=False)["stats"]
    assert st["total_score_q"] == auction["total_score_q"]
    assert (st["phases"], st["finish_passes"]) == (1, 1) and st["rounds"] <= passes
