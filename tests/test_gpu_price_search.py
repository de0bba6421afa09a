"""GPU parity of the search behind the price passes where its lists change form: more exchanges in one block of rows than are
gathered in LDS and more within reach than are kept in registers, all nodes of the largest expert count with and without spare
capacity and with unfilled slots, tokens on several paths.  Optimality is the checker's certificate (or its optimum); the lists are
filled in no fixed order, so three runs have to give the same assignment."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SHAPES = [  # T, E, k, C, largest reward
    (20, 32, 8, 5, 1 << 20), (20, 32, 8, 5, 60), (25, 21, 10, 12, 1 << 20), (100, 9, 4, 45, 200),      # every exchange listed
    (1536, 512, 8, 24, 1 << 20), (1500, 512, 8, 24, 1 << 20), (3000, 256, 4, 47, 1 << 20), (1200, 257, 3, 14, 1 << 18),
    (1000, 64, 16, 250, 1 << 20), (3000, 24, 12, 1500, 1 << 20), (90, 30, 3, 8, 1 << 20),
]


@pytest.mark.parametrize("T,E,k,C,top", SHAPES)
def test_search(T, E, k, C, top):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2508_12801_amd as ms
    print(f"price search T={T} E={E} k={k} C={C} top={top}", flush=True)
    rng = np.random.default_rng(T * 31 + E + top)
    popular = rng.random(E) ** 3
    q = ((rng.random((T, E)) ** 2 + popular) / 2 * top).astype(np.int64)
    qd = torch.from_numpy(q.astype(np.int32)).cuda()
    runs = [ms.assign_i32(qd, k, C) for _ in range(3)]
    a = runs[0]["assign"].cpu().numpy()
    print(runs[0]["stats"], flush=True)
    for r in runs[1:]:
        assert np.array_equal(r["assign"].cpu().numpy(), a)
    filled = a >= 0
    total = int(np.take_along_axis(q, np.where(filled, a, 0).astype(np.int64), axis=1)[filled].sum())
    assert total == runs[0]["stats"]["total_score_q"] and int(filled.sum()) == min(T * k, E * C)
    if T * k <= E * C:
        P = oracle.assignment_matrix(a, E)
        assert (P.sum(axis=1) == k).all() and P.sum(axis=0).max() <= C and oracle.verify_optimal(q, P, k, C)["optimal"]
    else:
        assert np.bincount(a[filled], minlength=E).max() <= C
        assert total == oracle.assign_literal_graph(q, k, C)["total"]


@pytest.mark.parametrize("T,E,k,room", [(1000, 20, 2, 1.0), (1000, 20, 2, 0.75), (1500, 64, 6, 1.1), (1500, 64, 6, 1.0), (700, 100, 4, 1.05), (400, 24, 3, 0.8)])
def test_targets_out_of_reach(T, E, k, room):
    """Experts so uneven that searches find no target within the first reaches, and tries that end without one at any: the search
    goes on from the bound to all arcs at once, and the total is the optimum whichever try or solver ends with it."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2508_12801_amd as ms
    C = -int(-room * T * k // E)
    print(f"targets out of reach T={T} E={E} k={k} C={C}", flush=True)
    rng = np.random.default_rng(T + E)
    L = (rng.standard_normal((T, E)) + 2.0 * rng.standard_normal(E)).astype(np.float32)
    q = ms.softtopk(torch.from_numpy(L).cuda(), k, 1.0)[1]
    runs = [ms.assign_i32(q, k, C) for _ in range(2)]
    print(runs[0]["stats"], flush=True)
    assert torch.equal(runs[0]["assign"], runs[1]["assign"])
    a, qh = runs[0]["assign"].cpu().numpy(), q.cpu().numpy().astype(np.int64)
    filled = a >= 0
    total = int(np.take_along_axis(qh, np.where(filled, a, 0).astype(np.int64), axis=1)[filled].sum())
    assert total == runs[0]["stats"]["total_score_q"] and int(filled.sum()) == min(T * k, E * C)
    if room >= 1:
        P = oracle.assignment_matrix(a, E)
        assert (P.sum(axis=1) == k).all() and P.sum(axis=0).max() <= C and oracle.verify_optimal(qh, P, k, C)["optimal"]
    else:
        assert np.bincount(a[filled], minlength=E).max() <= C
        plain = ms.assign_i32(q, k, C, finisher=False)["stats"]
        assert (total, int(filled.sum())) == (plain["total_score_q"], plain["flow_value"])


@pytest.mark.parametrize("T,E,k,room,uneven", [(200, 16, 8, 1.0, 1.0), (1024, 256, 1, 1.0, 0.0), (600, 65, 5, 1.0, 1.5), (5623, 96, 2, 1.02, 1.5),
                                               (1300, 129, 6, 1.0, 1.0), (640, 160, 2, 0.9, 1.5), (1600, 512, 4, 1.0, 0.5)])
def test_moved_tokens_and_their_places(T, E, k, room, uneven):
    """Tokens that move more than once, in one search and in several: slots, lists, counts and positions are those of where they end,
    the reported total is the sum of their rewards, and the certificate holds with the exchanges that the list does not have."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2508_12801_amd as ms
    C = -int(-room * T * k // E)
    print(f"moved tokens T={T} E={E} k={k} C={C} uneven={uneven}", flush=True)
    rng = np.random.default_rng(T + 7 * E)
    L = (rng.standard_normal((T, E)) + uneven * rng.standard_normal(E)).astype(np.float32)
    r = ms.route_logits(torch.from_numpy(L).cuda(), k, C)
    print(r["stats"], flush=True)
    a, q = r["assign"].cpu().numpy(), r["q"].cpu().numpy().astype(np.int64)
    filled = a >= 0
    assert int(filled.sum()) == min(T * k, E * C) and np.bincount(a[filled], minlength=E).max() <= C
    assert int(np.take_along_axis(q, np.where(filled, a, 0).astype(np.int64), axis=1)[filled].sum()) == r["stats"]["total_score_q"]
    if room >= 1:
        st = r["stats"]                      # (an auction would end at the same optimum)
        assert (st["phases"], st["finish_passes"]) == (1, 1) and st["finish_cycles"] >= 5
        P = oracle.assignment_matrix(a, E)
        assert oracle.verify_optimal(q, P, k, C)["optimal"]
    d = oracle.dispatch(a, r["gates"].cpu().numpy(), E)
    for name in ("expert_offsets", "disp_token", "token_pos"):
        assert np.array_equal(r[name].cpu().numpy(), d[name]), name
