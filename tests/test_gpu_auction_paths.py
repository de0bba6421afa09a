"""GPU parity of the auction, its tail pass and its finisher.  Calls with one capacity for all experts are price solves as a rule, so
the auction is reached here in the two ways a caller reaches it: with a capacity per expert (all equal, so that the scalar problem
is the reference), and with rewards too wide for the price solve's keys, whose tries then end in the auction."""
import ctypes

import numpy as np
import pytest

import oracle
from workloads import CONFIGS, capacity, make_logits

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

@pytest.fixture(scope="module")
def ms():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2508_12801_amd as m
    m.load_library()
    return m


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def auction(ms, q64, k, C, **opts):
    """maxscore_assign_caps_i32 with C for every expert, and all options of the scalar entry point."""
    from paper_2508_12801_amd import binding as b
    T, E = q64.shape
    q = dev(q64.astype(np.int32))
    caps = (ctypes.c_int32 * E)(*[C] * E)
    assign = torch.empty((T, k), dtype=torch.int32, device="cuda")
    prices = torch.empty(E, dtype=torch.int64, device="cuda")
    scale = torch.empty(1, dtype=torch.int64, device="cuda")
    need = ms.workspace_bytes(T, 0, E, k, 1)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    st, o = b.Stats(), b._opts(**opts)
    rc = ms.load_library().maxscore_assign_caps_i32(q.data_ptr(), T, E, k, ctypes.addressof(caps), ctypes.byref(o), assign.data_ptr(),
                                                    prices.data_ptr(), scale.data_ptr(), ctypes.byref(st), ws.data_ptr(), need,
                                                    torch.cuda.current_stream().cuda_stream)
    assert rc == 0, rc
    return dict(assign=assign, prices=prices, price_scale=int(scale.item()), stats=st.as_dict())


def check(q, out, k, C, total):
    """The given total, a feasible assignment, and prices that certify it: complementary slackness within one unit of the scaled
    rewards, price 0 on experts with room."""
    T, E = q.shape
    P = oracle.assignment_matrix(out["assign"].cpu().numpy(), E)
    ok, why = oracle.check_feasible(P, k, C)
    assert ok, why
    P = P.astype(bool)
    assert int(q[P].sum()) == out["stats"]["total_score_q"] == total, out["stats"]
    p = out["prices"].cpu().numpy()
    assert (p >= 0).all() and (p[P.sum(axis=0) < min(C, T)] == 0).all()
    net, big = q * out["price_scale"] - p[None, :], np.int64(1) << 60
    assert (np.where(P, net, big).min(axis=1) >= np.where(P, -big, net).max(axis=1) - 1).all()


def instance(name, T, seed, slack=0):
    cfg = CONFIGS[name]
    E, k = cfg["E"], cfg["k"]
    q = oracle.quantise(oracle.soft_topk(make_logits(name, seed=seed, T=T), k, cfg["t"]))
    C = capacity(T, E, k, cfg["C"] * E / (cfg["T"] * k)) + slack
    return q, k, C


@pytest.mark.parametrize("eps_div", [2, 5, 64])
@pytest.mark.parametrize("hi_bits", [12, 21, 27])
def test_eps_schedule_and_value_width(ms, eps_div, hi_bits):
    print(f"auction eps_div {eps_div} bits {hi_bits}", flush=True)
    rng = np.random.default_rng(9 + hi_bits)
    L = rng.normal(size=(1024, 32)) + 2.0 * rng.normal(size=(1, 32))
    p = np.exp(L - L.max(axis=1, keepdims=True))
    q = np.rint(p / p.sum(axis=1, keepdims=True) * ((1 << hi_bits) - 1)).astype(np.int64)
    total = oracle.max_score_assignment(q, 4, 128)["total"]
    rounds = [auction(ms, q, 4, 128, eps_div=d, finisher=False)["stats"]["rounds"] for d in (eps_div, 12)]
    assert rounds[0] != rounds[1]                          # the schedule did change something
    check(q, auction(ms, q, 4, 128, eps_div=eps_div), 4, 128, total)


@pytest.mark.parametrize("T,E,k,slack", [(4096, 64, 8, 0), (4096, 160, 5, 0), (3072, 200, 8, 3), (2048, 256, 8, 0), (4096, 512, 4, 2),
                                        (2560, 640, 5, 0), (2048, 1000, 8, 1)])
def test_tail_pass_and_finisher(ms, T, E, k, slack):
    """Every size class of both: the same optimum with and without them, and either saves rounds or at least runs."""
    print(f"auction tail and finisher T={T} E={E} k={k}", flush=True)
    rng = np.random.default_rng(E + 7 * k)
    L = rng.normal(size=(T, E)) + 2.0 * rng.normal(size=(1, E))
    p = np.exp(L - L.max(axis=1, keepdims=True))
    q = np.rint(p / p.sum(axis=1, keepdims=True) * ((1 << 20) - 1)).astype(np.int64)
    C = -(-T * k // E) + slack
    total = oracle.max_score_assignment(q, k, C)["total"]
    both = auction(ms, q, k, C)
    check(q, both, k, C, total)
    assert both["stats"]["finish_passes"] >= 1
    alone = auction(ms, q, k, C, finisher=False)
    check(q, alone, k, C, total)
    assert alone["stats"]["finish_passes"] == 0
    dense = auction(ms, q, k, C, tail_pass=False, finisher=False)
    check(q, dense, k, C, total)
    assert dense["stats"]["rounds"] > alone["stats"]["rounds"]


@pytest.mark.parametrize("name,T,seed", [("cfg5", 8192, 0), ("cfg3", 4096, 2), ("cfg4b_exact", 4096, 0), ("cfg4b_near", 4096, 1)])
def test_behind_price_tries(ms, name, T, seed):
    """Wide rewards: the price solve gives the problem up, the auction with tail pass and finisher takes it."""
    print(f"auction behind price tries {name}", flush=True)
    q, k, C = instance(name, T, seed)
    q = q << (28 - int(q.max()).bit_length())            # (2^(31 - 6) at most fit beside a 6-bit column)
    total = oracle.max_score_assignment(q, k, C)["total"]
    for _ in range(2):
        out = ms.assign_i32(dev(q.astype(np.int32)), k, C)
        check(q, out, k, C, total)
        assert out["stats"]["phases"] > 1 and out["stats"]["finish_passes"] >= 1, out["stats"]


@pytest.mark.parametrize("T,E,k,spread,seed", [(16384, 128, 2, 2.0, 0), (8192, 32, 4, 2.0, 1), (4096, 64, 8, 2.0, 2)])
def test_finisher_that_hands_back(ms, T, E, k, spread, seed):
    """Strongly skewed popularity: more arcs under the finisher's bound than it holds at its first rung."""
    print(f"auction finisher retry T={T} E={E} k={k}", flush=True)
    rng = np.random.default_rng(seed)
    L = rng.normal(size=(T, E)) + spread * rng.normal(size=(1, E))
    p = np.exp(L - L.max(axis=1, keepdims=True))
    q = np.rint(p / p.sum(axis=1, keepdims=True) * ((1 << 20) - 1)).astype(np.int64)
    C = -(-T * k // E)
    check(q, auction(ms, q, k, C), k, C, oracle.max_score_assignment(q, k, C)["total"])


@pytest.mark.parametrize("name,T,slack", [("cfg5", 8192, 0), ("cfg4a", 4096, 9)])
def test_starting_prices(ms, name, T, slack):
    print(f"auction starting prices {name}", flush=True)
    q, k, C = instance(name, T, 0, slack)
    E = q.shape[1]
    total = oracle.max_score_assignment(q, k, C)["total"]
    cold = auction(ms, q, k, C)
    check(q, cold, k, C, total)
    rng = np.random.default_rng(3)
    S = cold["price_scale"]
    for p_in, eps_start in [(cold["prices"], 1), (cold["prices"], 1 << 40), (dev(rng.integers(0, (1 << 20) * S, E).astype(np.int64)), 0),
                            (dev(np.zeros(E, dtype=np.int64)), 0)]:
        check(q, auction(ms, q, k, C, prices_in=p_in, eps_start=eps_start), k, C, total)
    assert auction(ms, q, k, C, prices_in=cold["prices"], eps_start=1)["stats"]["rounds"] < cold["stats"]["rounds"]


def test_short_capacity_with_padding_experts(ms):
    """More experts than a price solve takes, and room for 70 % of the demand: the padded problem goes through the auction with its
    accelerators."""
    print("auction short capacity E=520", flush=True)
    rng = np.random.default_rng(23)
    T, E, k = 600, 520, 4
    q = rng.integers(0, 1 << 17, (T, E)) + rng.integers(0, 1 << 16, E)[None, :]        # (the padded range has to fit 64-bit bids)
    C = int(0.7 * T * k / E)
    ref = oracle.assign_literal_graph(q, k, C)
    for kw in ({}, dict(finisher=False), dict(finisher=False, tail_pass=False)):
        st = ms.assign_i32(dev(q.astype(np.int32)), k, C, **kw)["stats"]
        assert (st["flow_value"], st["total_score_q"]) == (ref["flow"], ref["total"]), kw
        assert st["rounds"] < (400 if kw == {} else 100000), st
