"""GPU parity of the rerouting rounds and of the dispatch behind them at the edges of their kernels: token counts around a
block, expert counts around the lanes and columns of a row, slot counts around what the counted dispatch takes."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def ms():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2508_12801_amd as m
    m.load_library()
    return m


@pytest.mark.parametrize("T,E,k,C", [
    (1, 1, 1, 1), (1, 9, 2, 1), (63, 8, 8, 63), (64, 9, 3, 20), (65, 64, 16, 17), (129, 65, 17, 36), (200, 128, 5, 7),
    (190, 129, 2, 2), (300, 256, 16, 19), (300, 257, 4, 4), (130, 512, 3, 1), (130, 513, 3, 1), (1000, 20, 6, 200), (2049, 12, 4, 683),
])
def test_edges(ms, T, E, k, C):
    print(f"iter edges T={T} E={E} k={k} C={C}", flush=True)
    rng = np.random.default_rng(T + E + k)
    L = (rng.standard_normal((T, E)) + rng.standard_normal(E)).astype(np.float32)
    out = ms.route_logits(torch.from_numpy(L).cuda(), k, C, assignment="iter", allow_not_converged=True)
    ref = oracle.iter_reroute(out["q"].cpu().numpy().astype(np.int64), k, C)
    a = out["assign"].cpu().numpy()
    assert np.array_equal(a, ref["assign"])
    s = out["stats"]
    assert (s["total_score_q"], s["flow_value"], s["rounds"]) == (ref["total"], ref["flow"], ref["rounds"])
    g = out["gates"].cpu().numpy()
    scores = out["scores"].cpu().numpy()
    assert np.array_equal(g, np.where(a >= 0, np.take_along_axis(scores, np.maximum(a, 0), axis=1), 0))
    want = oracle.dispatch(a, g, E)
    n = ref["flow"]
    assert np.array_equal(out["expert_offsets"].cpu().numpy(), want["expert_offsets"])
    assert np.array_equal(out["disp_token"].cpu().numpy()[:n], want["disp_token"])
    assert np.array_equal(out["disp_gate"].cpu().numpy()[:n], want["disp_gate"])
    assert np.array_equal(out["token_pos"].cpu().numpy(), want["token_pos"])


@pytest.mark.parametrize("T,E,k,C", [(9000, 320, 64, 1700), (9003, 257, 60, 2300), (3000, 1024, 64, 180)])
def test_many_slots_and_experts(ms, T, E, k, C):
    """Where the counts per (slot, 64 tokens, expert) only fit as bytes."""
    print(f"iter byte tiles T={T} E={E} k={k} C={C}", flush=True)
    rng = np.random.default_rng(T + E + k)
    q = rng.integers(0, 1 << 18, (T, E)) + (rng.standard_normal(E) * (1 << 17)).astype(np.int64)
    ref = oracle.iter_reroute(q, k, C)
    out = ms.assign_iter_i32(torch.from_numpy(q.astype(np.int32)).cuda(), k, C, allow_not_converged=True)
    assert np.array_equal(out["assign"].cpu().numpy(), ref["assign"])
    assert (out["total"], out["flow"], out["rounds"]) == (ref["total"], ref["flow"], ref["rounds"])


@pytest.mark.parametrize("T,E,k,C,hi", [
    (3000, 32, 32, 2900, 1 << 20), (2000, 33, 32, 2000, 5),          # as many slots as the last rounds' workgroup takes
    (6000, 8, 4, 2900, 1 << 20), (6000, 8, 4, 3000, 4),              # tokens whose slots run out of experts to ask
    (66, 2, 1, 33, 3), (130, 16, 2, 9, 1 << 10), (20000, 4, 1, 5001, 2),      # one round of all tokens, then the last ones
    (4100, 512, 2, 17, 1 << 20), (4100, 1024, 3, 13, 1 << 16), (40000, 64, 2, 1250, 1 << 29),        # the fewest pairs, keys that do not pack
])
@pytest.mark.parametrize("max_rounds", [-1, 2, 4])
def test_last_rounds(ms, T, E, k, C, hi, max_rounds):
    """The rounds one workgroup goes through by itself: uneven experts, so that many rounds follow, and rounds that are cut short."""
    print(f"iter last rounds T={T} E={E} k={k} C={C} hi={hi} max_rounds={max_rounds}", flush=True)
    rng = np.random.default_rng(T + E + k + hi)
    q = rng.integers(0, hi, (T, E)) + (rng.random(E) ** 3 * hi).astype(np.int64)
    ref = oracle.iter_reroute(q, k, C, max_rounds=max_rounds if max_rounds >= 0 else None)
    out = ms.assign_iter_i32(torch.from_numpy(q.astype(np.int32)).cuda(), k, C, max_rounds=max_rounds, allow_not_converged=True)
    assert np.array_equal(out["assign"].cpu().numpy(), ref["assign"])
    assert (out["total"], out["flow"], out["rounds"]) == (ref["total"], ref["flow"], ref["rounds"])


@pytest.mark.parametrize("T", [358336, 358337])
def test_last_rounds_of_many_blocks(ms, T):
    """Eight slots of 16 experts at the largest number of 64-token blocks whose first rows fit beside a workgroup's rounds, and one more."""
    E, k = 16, 8
    C = T * k // E + T // 100
    print(f"iter many blocks T={T}", flush=True)
    rng = np.random.default_rng(T)
    q = (rng.random((T, E)) * 1e6).astype(np.int64) + (rng.random(E) * 1e5).astype(np.int64)
    ref = oracle.iter_reroute(q, k, C)
    out = ms.assign_iter_i32(torch.from_numpy(q.astype(np.int32)).cuda(), k, C, allow_not_converged=True)
    assert np.array_equal(out["assign"].cpu().numpy(), ref["assign"])
    assert (out["total"], out["flow"], out["rounds"]) == (ref["total"], ref["flow"], ref["rounds"])
