"""GPU parity of the dispatch lists behind a price solve and behind iterative rerouting on both sides of the rule by which the
workgroups add up the counts of the others themselves (blocks times experts up to 4096, 256 experts)."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("assignment", ["exact", "iter"])
@pytest.mark.parametrize("T,E,k,C", [(1, 2, 1, 1), (64, 8, 2, 16), (8192, 16, 2, 1024), (8200, 16, 2, 1100), (1000, 130, 2, 20), (500, 256, 2, 5),
                                     (500, 257, 2, 5), (16400, 16, 1, 1200), (70, 200, 3, 1)])
def test_lists(T, E, k, C, assignment):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2508_12801_amd as ms
    print(f"count dispatch T={T} E={E} k={k} C={C} {assignment}", flush=True)
    rng = np.random.default_rng(T + E)
    L = (rng.standard_normal((T, E)) + 0.5 * rng.standard_normal(E)).astype(np.float32)
    out = ms.route_logits(torch.from_numpy(L).cuda(), k, C, assignment=assignment)
    a, gates = out["assign"].cpu().numpy(), out["gates"].cpu().numpy()
    held = a >= 0
    scores = out["scores"].cpu().numpy()
    assert np.array_equal(gates, np.where(held, np.take_along_axis(scores, np.where(held, a, 0).astype(np.int64), axis=1), 0))
    want, n = oracle.dispatch(a, gates, E), int(held.sum())
    assert np.array_equal(out["expert_offsets"].cpu().numpy(), want["expert_offsets"])
    assert np.array_equal(out["disp_token"].cpu().numpy()[:n], want["disp_token"][:n])
    assert np.array_equal(out["disp_gate"].cpu().numpy()[:n], want["disp_gate"][:n].astype(np.float32))
    assert np.array_equal(out["token_pos"].cpu().numpy(), want["token_pos"])
