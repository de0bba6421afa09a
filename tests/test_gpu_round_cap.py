"""GPU: max_rounds holds for whichever solver takes the call.  The price solve of the second and third case takes 20 passes."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("max_rounds", [16, 19, 59, 60])
@pytest.mark.parametrize("T,E,k,C,same_rows", [(123, 8, 5, 77, True), (123, 8, 5, 62, False), (80, 4, 1, 22, True), (6000, 32, 3, 563, True)])
def test_rounds_stay_under_the_cap(T, E, k, C, same_rows, max_rounds):
    import paper_2508_12801_amd as ms
    print(f"round cap T={T} E={E} k={k} C={C} max_rounds={max_rounds}", flush=True)
    rng = np.random.default_rng(231)
    row = rng.integers(0, 1 << 20, (1, E))
    q = np.tile(row, (T, 1)) if same_rows else (np.exp(rng.normal(size=(T, E)) * 2 + 3 * rng.normal(size=(1, E))) * 1000).clip(0, 1 << 20)
    out = ms.assign_i32(torch.from_numpy(q.astype(np.int32)).cuda(), k, C, max_rounds=max_rounds, allow_not_converged=True)
    st = out["stats"]
    print(st, flush=True)
    assert st["rounds"] <= max_rounds and st["status"] == out["rc"]
    P = oracle.assignment_matrix(out["assign"].cpu().numpy(), E)
    assert P.max() <= 1 and P.sum(axis=1).max() <= k and P.sum(axis=0).max() <= C
    if out["rc"] == 0:
        assert int(P.sum()) == min(T * k, E * C)
        assert st["total_score_q"] == oracle.max_score_assignment(q.astype(np.int64), k, C)["total"]
