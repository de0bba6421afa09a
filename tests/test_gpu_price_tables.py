"""GPU: a price solve of as many experts as it takes, with the extra column of spare and of short capacity, does not depend on
the order of execution (the copies of its tables are separate words), and reaches the auction's total."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("T,E,k,C", [(4096, 512, 2, 17), (4096, 512, 2, 15), (3000, 509, 3, 19)])
def test_same_result_every_time(T, E, k, C):
    import paper_2508_12801_amd as ms
    print(f"price tables T={T} E={E} k={k} C={C}", flush=True)
    rng = np.random.default_rng(E + C)
    L = torch.from_numpy((rng.standard_normal((T, E)) + 0.7 * rng.standard_normal(E)).astype(np.float32)).cuda()
    q = ms.softtopk(L, k, 1.0)[1]
    first = ms.assign_i32(q, k, C)
    for _ in range(5):
        again = ms.assign_i32(q, k, C)
        assert torch.equal(again["assign"], first["assign"]) and torch.equal(again["prices"], first["prices"])
        assert again["stats"]["rounds"] == first["stats"]["rounds"]
    plain = ms.assign_i32(q, k, C, finisher=False)["stats"]
    assert plain["total_score_q"] == first["stats"]["total_score_q"] and plain["flow_value"] == first["stats"]["flow_value"]
