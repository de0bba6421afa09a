"""GPU: the reported solver time holds everything the call spent on the assignment, price tries that do not stand included."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def test_time_of_failed_price_tries():
    """Rewards of 27 bits do not fit the price solve's packed keys beside a 6-bit column, which its last pass finds out; the
    auction then has an easy problem: some 0.16 ms, and 0.07 ms for the passes before it.  An auction without a finisher
    alone takes 0.21 ms: the two together are 1.09 to 1.12 times that, without the passes they would be 0.75 times.  (At 65536 tokens they were
    1.05 to 1.09 times, too close to the 1.05 that was asked for there.)"""
    import paper_2508_12801_amd as ms
    print("solver time", flush=True)
    T, E, k, C = 131072, 64, 2, 131072
    rng = np.random.default_rng(4)
    q = torch.from_numpy(rng.integers(0, 1 << 27, (T, E)).astype(np.int32)).cuda()

    def solver_ms(**kw):
        runs = [ms.assign_i32(q, k, C, **kw)["stats"] for _ in range(10)]
        assert all(r["flow_value"] == T * k and r["total_score_q"] == runs[0]["total_score_q"] for r in runs)
        return min(r["solver_ms"] for r in runs)

    both, auction = solver_ms(), solver_ms(finisher=False)
    print(both, auction, flush=True)
    assert both > auction
