"""GPU: column sums of the one-workgroup Sinkhorn step, of batches whose threads take several rows: up to 1024 tokens everything behind the product is
in 64 bits, so that a plan of one iteration whose kernel is zeros and ones comes out to the last bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("T,E", [(64, 8), (300, 8), (1000, 8), (1024, 8), (64, 16), (257, 16), (700, 16), (1000, 15), (1024, 16)])
def test_sums_of_a_few_rows(T, E):
    import paper_2508_12801_amd as ms
    print(f"sinkhorn sums T={T} E={E}", flush=True)
    rows = np.arange(T)
    ones = np.array([3, 5, 7, 6])[rows // 256 % 4]                  # reciprocals that do not fit each other
    A = np.full((T, E), -10.0, dtype=np.float32)                    # a kernel entry of exp(-400), zero
    for j in range(7):
        A[rows[ones > j], (rows[ones > j] + j) % E] = 10.0          # ... of one
    first = (rows + E - 1) % E
    A[rows, first] = 11.0                                           # the best expert, a kernel entry of exp(-200)
    C = T
    out = ms.assign_top1_sinkhorn(torch.from_numpy(A).cuda(), C, 0.05, 1, want_plan=True)
    caps = C - np.bincount(first, minlength=E)
    assert np.array_equal(out["assign"].cpu().numpy()[:, 0], first) and out["caps"] == caps.tolist()
    K = A == 10.0
    u = np.float32(1) / ones.astype(np.float32)
    target = (caps * float(T) / caps.sum()).astype(np.float32)
    total = (K * u[:, None].astype(np.float64)).sum(axis=0)
    v = (target.astype(np.float64) / total).astype(np.float32)
    assert np.array_equal(out["plan"].cpu().numpy(), np.where(K, u[:, None] * v[None, :], np.float32(0)))
