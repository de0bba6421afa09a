"""GPU parity of the Sinkhorn step where its kernels change hands: the row counts up to which one workgroup takes the call, the
expert counts up to which eight lanes own a row, ragged columns, no and one iteration."""
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


@pytest.mark.parametrize("T,E,n_iter", [
    (1, 2, 3), (63, 7, 5), (65, 8, 0), (8192, 8, 4), (8193, 8, 4), (4095, 12, 1), (4096, 16, 5), (4097, 16, 5), (1024, 32, 3),
    (1025, 31, 3), (512, 64, 4), (513, 64, 4), (300, 63, 0), (700, 33, 1), (600, 65, 2), (20000, 20, 3), (17000, 61, 0),
])
def test_edges(ms, T, E, n_iter):
    print(f"sinkhorn edges T={T} E={E} n={n_iter}", flush=True)
    rng = np.random.default_rng(T + E)
    A = oracle.soft_topk(rng.normal(size=(T, E)) + 0.5 * rng.normal(size=(1, E)), 2, 1.0).astype(np.float32)
    C = -(-2 * T // E)
    out = ms.assign_top1_sinkhorn(torch.from_numpy(A).cuda(), C, 0.1, n_iter, want_plan=True)
    ref = oracle.top1_then_sinkhorn(A.astype(np.float64), C, 0.1, n_iter)
    a, plan = out["assign"].cpu().numpy(), out["plan"].cpu().numpy().astype(np.float64)
    assert np.array_equal(a[:, 0], ref["assign"][:, 0]) and out["caps"] == ref["caps"].tolist()
    top = ref["plan"].max(axis=1, keepdims=True)
    assert (np.abs(plan - ref["plan"]) <= 2e-4 * top + 1e-30).all()
    assert np.array_equal(a[:, 1] >= 0, ref["assign"][:, 1] >= 0)
    chosen = np.take_along_axis(ref["plan"], np.maximum(a[:, 1:], 0).astype(np.int64), axis=1)
    assert (chosen >= (1 - 4e-4) * top)[a[:, 1] >= 0].all()
