"""GPU: the one-workgroup Sinkhorn step where row sums lie below the range in which a reciprocal and a Newton step stand for the division:
every token's best two experts are full, and what is left of its kernel row is e^-72."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("tau", [0.0125, 0.1])
@pytest.mark.parametrize("T,E", [(8192, 8), (4096, 16), (4095, 16), (2048, 32), (64, 8), (257, 16), (1025, 16), (2049, 8), (300, 32)])
def test_rows_of_tiny_sums(T, E, tau):
    import paper_2508_12801_amd as ms
    print(f"sinkhorn tiny sums T={T} E={E} tau={tau}", flush=True)
    rng = np.random.default_rng(T + E)
    A = (0.01 * rng.random((T, E))).astype(np.float32)
    first = np.arange(T) % 2
    A[np.arange(T), first], A[np.arange(T), 1 - first] = 1.0, 0.9
    C = T // 4
    out = ms.assign_top1_sinkhorn(torch.from_numpy(A).cuda(), C, tau, 5, want_plan=True)
    ref = oracle.top1_then_sinkhorn(A.astype(np.float64), C, tau, 5)
    plan = out["plan"].cpu().numpy().astype(np.float64)
    assert np.array_equal(out["assign"].cpu().numpy()[:, 0], first) and out["caps"] == ref["caps"].tolist()
    # the exponents are exact to 2^-24 of 72 or less, twice in a row's ratios, and each of the sums to 2^-20
    assert (np.abs(plan - ref["plan"]) <= (2 * 72 * 2.0 ** -24 + 10 * 2.0 ** -20) * ref["plan"].max(axis=1, keepdims=True)).all()
