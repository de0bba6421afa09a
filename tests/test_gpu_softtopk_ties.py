"""GPU parity of the score kernel's two ways to rank a row: by counting where the largest logits differ, one by one where some
of them are equal; ragged and padded rows, every reading of Eq. 6."""
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


@pytest.mark.parametrize("reading", ["A", "A1", "B", "C"])
@pytest.mark.parametrize("E,k", [(1, 1), (5, 5), (8, 2), (20, 4), (31, 8), (64, 64), (96, 6), (128, 8), (200, 3), (256, 8), (1000, 16)])
def test_rows_with_and_without_ties(ms, E, k, reading):
    print(f"softtopk ties E={E} k={k} {reading}", flush=True)
    rng = np.random.default_rng(E + k)
    L = rng.standard_normal((260, E)).astype(np.float32)
    L[40:80] = np.round(L[40:80] * 2) / 2                              # many equal values
    L[80:90] = 0.25                                                    # all equal
    for i in range(90, 120):                                           # one pair, at the top, at the last rank and below it
        o = np.argsort(-L[i])
        j = min([0, max(k - 2, 0), k - 1, k][i % 4], E - 2) if E > 1 else 0
        if E > 1:
            L[i, o[j + 1]] = L[i, o[j]]
    L += 0.0                                                           # (no negative zeros: they rank below positive ones)
    scores, _ = ms.softtopk(torch.from_numpy(L).cuda(), k, 1.0, reading=reading)
    ref = oracle.soft_topk_reading(L.astype(np.float64), k, 1.0, reading)
    assert (np.abs(scores.cpu().numpy() - ref) <= 1e-5 * np.maximum(np.abs(ref), 1e-3)).all()
