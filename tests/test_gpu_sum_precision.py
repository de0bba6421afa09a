"""GPU: sums that one thread adds up for many rows or columns round no oftener than stated, on inputs whose roundings add up."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

ULP = 2.0 ** -24


@pytest.fixture(scope="module")
def ms():
    import paper_2508_12801_amd as m
    m.load_library()
    return m


@pytest.mark.parametrize("T,E", [(1, 4), (15, 8), (65, 130), (4097, 3), (65536, 128), (262144, 128), (262145, 129), (300001, 64)])
def test_column_means(ms, T, E):
    """A column of equal values: 15 roundings of the 16 rows a thread adds up in fp32, one of a block's sum and one of the mean."""
    print(f"column means T={T} E={E}", flush=True)
    c = torch.rand(E, generator=torch.Generator().manual_seed(T), dtype=torch.float32) * 0.9 + 0.05
    scores = c.cuda()[None, :].expand(T, E).contiguous()
    offsets = torch.full((E + 1,), T, dtype=torch.int32).cuda()
    got = ms.aux_loss(scores, offsets, 1.0)["mean_scores"].cpu().double()
    worst = float(((got - c.double()).abs() / c.double()).max())
    print(worst / ULP, flush=True)
    assert worst <= 17 * ULP
