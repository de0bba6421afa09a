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


@pytest.mark.parametrize("T,E", [(1, 4), (15, 8), (65, 130), (4097, 3), (65536, 128), (262144, 128), (262145, 129), (300001, 64),
                                 (3584, 128), (4033, 128), (4096, 128), (4160, 100), (450, 1024), (513, 1023), (20000, 128)])
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


@pytest.mark.parametrize("E,G,EPL", [(32, 8, 4), (64, 16, 4), (128, 16, 8), (256, 32, 8), (512, 64, 8), (1024, 64, 16)])
def test_gate_backward_sums(ms, E, G, EPL):
    """A row's sum of gA_j * A_j rounds log2(E) times, as a tree of its E terms does.  Here G lanes hold EPL columns each: added up
    one by one, each of lane 0's further columns, and each of the lanes it meets, is lost in a tie beside the 1 of its first
    column.  Softmax of equal logits and the division by their number are exact, so a column without a score shows the sum."""
    levels = E.bit_length() - 1
    print(f"gate backward sums E={E}", flush=True)
    scores = torch.zeros(4, E)
    for m in range(EPL):
        scores[:, (m >> 2) * 4 * G + (m & 3)] = ULP if m else 1.0
    off = 1
    while off < G:
        scores[:, 4 * off] = ULP
        off *= 2
    assign = torch.full((4, 1), -1, dtype=torch.int32, device="cuda")
    got = ms.gates_backward(torch.zeros(4, E, device="cuda"), scores.cuda(), assign, torch.zeros(4, 1, device="cuda"),
                            torch.ones(E, device="cuda")).cpu().double()
    total = scores.double().sum(dim=1, keepdim=True)
    error = float(((-got * E / total - 1)[scores == 0]).abs().max())
    print(error / ULP, "of", levels, flush=True)
    assert error <= levels * ULP


@pytest.mark.parametrize("T,E,order", [(512, 64, "chains"), (1024, 32, "chains"), (4096, 16, "chains"), (600, 64, "lanes"), (1100, 32, "lanes")])
def test_sinkhorn_row_sums(ms, T, E, order):
    """u = 1 / (sum of a row of K) after one iteration, from the plan's ratio to that of a row whose sum is exactly 1.  The sum rounds
    log2(E) times as a tree; u and the plan's entry round once each.  Beside the row's one entry of 1 there are entries just short
    of a tie: at every fourth column, as four chains add them, or where one lane of eight adds its own one by one and then meets
    the others."""
    print(f"sinkhorn row sums T={T} E={E} {order}", flush=True)
    levels, M, t = E.bit_length() - 1, 200.0, 0.99 * ULP
    scores = torch.zeros(T, E)
    scores[:, E - 1] = M + 1                                  # everybody's first choice: its residual affinity is 0, its K too
    low = M + float(np.log(t))
    epl = E // 8
    cols = list(range(4, E - 1, 4)) if order == "chains" else list(range(1, epl)) + [epl, 2 * epl, 4 * epl]
    scores[0::2, 0] = M
    scores[1::2, 0] = M
    scores[0::2, cols] = low
    out = ms.assign_top1_sinkhorn(scores.cuda(), T, 1.0, 1, want_plan=True)
    plan = out["plan"].cpu().double()[:, 0]
    K = np.exp(scores.double().numpy()[0, cols] - M).sum()
    ratio = float(plan[0] / plan[1])
    error = abs(ratio * (1 + K) - 1)
    print(error / ULP, "of", levels + 2, flush=True)
    assert error <= (levels + 2) * ULP
