"""GPU: the tables of a price pass on both sides of the rules that choose their counts (16 bits where no copy's count can reach
2^16: one per row with demand equal to capacity, four with spare capacity, k with less) and the number of their copies (by
workgroups).  Rows that differ little put nearly all counts into a few bins.  Totals against the auction's, three runs alike."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SHAPES = [  # T, E, k, C
    (64000, 16, 8, 30000), (65536, 16, 8, 30000),              # unfilled slots: 63 and 64 workgroups of 128 rows a copy
    (130000, 8, 1, 17000), (131072, 8, 1, 17000),              # spare capacity
    (524160, 8, 1, 65520), (524288, 8, 1, 65536),              # demand equal to capacity
    (2100, 20, 2, 210), (8191, 24, 3, 1100), (8192, 24, 3, 1024), (16383, 24, 3, 2200), (16384, 24, 3, 2048),
    (9000, 260, 2, 75),
]


@pytest.mark.parametrize("T,E,k,C", SHAPES)
def test_counts(T, E, k, C):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2508_12801_amd as ms
    print(f"price counts T={T} E={E} k={k} C={C}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(T + E)
    L = 0.05 * torch.randn(T, E, generator=gen, device="cuda") + 0.3 * torch.randn(E, generator=gen, device="cuda")
    q = ms.softtopk(L, k, 1.0)[1]
    first = ms.assign_i32(q, k, C)
    for _ in range(2):
        again = ms.assign_i32(q, k, C)
        assert again["stats"]["total_score_q"] == first["stats"]["total_score_q"]
        if first["stats"]["rounds"] < 60 and first["stats"]["phases"] == 1:
            assert torch.equal(again["assign"], first["assign"]) and again["stats"]["rounds"] == first["stats"]["rounds"]
    a = first["assign"].long()
    held = a >= 0
    assert int(q.gather(1, a.clamp(min=0))[held].sum()) == first["stats"]["total_score_q"]
    assert int(held.sum()) == min(T * k, E * C) and int(torch.bincount(a[held], minlength=E).max()) <= C
    plain = ms.assign_i32(q, k, C, finisher=False)["stats"]
    assert plain["total_score_q"] == first["stats"]["total_score_q"]
