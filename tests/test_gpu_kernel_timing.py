"""GPU: the per-launch times that maxscore_set_kernel_timing asks for, on every way an assignment is solved."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture
def ms():
    import paper_2508_12801_amd as m
    m.load_library()
    yield m
    m.set_kernel_timing(False)


def rewards(ms, T, E, k):
    rng = np.random.default_rng(T + E)
    L = torch.from_numpy((rng.standard_normal((T, E)) + 0.7 * rng.standard_normal(E)).astype(np.float32)).cuda()
    return ms.softtopk(L, k, 1.0)[1]


@pytest.mark.parametrize("T,E,k,C,one_launch", [(256, 8, 2, 64, True), (5000, 64, 4, 320, False), (20000, 32, 2, 1250, False),
                                                (5000, 64, 4, 250, False)])
def test_price_solve(ms, T, E, k, C, one_launch):
    print(f"kernel timing T={T} E={E} k={k} C={C}", flush=True)
    q = rewards(ms, T, E, k)
    off = ms.assign_i32(q, k, C)
    assert off["stats"]["bid_ms"] == off["stats"]["select_ms"] == off["stats"]["bid_launches"] == 0
    ms.set_kernel_timing(True)
    on = ms.assign_i32(q, k, C)
    st = on["stats"]
    assert torch.equal(on["assign"], off["assign"]) and st["rounds"] == off["stats"]["rounds"] > 0
    assert st["bid_launches"] == (1 if one_launch else st["rounds"])
    assert 0 < st["bid_ms"] < st["solver_ms"] and (st["select_ms"] == 0) == one_launch
    if T * k <= E * C and not one_launch:
        # the pass that checks given prices is a launch that is not counted among the rounds
        own = ms.assign_i32(q, k, C, prices_in=on["prices"])["stats"]
        assert own["bid_launches"] == own["rounds"] + 1


def test_auction(ms):
    print("kernel timing auction", flush=True)
    q = rewards(ms, 5000, 64, 4)
    ms.set_kernel_timing(True)
    st = ms.assign_i32(q, 4, 320, finisher=False)["stats"]
    assert st["bid_launches"] == st["rounds"] > 0
    assert 0 < st["bid_ms"] + st["select_ms"] < st["solver_ms"] and st["select_ms"] > 0
