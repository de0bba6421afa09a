"""bench.py's account of the solver (no GPU), from statistics as either solver reports them, with and without launch times; and,
on a GPU, one short run of the whole benchmark."""
import json
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402

PRICE = dict(rounds=6, phases=1, solver_ms=0.5, bid_ms=0.1, bid_launches=6, select_ms=0.05, finish_passes=1, finish_cycles=40)
AUCTION = dict(rounds=46, phases=3, solver_ms=1.6, bid_ms=0.5, bid_launches=46, select_ms=0.6, finish_passes=1, finish_cycles=6)
UNTIMED = dict(bid_ms=0.0, bid_launches=0, select_ms=0.0)


@pytest.mark.parametrize("T", [65536, 131071, 131072])
@pytest.mark.parametrize("st", [PRICE, AUCTION, dict(PRICE, **UNTIMED), dict(AUCTION, **UNTIMED), dict(PRICE, rounds=0, **UNTIMED)])
def test_roofline(st, T):
    E, k = 128, 8
    r = bench.solver_roofline(st, T, E, k, 0.5, 0.02)
    assert r["solver"] == ("price" if st["phases"] == 1 else "auction")
    assert r["bytes"] > r["floor_bytes"] == T * E * 4 + T * k * 4 + 8 * E
    assert abs(r["frac"] - r["bytes"] / 0.52e-3 / 8e12) < 1e-9
    for name in (("k_price", "k_price_update") if st["phases"] == 1 else ("k_bid", "k_select")):
        assert (r["kernels"][name]["launch_us"] is None) == (st["bid_launches"] == 0)
    if st["phases"] == 1 and st["rounds"]:
        # six passes, of which the first two of many tokens read 8192 rows only, and the last one
        rows = 7 * T if T < 131072 else 2 * 8192 + 5 * T
        assert r["bytes"] - r["kernels"]["gates_dispatch"]["bytes"] == E * 4 * rows + T * k * 4 + (T + 127) // 128 * E * 4
    json.dumps(r)


def test_traffic_is_that_of_as_many_passes():
    rounds = bench.profile_value("pass_cfg5_pmc_traffic.txt", "pass_rounds")
    assert rounds and bench.profile_traffic(int(rounds)) == bench.profile_value("pass_cfg5_pmc_traffic.txt", "pass_traffic_bytes") > 0
    assert bench.profile_traffic(int(rounds) + 1) is None


@pytest.mark.gpu
@pytest.mark.parametrize("config", ["cfg2", "cfg5"])
def test_one_line(config, monkeypatch, capsys):
    print(f"bench {config}", flush=True)
    monkeypatch.setattr(sys, "argv", ["bench.py", "--steps", "2", "--warmup", "1", "--config", config, "--no-cpu-baseline", "--no-concurrent"])
    bench.main()
    line = json.loads(capsys.readouterr().out.strip().splitlines()[-1])
    assert line["value"] > 0 and line["steps"] == 2 and line["n_gpus"] == 1
    r = line["roofline"]
    assert r["solver"] == "price" and r["kernels"]["k_price"]["launches"] >= 1 and 0 < r["frac"] < 1
