"""The host's loop over the passes of a price solve against a model of the stream in which words are lost (no GPU): the end runs once."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_the_end_runs_once(tmp_path):
    exe = str(tmp_path / "price_loop")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2508_12801_amd", "csrc"),
                           os.path.join(ROOT, "tests", "sanitize", "price_loop.cpp"), "-o", exe])
    r = subprocess.run([exe], stdout=subprocess.PIPE, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
