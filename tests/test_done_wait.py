"""The host's wait for the words that end a call, against a model of them (no GPU)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_words_that_come_late_or_never(tmp_path):
    exe = str(tmp_path / "done_wait")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2508_12801_amd", "csrc"),
                           os.path.join(ROOT, "tests", "sanitize", "done_wait.cpp"), "-o", exe])
    r = subprocess.run([exe], stdout=subprocess.PIPE, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
