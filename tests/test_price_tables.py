"""The tables of the price solve at every expert count it accepts (no GPU): no copy reaches into the next one."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_copies_of_the_tables_do_not_overlap(tmp_path):
    exe = str(tmp_path / "price_tables")
    subprocess.check_call(["g++", "-std=c++17", "-I", os.path.join(ROOT, "paper_2508_12801_amd", "csrc"),
                           os.path.join(ROOT, "tests", "sanitize", "price_tables.cpp"), "-o", exe])
    r = subprocess.run([exe], stdout=subprocess.PIPE, text=True)
    assert r.returncode == 0, r.stdout
