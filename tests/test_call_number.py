"""The numbers that mark a call's workgroups as done: another one for every call."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_no_two_counts_have_one_number(tmp_path):
    exe = str(tmp_path / "call_number")
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-Wall", "-I", os.path.join(ROOT, "paper_2404_05019_amd", "csrc"),
                           os.path.join(ROOT, "tests", "call_number_main.cpp"), "-o", exe])
    assert subprocess.check_output([exe], text=True) == "ok\n"
