"""Error of the polynomial GELU in the bf16 epilogues, evaluated on the host in fp32."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_gelu_error_is_smallest_where_hidden_values_lie(tmp_path):
    """Bounds: what a fit with an even error of 1e-5 in Phi gives (v Phi(v): |v| times that, less below
    1), and the clamp's v (1 - Phi(v)) where it takes over; 1 % for the fp32 evaluation."""
    exe = str(tmp_path / "gelu_error")
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-ffp-contract=off", "-I",
                           os.path.join(ROOT, "paper_2404_05019_amd", "csrc"),
                           os.path.join(ROOT, "tests", "gelu_error_main.cpp"), "-o", exe])
    lines = [line.split() for line in subprocess.check_output([exe], text=True).splitlines()]
    worst = {float(w[2]): float(w[3]) for w in lines if w[0] == "max"}
    rms = {float(w[1]): float(w[2]) for w in lines if w[0] == "rms"}
    for hi, bound in {0.1: 3.8e-7, 0.25: 1.94e-6, 0.5: 3.26e-6, 1.0: 8.42e-6, 1.5: 9.67e-6, 2.0: 1.40e-5, 2.5: 1.93e-5,
                      3.0: 2.39e-5, 3.5: 2.91e-5, 4.0: 4.05e-5, 4.2: 4.48e-5, 12.0: 4.7e-5}.items():
        assert worst[hi] <= 1.01 * bound, (hi, worst[hi])
    for s, bound in {0.1: 1.12e-5, 0.25: 1.27e-5, 0.5: 1.02e-5, 1.0: 9.05e-6, 1.5: 8.56e-6, 2.0: 7.87e-6, 4.0: 5.46e-6}.items():
        assert rms[s] <= 1.01 * bound, (s, rms[s])
    assert lines[-1] == ["special", "1", "1", "1"]
