"""The corrected quotient of the smoother's solves against the division (CPU)."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_corrected_quotient_is_the_division(tmp_path):
    """All edges of both operands and 20 million random bit patterns: equal to the
    division bit for bit, one ulp off only for dividends below 1e-30."""
    exe = str(tmp_path / "quotient_check")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-ffp-contract=off", "-o", exe,
                    os.path.join(HERE, "quotient_check.cpp")], check=True)
    r = subprocess.run([exe, "20000000"], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout
