"""Accuracy of the complex transforms' factor tables."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2409_03568_amd", "csrc")


def test_factors(tmp_path):
    exe = str(tmp_path / "fft_tables_test")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-ffp-contract=off", "-o", exe,
                    os.path.join(HERE, "native", "fft_tables_test.cpp"), os.path.join(CSRC, "host_math.cpp")], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip() == "OK", r.stdout[-2000:]
