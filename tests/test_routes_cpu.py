"""The rules that choose kernels (routes.hpp), compiled and run on the host."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_routes(tmp_path):
    exe = str(tmp_path / "routes_test")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-o", exe,
                    os.path.join(HERE, "native", "routes_test.cpp")], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout
