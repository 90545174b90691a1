"""Host logic of the quadrant state kernel compiled with g++ and run here: how its grid is dealt, and when it is used."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_quadrants_are_dealt_once(tmp_path):
    exe = tmp_path / "host_quad_role"
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Wextra", os.path.join(ROOT, "tests", "host_quad_role.cpp"),
                    "-o", str(exe)], check=True)
    res = subprocess.run([str(exe)], stdout=subprocess.PIPE, text=True)
    assert res.returncode == 0 and res.stdout.startswith("OK"), res.stdout
