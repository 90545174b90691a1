"""The launcher's rules on strides (csrc/layout_rules.hpp), compiled with g++ and run here."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_layout_rules(tmp_path):
    exe = tmp_path / "host_layout_rules"
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Wextra", os.path.join(ROOT, "tests", "host_layout_rules.cpp"),
                    "-o", str(exe)], check=True)
    res = subprocess.run([str(exe)], stdout=subprocess.PIPE, text=True)
    assert res.returncode == 0 and res.stdout.startswith("OK"), res.stdout
