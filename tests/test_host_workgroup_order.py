"""Host logic of the kernels compiled with g++ and run here: the chunk-major order of the layer kernels' workgroups and the
taps a convolution tile leaves out."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_chunk_major_order_covers_every_chunk_once(tmp_path):
    exe = tmp_path / "host_workgroup_order"
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Wextra", os.path.join(ROOT, "tests", "host_workgroup_order.cpp"),
                    "-o", str(exe)], check=True)
    res = subprocess.run([str(exe)], stdout=subprocess.PIPE, text=True)
    assert res.returncode == 0 and res.stdout.startswith("OK"), res.stdout


def test_taps_left_out_are_zero(tmp_path):
    exe = tmp_path / "host_tconv_taps"
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Wextra", os.path.join(ROOT, "tests", "host_tconv_taps.cpp"),
                    "-o", str(exe)], check=True)
    res = subprocess.run([str(exe)], stdout=subprocess.PIPE, text=True)
    assert res.returncode == 0 and res.stdout.startswith("OK"), res.stdout
