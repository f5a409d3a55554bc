"""Per-device set-up of the kernels that need more LDS than a launch may take
by default: a second device of a process is set up too, and a failure is not
kept (no GPU needed)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_each_device_is_set_up(tmp_path):
    exe = str(tmp_path / "device_once_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-pthread", "-I", os.path.join(ROOT, "paper_1612_08312_amd", "csrc"),
                    os.path.join(ROOT, "tests", "device_once_check.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "device_once ok" in r.stdout, r.stderr
