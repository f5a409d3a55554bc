"""Job server when a lane's stream cannot be made (no GPU needed: the host
code of server.hip over stand-ins for the HIP calls and the lattices)."""
import os
import subprocess

from paper_1612_08312_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_a_refused_lane_stream_fails_its_job_only(tmp_path):
    obj, exe = str(tmp_path / "server.o"), str(tmp_path / "server_check")
    subprocess.run([build.HIPCC, "--offload-host-only", "-fPIC", "-O1", "-std=c++17", "-w", "-c",
                    os.path.join(build.CSRC, "server.hip"), "-o", obj], check=True)
    subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include",
                    os.path.join(ROOT, "tests", "server_check.cpp"), obj, "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "server ok" in r.stdout, r.stderr
