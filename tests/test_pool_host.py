"""The factor pool that a stored ACA starts with stays within the caller's budget."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_first_pool_and_budget(tmp_path):
    exe = str(tmp_path / "pool_host")
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-w", "-I",
                    "/opt/rocm/include", os.path.join(HERE, "pool_host.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stdout[-2000:]
