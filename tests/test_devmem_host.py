"""Kept device blocks against a host model of streams (devmem_host.cpp): no block is
handed out, and none returned to the runtime, ahead of the work that uses it."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("devmem") / "devmem_host")
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-D__HIP_PLATFORM_AMD__", "-x", "c++", "-w",
                    "-I", "/opt/rocm/include", os.path.join(HERE, "devmem_host.cpp"), "-o", exe],
                   check=True)
    return exe


@pytest.mark.parametrize("scenario", ["destroy_same_stream", "destroy_restreamed", "reuse",
                                      "restream", "restream_capture", "trim_other_device",
                                      "other_device_goes_on", "graph_memory", "no_host_memory",
                                      "stay_after_capture"])
def test_scenario(model, scenario):
    r = subprocess.run([model, scenario], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stdout + r.stderr
