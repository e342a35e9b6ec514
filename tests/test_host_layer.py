"""The layer's host code on the CPU, built with stand-ins for the HIP runtime and the kernels' launchers (host_layer.cpp):
what it does when device memory runs out, how much it takes, in which order it enqueues what runs on two streams, what it waits for
before it reads, what it does with a call that fails, and that what has to be allowed once per device is."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("host_layer") / "host_layer")
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2309_03523_amd", "csrc"), os.path.join(HERE, "host_layer.cpp"), "-o", out,
                    "-Wl,--unresolved-symbols=ignore-all"], check=True, timeout=120)     # launchers that no check reaches
    return out


@pytest.mark.parametrize("check", ["input gradient memory", "label memory", "neighbour table", "stage events", "one stream", "lds per device", "evolve memory", "gradient read", "folded weights"])
def test_host_layer(program, check):
    r = subprocess.run([program, check], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
