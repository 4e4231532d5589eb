"""The launch shapes of the few-row GEMM on the CPU (csrc/strips.h in the host program strips_host.cpp)."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def strips_host(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not found")
    exe = str(tmp_path_factory.mktemp("strips") / "strips_host")
    res = subprocess.run([HIPCC, "--offload-arch=gfx950", "-O1", "-std=c++17", os.path.join(HERE, "strips_host.cpp"), "-o", exe],
                         stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert res.returncode == 0, res.stdout[-2000:]
    return exe


def test_shapes_of_every_size_keep_their_rules(strips_host):
    """Whole K shares to whole waves, and below 128 MB one order of a row's sums from 1 to 32 rows."""
    run = subprocess.run([strips_host], stdout=subprocess.PIPE, text=True)
    assert run.returncode == 0, run.stdout
