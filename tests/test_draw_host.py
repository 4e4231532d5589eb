"""The decisions of the inverse-CDF draw on the CPU: csrc/draw.h compiled into a host program (tests/draw_host.cpp) that forms
a workgroup's sums in the kernel's order, over residual rows max(0, p - q) and millions of uniform numbers, half of them within
a few units in the last place of an edge between lanes or chunk groups, where the prefixes of neighbours are rounded apart."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def draw_host(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not found")
    exe = str(tmp_path_factory.mktemp("draw") / "draw_host")
    res = subprocess.run([HIPCC, "--offload-arch=gfx950", "-O2", "-std=c++17", "-ffp-contract=off", os.path.join(HERE, "draw_host.cpp"),
                          "-o", exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert res.returncode == 0, res.stdout[-2000:]
    return exe


# 130: one wave; 32000, 128256: several chunks per wave; 300003: more than 64 chunks per wave, two to a group
@pytest.mark.parametrize("vocab", [130, 1000, 32000, 128256, 300003])
def test_no_draw_returns_a_token_of_weight_zero(draw_host, vocab):
    out = subprocess.run([draw_host, str(vocab), "45", "20000", "7"], stdout=subprocess.PIPE, text=True, check=True).stdout
    draws, zero, far = map(int, out.split())
    assert draws > 800000 and zero == 0, (draws, zero)
    # the interval [cdf(tok - 1), cdf(tok)] against u * total: partial sums of a dozen levels on both sides, 2^-24 each
    assert far == 0, (draws, far)
