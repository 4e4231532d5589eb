"""The layout of a KV page on the CPU (csrc/common.h in the host program kv_page_host.cpp): for every even head size up to 256
each position and dimension of K and V has an element of its own inside the page's slab, and 16-byte reads start on one."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not found")
def test_every_element_of_a_page_has_its_own_place(tmp_path):
    exe = str(tmp_path / "kv_page_host")
    res = subprocess.run([HIPCC, "--offload-arch=gfx950", "-O1", "-std=c++17", os.path.join(HERE, "kv_page_host.cpp"), "-o", exe],
                         stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert res.returncode == 0, res.stdout[-2000:]
    run = subprocess.run([exe], stdout=subprocess.PIPE, text=True)
    assert run.returncode == 0, run.stdout
