"""The row factors of the deferred RMSNorm on the CPU: the order of their sums (csrc/norm_factor.h in the host program
norm_factor_host.cpp), and the compiled gfx950 code of the kernel, whose time is trips to memory."""
import os
import re
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
pytestmark = pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not found")


def test_sums_keep_their_order_at_every_number_of_partials(tmp_path):
    exe = str(tmp_path / "norm_factor_host")
    res = subprocess.run([HIPCC, "--offload-arch=gfx950", "-O2", "-std=c++17", "-ffp-contract=off", os.path.join(HERE, "norm_factor_host.cpp"),
                          "-o", exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert res.returncode == 0, res.stdout[-2000:]
    run = subprocess.run([exe], stdout=subprocess.PIPE, text=True)
    assert run.returncode == 0, run.stdout


def trips(asm_text):
    """Loads of every group of loads of norm_factor_kernel that are requested with no wait for one of them in between."""
    groups, n, inside = [], 0, False
    for line in asm_text.splitlines():
        if re.match(r"^_Z\d+norm_factor_kernel\w*:", line):
            inside = True
        t = line.split()
        if not inside or not t:
            continue
        if t[0] == "s_endpgm":
            break
        if t[0].startswith("global_load"):
            n += 1
        elif n and t[0] == "s_waitcnt" and "vmcnt" in line:
            groups.append(n)
            n = 0
    return groups


def test_all_loads_of_a_turn_are_in_flight_whatever_the_number_of_partials(tmp_path):
    out = tmp_path / "norm_factor.s"
    res = subprocess.run([HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-fno-gpu-rdc", "-Xclang", "-target-feature", "-Xclang",
                          "-packed-fp32-ops", "--cuda-device-only", "-S", os.path.join(HERE, "norm_factor_host.cpp"), "-o", str(out)],
                         stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert res.returncode == 0, res.stdout[-2000:]
    assert trips(out.read_text()) == [8]          # two chains of four a lane, in one group, and no other loads (remainders) beside it


def test_scanner_sees_a_serial_chain():
    one = " global_load_dword v1, v[2:3], off\n s_waitcnt vmcnt(0)\n v_add_f32 v4, v4, v1\n"
    assert trips("_Z18norm_factor_kernelPKf:\n" + one * 3 + " s_endpgm\n") == [1, 1, 1]
