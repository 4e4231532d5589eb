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
    """Whole K shares to whole waves, and below 128 MB one order of a row's sums from 1 to 32 rows; half strips and every block of a blocked launch once."""
    run = subprocess.run([strips_host], stdout=subprocess.PIPE, text=True)
    assert run.returncode == 0, run.stdout


@pytest.mark.parametrize("ntiles,ktiles,want", [(8016, 64, "1 4 1"), (5000, 96, "1 4 1"), (5000, 128, "1 4 1"), (8016, 128, "1 8 1"), (2000, 256, "1 8 1"),
                                                (1792, 64, "1 7 1"), (1792, 128, "1 7 1"), (3584, 256, "1 7 1"), (1376, 128, "1 6 1"), (1024, 64, "1 4 1")])
def test_of_equal_deals_four_waves_for_a_short_k(strips_host, ntiles, ktiles, want):
    assert subprocess.run([strips_host, str(ntiles), str(ktiles), "9"], stdout=subprocess.PIPE, text=True, check=True).stdout.strip() == want


# weight tiles, k-tiles: kernel at 17, 24 and 32 rows
@pytest.mark.parametrize("ntiles,ktiles,want", [
    (640, 256, ["rows"] * 3),                           # 70B QKV: 160 workgroups of strips
    (320, 432, ["rows"] * 3),                           # 13B down
    (512, 256, ["2 4 4"] * 3),                          # 70B O
    (512, 896, ["2 4 4", "rows", "rows"]),              # 70B down
    (1792, 128, ["7 8 8"] * 3), (3584, 256, ["7 8 8"] * 3), (8016, 128, ["7 8 8"] * 3),      # 8B, 70B gate/up, 8B head
    (1376, 128, ["7 8 8"] * 3), (2752, 256, ["7 8 8"] * 3),                                  # a third more than an even deal
    (8016, 96, ["rows"] * 3), (2000, 256, ["rows"] * 3),
    (2000, 128, ["1 8 1"] * 3),
    (256, 448, ["1 8 8"] * 3), (384, 128, ["2 4 4"] * 3),                                    # below 128 MB
])
def test_calls_of_17_to_32_rows_get_the_quicker_kernel(strips_host, ntiles, ktiles, want):
    got = [subprocess.run([strips_host, str(ntiles), str(ktiles), str(m)], stdout=subprocess.PIPE, text=True, check=True).stdout.strip()
           for m in (17, 24, 32)]
    assert got == want


# the shapes that the GPU tests of the few-row GEMM are made for: weight tiles, k-tiles, at 8 and 18 rows (gate/up, then the large heads)
@pytest.mark.parametrize("ntiles,ktiles,few,more", [
    (1792, 8, "1 7 1", "1 7 1"), (1788, 9, "1 7 1", "1 7 1"), (1794, 9, "1 4 1", "1 4 1"), (770, 9, "1 4 1", "1 4 1"), (642, 9, "4 8 8", "4 8 8"),
    (386, 8, "2 4 4", "2 4 4"), (224, 256, "1 4 4", "1 4 4"), (256, 344, "1 4 4", "1 4 4"), (256, 448, "1 8 8", "1 8 8"), (512, 8, "1 4 4", "2 4 4"),
    (1790, 75, "1 7 1", "7 8 8"), (1790, 85, "1 7 1", "7 8 8"), (1790, 97, "1 7 1", "7 8 8"), (1376, 97, "1 6 1", "7 8 8"),
    (3584, 256, "1 7 1", "7 8 8"), (640, 256, "4 8 8", "rows"), (2000, 256, "1 8 1", "rows")])
def test_shapes_of_the_gpu_tests(strips_host, ntiles, ktiles, few, more):
    got = [subprocess.run([strips_host, str(ntiles), str(ktiles), m], stdout=subprocess.PIPE, text=True, check=True).stdout.strip() for m in ("8", "18")]
    assert got == [few, more]


# down projections of 600 to 1024 rows, the form that measured quicker
@pytest.mark.parametrize("ntiles,ktiles,blocks,parts", [
    (256, 448, [690, 784, 880, 928, 1024], [600, 736, 768]),
    (320, 432, [690, 736, 768], [600]),
    (192, 256, [690, 736, 768, 784, 880, 928], [600]),
    (128, 256, [784, 832, 928, 1016], [600, 720, 736, 768]),
    (224, 592, [784, 832, 928, 976], [600, 690, 720, 768, 880]),
    (320, 864, [1025], [690, 736, 768, 1024]),
    (512, 896, [900, 1024], [520, 700]),
    (256, 128, [513, 1024], []),
])
def test_narrow_matrix_of_a_long_k_runs_in_the_quicker_form(strips_host, ntiles, ktiles, blocks, parts):
    form = {rows: subprocess.run([strips_host, "narrow", str(ntiles), str(ktiles), str(rows)], stdout=subprocess.PIPE, text=True, check=True).stdout.strip()
            for rows in blocks + parts}
    assert form == {**{rows: "blocks" for rows in blocks}, **{rows: "parts" for rows in parts}}


# blocked calls whose forms measured furthest apart: us in the form named here, and in the one that a model fitted to two widths named
@pytest.mark.parametrize("kind,ntiles,ktiles,rows,want", [
    ("gateup", 1792, 128, 1040, "12 16"),               # 208, 224
    ("gateup", 3584, 256, 576, "16 16"),                # 480, 530
    ("other", 384, 512, 2600, "12 12"),                 # 467, 591
    ("other", 320, 432, 1300, "8 16"),                  # 176, 184
    ("other", 256, 448, 1096, "8 12"), ("other", 256, 448, 2048, "8 16"), ("other", 384, 128, 2048, "12 16"), ("other", 256, 448, 4096, "16 16"),
])
def test_form_of_a_blocked_call(strips_host, kind, ntiles, ktiles, rows, want):
    assert subprocess.run([strips_host, kind, str(ntiles), str(ktiles), str(rows)], stdout=subprocess.PIPE, text=True, check=True).stdout.strip() == want
