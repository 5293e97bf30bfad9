"""The rule that picks the form of the point backward (csrc/point_forms.hpp),
compiled for the host: the sizes of the GPU tests reach the forms they name."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# (H, W, K, points of each cloud, radius, gradients of zbuf and dists): calls that
# take the box-staged and the one-thread-per-point form, on the GPU in
# test_gpu_splits.py
BOX = [(64, 64, 4, [300], 0.36, True, True), (64, 64, 8, [250, 0, 90], 0.36, False, True),
       (64, 64, 7, [300], 0.37, True, False), (43, 70, 3, [40, 200], 0.5, True, True),
       (40, 96, 1, [200], 0.4, True, True)]
POINTS = [(64, 64, 8, [300], 0.36, True, True), (64, 64, 32, [400], 0.36, True, True),
          (43, 70, 6, [100, 0, 120], 0.6, True, True), (40, 96, 64, [150], 0.5, False, True),
          (33, 40, 16, [200], 1.1, True, False)]

MAIN = r"""
#include <cstdio>
#include <cstdlib>
#include "%s/paper_2007_08501_amd/csrc/point_forms.hpp"
int main(int argc, char** argv) {
    const int N = atoi(argv[1]), H = atoi(argv[2]), W = atoi(argv[3]), K = atoi(argv[4]);
    const long long P = atoll(argv[5]);
    const float r = (float)atof(argv[6]);
    const int gz = atoi(argv[7]), gd = atoi(argv[8]);
    const int sx = rast::pt_span(r, W), sy = rast::pt_span(r, H);
    const long long T = (long long)N * ((H + 7) / 8) * ((W + 7) / 8), ncell = (long long)(sx + 1) * (sy + 1);
    const rast::PtSlots s = rast::pt_slots(P, T, ncell);
    std::printf("%%d %%d %%d %%zu\n", (int)rast::pt_bwd_form(N, H, W, K, P, r, gz, gd),
                s.lg_cap ? 1 << s.lg_cap : 0, s.lg_cap ? 1 << s.lg_table : 0, s.bytes);
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("forms")
    (d / "main.cpp").write_text(MAIN % ROOT)
    subprocess.check_call(["g++", "-std=c++17", "-O1", str(d / "main.cpp"), "-o", str(d / "forms")])

    def ask(N, H, W, K, P, r, gz=True, gd=True):
        out = subprocess.check_output([str(d / "forms")] + [str(x) for x in (N, H, W, K, P, repr(float(r)), int(gz),
                                                                             int(gd))], text=True).split()
        return ("slots", "box", "points")[int(out[0])], int(out[1]), int(out[2]), int(out[3])

    return ask


def test_chunk_capacities(rule):
    # a tile's chunk is the largest of which eight share a compute unit's LDS, at any density
    for P in (1, 500, 20000):
        assert rule(1, 256, 256, 8, P, 2.0 / 256)[:2] == ("slots", 512)
        assert rule(1, 256, 256, 8, P, 5.0 / 256)[:2] == ("slots", 256)
        assert rule(1, 256, 256, 8, P, 9.0 / 256)[:2] == ("slots", 128)
    # and more where the tiles hold more on average
    assert rule(8, 256, 256, 50, 1600000, 0.01)[:2] == ("slots", 1024)
    # within the LDS of a workgroup for every range and density
    for P in (1, 10 ** 4, 10 ** 6, 2 ** 30):
        for rpx in range(0, 40):
            form, cap, table, lds = rule(1, 256, 256, 8, P, rpx / 256)
            assert (form == "slots") == ((rpx + 1) ** 2 <= 492)
            assert form != "slots" or (128 <= cap <= 1024 and 2 * cap <= table and 0 < lds <= 65536)


def test_sizes_of_the_gpu_tests(rule):
    # tiles of several chunks
    for P in (512, 513, 1536, 4253, 6024):
        assert rule(1, 64, 64, 40, P, 2.0 / 64)[:2] == ("slots", 512)
    assert rule(4, 104, 104, 2, 180000, 13.0 / 104)[:2] == ("slots", 256)
    assert rule(4, 104, 104, 1, 180000, 19.0 / 104)[:2] == ("slots", 128)


@pytest.mark.parametrize("form,cases", [("box", BOX), ("points", POINTS)])
def test_forms_of_large_discs(rule, form, cases):
    for H, W, K, sizes, r, gz, gd in cases:
        assert rule(len(sizes), H, W, K, sum(sizes), r, gz, gd)[0] == form, (H, W, K, r)
