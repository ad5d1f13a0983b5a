"""The strips of the fused variable-coefficient passes (host check of the
kernels' own mapping, no device): every cell of a row is stored by exactly one
lane of one strip, for every row length.  The reverse sweep adds to its
accumulator in place, so a second storing lane would count a step's terms
twice."""
import os
import subprocess

from conftest import ROOT

SRC = r'''
#include <cstdio>
#include <vector>
#include "hx_vcstrip.hpp"
using namespace hx;
int main() {
    for (int64_t nx = 4; nx <= 4 * kVcStripCols + 8; ++nx) {
        std::vector<int> stores(nx, 0);
        for (int64_t s = 0; s < vc_strips(nx); ++s)
            for (int lane = 0; lane < 64; ++lane) {
                const int64_t x = vc_lane_column(s, lane);
                for (int j = 0; j < kVcCols; ++j)
                    if (vc_lane_stores(lane, x, nx) && x + j >= 0 && x + j < nx) ++stores[x + j];
            }
        for (int64_t x = 0; x < nx; ++x)
            if (stores[x] != 1) {
                std::printf("nx %lld column %lld: %d stores\n", (long long)nx, (long long)x,
                            stores[x]);
                return 1;
            }
    }
    return 0;
}
'''


def test_every_cell_has_one_storing_lane(tmp_path):
    src, exe = tmp_path / "strips.cpp", str(tmp_path / "strips")
    src.write_text(SRC)
    inc = os.path.join(ROOT, "paper_1810_11482_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", f"-I{inc}", str(src), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
