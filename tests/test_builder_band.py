"""The band of cells a row of the linear chirp is made from: what its cells read of the spectrum, and that what is held
against the cells outside covers all that they read.  The header is compiled for the host and every cell of every axis
is walked; nothing here runs on a GPU."""
import os
import shutil
import subprocess

import pytest

from paper_1307_3424_amd import build

SRC = r"""
#include "builder_band.h"
#include <algorithm>
#include <cstdio>

int main() {
    long bands = 0;
    for (int Ng = 64; Ng <= 4096; Ng *= 2) {
        const int room = Ng <= 256 ? Ng : Ng == 4096 ? 512 : 256;       // cells the kernels hold of an axis
        for (int W = 2; W <= 16; W += 2)
            for (double reach = 0.0; reach < Ng; reach += reach < 150 ? 0.75 : 0.2 * Ng)
                for (int q0 : {-3, 0, Ng / 2 - 1, Ng - 1}) {
                    const Band b = row_band(Ng, room, reach, W, q0, q0 + 5);
                    if (b.cnt == Ng) {
                        if (b.su != 0 || b.sv != 0) return std::printf("Ng %d: whole axis from %d, %d\n", Ng, b.su, b.sv), 1;
                        continue;
                    }
                    if (b.cnt > room) {                                 // only where the margin alone does not fit
                        if (2 * ((int)reach + 1 + BAND_MARGIN) - W + 2 <= room) return std::printf("Ng %d given up\n", Ng), 1;
                        continue;
                    }
                    ++bands;
                    const int from = outside_from(b, W);
                    if (from < 0 || from > Ng / 2) return std::printf("Ng %d: nothing held against the cells outside\n", Ng), 1;
                    for (int ax = 0; ax < 2; ++ax)
                        for (int p = 0; p < Ng; ++p) {                  // cell p of the axis from the band's first one on
                            const int q = (ax ? b.sv : b.su) + p, o = ax ? q0 + 5 : q0;
                            int lo = Ng, hi = 0;
                            for (int i = 0; i < W; ++i) {
                                const int d = (o + i - q) & (Ng - 1), a = std::min(d, Ng - d);
                                lo = std::min(lo, a);
                                hi = std::max(hi, a);
                            }
                            if (p < b.cnt ? hi > b.D : lo < from)
                                return std::printf("Ng %d W %d reach %g: cell %d of %d reads %d .. %d, D %d, from %d\n", Ng, W,
                                                   reach, p, b.cnt, lo, hi, b.D, from), 1;
                        }
                }
    }
    return bands > 1000 ? 0 : 1;
}
"""


@pytest.mark.skipif(shutil.which(build.hipcc()) is None, reason="needs hipcc")
def test_the_bound_covers_what_cells_outside_the_band_read(tmp_path):
    src, exe = tmp_path / "band.hip", tmp_path / "band"
    src.write_text(SRC)
    subprocess.run([build.hipcc(), "--offload-arch=gfx950", "--offload-host-only", "-O2", "-std=c++17", "-I", build.CSRC,
                    "-I", build.INCLUDE, str(src), "-o", str(exe)], check=True, timeout=300)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout
