"""Memory layouts that share space, swept on the host: the batch Stage 1's scratch lies
over the partial-y area of the same call, which Stage 2 fills afterwards."""
import shutil
import subprocess

import pytest

from paper_2607_27591_amd import build as B

SWEEP = r"""
#define __host__
#define __device__
#include "layout.hpp"
#include <cstdio>
using namespace prox;
int main() {
    long n = 0;
    for (int d = 128; d <= kMaxDModel; d += 128)
        for (int g = 128; g <= d; g += 128) {
            if (d % g) continue;
            for (int batch = 2; batch <= 64; ++batch)
                for (int wq : {4, 16})
                    for (int f : {1, 300, 28672}) {
                        const WsLayout L(d, f, batch, wq);
                        const BatchScratch S(d, g, stage2_row_tiles(batch));
                        if (S.total > L.sbuf - L.ypart) {
                            std::printf("d %d group %d batch %d wq %d\n", d, g, batch, wq);
                            return 1;
                        }
                        ++n;
                    }
        }
    std::printf("%ld\n", n);
    return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_batch_scratch_fits_the_partial_y_area(tmp_path):
    src, exe = tmp_path / "sweep.cpp", tmp_path / "sweep"
    src.write_text(SWEEP)
    subprocess.run(["g++", "-std=c++17", "-O1", "-include", "initializer_list", "-I", B.CSRC, str(src),
                    "-o", str(exe)], check=True, capture_output=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
    assert int(r.stdout) > 100000
