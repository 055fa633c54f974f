"""The bounds-checked loads of the kernels (buffer_load* of common.hpp) keep the whole
offset where the range check sees it: in the per-lane offset and the instruction's
immediate, never in the scalar offset.  Checked on the code generated for gfx950."""
import glob
import os
import re
import shutil
import subprocess

import pytest

from paper_2607_27591_amd import build as B

PROBE = r"""
#include "common.hpp"
using namespace prox;
extern "C" __global__ void probe(const unsigned char *p, uint32_t bytes, uint32_t *out) {
    const auto rs = buffer_of(p, bytes);
    const int l = threadIdx.x;
    uint32_t s = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {   // offsets below and past the 4095 of the immediate
        s += buffer_load16(rs, (k * 1536 + l) * 2);
        s += buffer_load32(rs, (k * 1024 + l) * 4);
        s += buffer_load64(rs, (k * 1024 + l) * 8).y;
        s += buffer_load128(rs, (k * 1024 + l) * 16).w;
    }
    out[l] = s;
}
"""


@pytest.mark.skipif(shutil.which(B.HIPCC) is None, reason="needs hipcc")
def test_scalar_offset_stays_zero(tmp_path):
    src, asm = tmp_path / "probe.hip", tmp_path / "probe.s"
    src.write_text(PROBE)
    subprocess.run([B.HIPCC, *B.CFLAGS, "--cuda-device-only", "-S", str(src), "-o", str(asm)],
                   check=True, capture_output=True)
    loads = re.findall(r"buffer_load_\w+ [^,]+, [^,]+, s\[[^\]]+\], (\S+)", asm.read_text())
    assert len(loads) == 16
    assert set(loads) == {"0"}


def test_only_these_helpers_load_through_buffers():
    for path in glob.glob(os.path.join(B.CSRC, "*")):
        n = open(path).read().count("raw_buffer_load")
        assert n == (4 if os.path.basename(path) == "common.hpp" else 0), path
