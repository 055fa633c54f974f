"""Host-side checks of the C-ABI that need no GPU.

The library must load, export every entry point include/prox.h declares, and
reject bad arguments with the documented status codes before any HIP call
(the pointers passed below are never dereferenced: validation fails first).
"""
import ctypes
import os
import re
import subprocess

import pytest

from paper_2607_27591_amd import prox

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "prox.h")

OK, INVALID, UNSUPPORTED, WORKSPACE = 0, 1, 2, 3
FAKE = 0x100000          # 256-byte aligned, never dereferenced
MISALIGNED = 0x100001


def _declared():
    text = open(HEADER).read()
    return sorted(set(re.findall(r"\b(prox_[a-z_]+)\s*\(", text)))


@pytest.mark.parametrize("lang", ["c", "c++"])
def test_header_compiles_as_c_and_cxx(tmp_path, lang):
    # The boundary is a C header: a C11 and a C++17 translation unit both take
    # it, and in C++ an out-of-range enum value (which C callers may pass) is a
    # valid value of the enum's fixed int type.
    comp = {"c": ["gcc", "-std=c11"], "c++": ["g++", "-std=c++17"]}[lang]
    src = tmp_path / ("t.c" if lang == "c" else "t.cpp")
    src.write_text('#include "prox.h"\n'
                   'int main(void) { prox_qfmt f = (prox_qfmt)7; prox_dtype t = PROX_BF16;\n'
                   '  return (int)f + (int)t + (int)sizeof(prox_status); }\n')
    r = subprocess.run([*comp, "-fsyntax-only", "-Wall", "-Werror", "-D__HIP_PLATFORM_AMD__",
                        "-I", os.path.dirname(HEADER), "-I", "/opt/rocm/include", str(src)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr


def test_header_declares_the_boundary():
    names = _declared()
    for must in ["prox_pack_proxy", "prox_ffn_dense", "prox_ffn_sparse", "prox_ffn_sparse_tau",
                 "prox_proxy_bytes", "prox_workspace_bytes", "prox_strerror"]:
        assert must in names


def test_library_exports_every_declared_symbol():
    L = prox.lib()
    for name in _declared():
        assert hasattr(L, name), name
    out = subprocess.run(["nm", "-D", "--defined-only", prox.LIB_PATH], capture_output=True,
                         text=True, check=True).stdout
    exported = set(re.findall(r"\sT\s(prox_\w+)", out))
    assert set(_declared()) <= exported


def test_binding_constants_match_the_header():
    text = open(HEADER).read()
    assert int(re.search(r"#define PROX_MAX_BATCH\s+(\d+)", text).group(1)) == prox.MAX_BATCH
    assert int(re.search(r"#define PROX_SPARSE_STAGES\s+(\d+)", text).group(1)) == prox.SPARSE_STAGES


def test_library_is_gfx950_only():
    out = subprocess.run(["strings", prox.LIB_PATH], capture_output=True, text=True).stdout
    assert "gfx950" in out
    for other in ["gfx90a", "gfx942", "gfx1100", "sm_"]:
        assert f"amdgcn-amd-amdhsa--{other}" not in out


def _weights(d=1024, f=3072, dtype=prox.BF16, g=FAKE, u=FAKE, dn=FAKE, act=prox.SILU):
    return prox._Weights(d, f, dtype, g, u, dn, act)


def _proxy(fmt=prox.INT4, group=128, blob=FAKE, nbytes=1 << 40):
    return prox._Proxy(fmt, group, blob, nbytes)


def _sparse(w=None, p=None, x=FAKE, B=1, k_in=10, k_ff=10, y=FAKE, mask=FAKE, ws=FAKE,
            ws_bytes=1 << 40):
    L = prox.lib()
    w = w if w is not None else _weights()
    p = p if p is not None else _proxy()
    return L.prox_ffn_sparse(ctypes.byref(w), ctypes.byref(p), x, B, k_in, k_ff, y, mask, None,
                             None, ws, ws_bytes, None)


def test_sizes():
    assert prox.proxy_bytes(8192, 28672, prox.INT4, 128) > 2 * 8192 * 28672 // 2
    assert prox.proxy_bytes(1024, 3072, prox.INT8, 1024) > 2 * 1024 * 3072
    assert prox.proxy_bytes(1000, 3072, prox.INT4, 128) == 0       # d % 128
    assert prox.proxy_bytes(1024, 3072, prox.INT4, 96) == 0        # group % 128
    assert prox.proxy_bytes(1024, 3072, prox.INT4, 512 * 3) == 0   # d % group
    assert prox.proxy_bytes(1024, 3072, 7, 128) == 0               # fmt
    assert prox.workspace_bytes(4096, 12288, 1) > 0
    assert prox.workspace_bytes(4096, 12288, 65) == 0
    assert prox.workspace_bytes(4096, 12288, 0) == 0
    assert prox.workspace_bytes(32768, 12288, 1) == 0
    assert prox.workspace_bytes(4096, 65537, 1) == 0
    assert prox.workspace_bytes(4096, 12288, 16) > prox.workspace_bytes(4096, 12288, 1)
    assert prox.workspace_bytes(4096, 12288, 64) > prox.workspace_bytes(4096, 12288, 16)
    # Partial y sized by path: up to 8 rows both weight kinds take one row set
    # per Stage 2 workgroup; past 8 rows at d_model >= 4096 the 16-bit path
    # keeps 16 groups or fewer (plus s; the size stays that of 8 rows), INT4
    # weights still 256 workgroups.
    for B in (1, 4, 8):
        assert prox.workspace_bytes(8192, 28672, B) == prox.workspace_bytes(8192, 28672, B, w4=True)
    assert prox.workspace_bytes(4096, 14336, 16) < prox.workspace_bytes(4096, 14336, 16, w4=True)
    assert prox.workspace_bytes(1024, 3072, 16) == prox.workspace_bytes(1024, 3072, 16, w4=True)
    assert prox.workspace_bytes(4096, 14336, 16) < 256 * 16 * 4096 * 4
    assert prox.workspace_bytes(4096, 12288, 65, w4=True) == 0


@pytest.mark.parametrize("w4", [False, True])
@pytest.mark.parametrize("d,f", [(1024, 3072), (4096, 14336), (4096, 100), (4224, 65536),
                                 (8192, 28672), (16384, 1), (16384, 65536)])
def test_workspace_of_the_largest_batch_serves_the_smaller_ones(d, f, w4):
    sizes = [prox.workspace_bytes(d, f, B, w4=w4) for B in range(1, 65)]
    assert sizes == sorted(sizes)
    # The 8-row kernel's partial y alone: 256 sets of 1, 2, 4 or 8 rows.
    for B, n in enumerate(sizes, 1):
        assert n >= 256 * (1 if B < 2 else 2 if B < 3 else 4 if B < 5 else 8) * d * 4
    if not w4:   # INT4 base weights never take less
        assert all(prox.workspace_bytes(d, f, B, w4=True) >= n for B, n in enumerate(sizes, 1))


def test_stage1_kernel_selection():
    # The 16-row matrix-core Stage 1 takes INT4 proxies for 5 to 16 batch rows up to
    # d_model 4096, 16 rows per launch while the kept-row list and 16 x rows fit the
    # LDS, else 8; every other call (0) takes the small-batch, the batch or, for INT8
    # and unquantised proxies, the dot-product kernel.
    rows = prox.stage1_mfma_rows
    for d in (128, 1024, 4096):
        for B in (1, 4, 5, 16, 17, 64):
            assert rows(d, prox.INT4, 128, B, d // 2) == (16 if 5 <= B <= 16 else 0), (d, B)
            # Threshold mode and a full keep: the list of every input.
            want = (8 if d == 4096 else 16) if 5 <= B <= 16 else 0
            assert rows(d, prox.INT4, 128, B, d) == want, (d, B)
    for d in (4224, 8192, 8320, 16384):
        for B in (1, 2, 4, 5, 16, 17, 64):
            assert rows(d, prox.INT4, 128, B, d // 3) == 0, (d, B)
            assert rows(d, prox.INT4, 128, B, d) == 0, (d, B)
    assert rows(4096, prox.INT4, 4096, 8, 3968) == 16      # per-row groups: few pads
    assert rows(4096, prox.INT8, 128, 16, 2048) == 0
    assert rows(4096, prox.NONE, 4096, 16, 2048) == 0
    assert rows(4096, prox.INT4, 96, 16, 2048) == 0        # group % 128
    assert rows(4096, prox.INT4, 128, 65, 2048) == 0       # batch
    assert rows(4096, prox.INT4, 128, 0, 2048) == 0
    assert rows(4096, prox.INT4, 128, 16, 0) == 0          # k_in
    assert rows(4096, prox.INT4, 128, 16, 4097) == 0


def test_stage2_kernel_selection():
    # More than eight batch rows of 16-bit weights with d_model >= 4096 take
    # the matrix-core Stage 2 (tiles of 16 rows); otherwise the VALU kernel
    # (8 rows per launch, fewer for INT4 weights at wide d_model).
    rows = prox.stage2_rows
    assert rows(4096, 14336, False, 16) == 16
    assert rows(4096, 14336, False, 9) == 16
    assert rows(4096, 14336, False, 8) == 8
    assert rows(8192, 28672, False, 64) == 16
    assert rows(16384, 320, False, 12) == 16
    assert rows(2048, 3000, False, 16) == 8         # narrow d: VALU kernel
    assert rows(8192, 28672, True, 16) == 4         # INT4 weights: x rows in LDS
    assert rows(16384, 320, True, 16) == 2
    assert rows(4096, 14336, False, 65) == 0        # batch
    assert rows(4096, 14336, False, 0) == 0
    assert rows(4000, 14336, False, 16) == 0        # d_model % 128


def _noalloc(w=None, p=None, x=FAKE, B=1, k_in=10, k_ff=10, y=FAKE, mask=FAKE):
    L = prox.lib()
    w = w if w is not None else _weights()
    p = p if p is not None else _proxy()
    return L.prox_ffn_sparse_noalloc(ctypes.byref(w), ctypes.byref(p), x, B, k_in, k_ff, y,
                                     mask, None, None, None)


def test_noalloc_checks_before_any_hip_call():
    """The entry point without a workspace validates like prox_ffn_sparse and
    rejects a call whose workspace would not fit its scratch, all before its
    first HIP call (the scratch lookup)."""
    cap = prox.noalloc_max_bytes()
    assert cap == 32 << 20
    assert _noalloc(k_in=0) == INVALID
    assert _noalloc(B=65) == INVALID
    assert _noalloc(x=None) == INVALID
    assert _noalloc(y=MISALIGNED) == INVALID
    assert _noalloc(p=_proxy(group=96)) == UNSUPPORTED
    assert _noalloc(p=_proxy(nbytes=100)) == WORKSPACE
    # 8192 x 28672: batch 2 fits the scratch, batch 4 does not.
    big = _weights(d=8192, f=28672)
    assert prox.workspace_bytes(8192, 28672, 2) <= cap < prox.workspace_bytes(8192, 28672, 4)
    assert _noalloc(w=big, B=4, k_in=3277, k_ff=8602) == WORKSPACE
    assert _noalloc(w=_weights(d=16384, f=65536), B=8, k_in=100, k_ff=100) == WORKSPACE


def test_sparse_rejects_bad_arguments():
    L = prox.lib()
    assert _sparse(k_in=0) == INVALID
    assert _sparse(k_in=1025) == INVALID
    assert _sparse(k_ff=0) == INVALID
    assert _sparse(k_ff=3073) == INVALID
    assert _sparse(B=0) == INVALID
    assert _sparse(B=65) == INVALID
    assert _sparse(x=None) == INVALID
    assert _sparse(y=None) == INVALID
    assert _sparse(mask=None) == INVALID
    assert _sparse(ws=None) == INVALID
    assert _sparse(x=MISALIGNED) == INVALID
    assert _sparse(ws=FAKE + 16) == INVALID
    assert _sparse(w=_weights(g=0)) == INVALID
    assert _sparse(w=_weights(dn=MISALIGNED)) == INVALID
    assert _sparse(w=_weights(dtype=5)) == INVALID
    assert _sparse(w=_weights(d=1000)) == UNSUPPORTED
    assert _sparse(w=_weights(d=32768)) == UNSUPPORTED
    assert _sparse(p=_proxy(group=96)) == UNSUPPORTED
    assert _sparse(p=_proxy(fmt=9)) == UNSUPPORTED
    assert _sparse(p=_proxy(nbytes=100)) == WORKSPACE
    assert _sparse(ws_bytes=100) == WORKSPACE
    p = _proxy()
    w = _weights()
    assert L.prox_ffn_sparse(ctypes.byref(w), None, FAKE, 1, 1, 1, FAKE, FAKE, None, None, FAKE,
                             1 << 40, None) == INVALID
    assert L.prox_ffn_sparse(None, ctypes.byref(p), FAKE, 1, 1, 1, FAKE, FAKE, None, None, FAKE,
                             1 << 40, None) == INVALID
    assert L.prox_ffn_sparse_staged(ctypes.byref(w), ctypes.byref(p), FAKE, 1, 1, 1, FAKE, FAKE,
                                    None, None, FAKE, 1 << 40, None, None) == INVALID


def test_sparse_tau_rejects_bad_arguments():
    L = prox.lib()
    w, p = _weights(), _proxy()
    nan = float("nan")

    def call(tau_x=0.5, tau_s=0.1, B=1, counts=None, mask=FAKE, ws_bytes=1 << 40):
        return L.prox_ffn_sparse_tau(ctypes.byref(w), ctypes.byref(p), FAKE, B, tau_x, tau_s,
                                     FAKE, mask, None, None, counts, FAKE, ws_bytes, None)

    assert call(tau_x=nan) == INVALID
    assert call(tau_s=nan) == INVALID
    assert call(counts=MISALIGNED) == INVALID
    assert call(B=0) == INVALID
    assert call(B=65) == INVALID
    assert call(mask=None) == INVALID
    assert call(ws_bytes=10) == WORKSPACE
    assert call(tau_x=float("inf"), ws_bytes=10) == WORKSPACE   # +inf is a valid threshold


def test_dense_pack_norm_reject_bad_arguments():
    L = prox.lib()
    w = _weights()
    assert L.prox_ffn_dense(ctypes.byref(w), FAKE, 0, FAKE, FAKE, 1 << 40, None) == INVALID
    assert L.prox_ffn_dense(ctypes.byref(w), FAKE, 1, FAKE, FAKE, 10, None) == WORKSPACE
    assert L.prox_ffn_dense(ctypes.byref(w), MISALIGNED, 1, FAKE, FAKE, 1 << 40, None) == INVALID
    p = _proxy(nbytes=10)
    assert L.prox_pack_proxy(ctypes.byref(w), ctypes.byref(p), None) == WORKSPACE
    p = _proxy(group=1024 * 3)
    assert L.prox_pack_proxy(ctypes.byref(w), ctypes.byref(p), None) == UNSUPPORTED
    p = _proxy(blob=None)
    assert L.prox_pack_proxy(ctypes.byref(w), ctypes.byref(p), None) == INVALID
    p = _proxy()
    assert L.prox_unpack_proxy(ctypes.byref(p), 1024, 3072, None, FAKE, FAKE, FAKE, None) == INVALID
    assert L.prox_add_rmsnorm(FAKE, FAKE, 0, 1024, 1, ctypes.c_float(1e-6), FAKE, None) == INVALID
    assert L.prox_add_rmsnorm(FAKE, FAKE, 1, 1024, 3, ctypes.c_float(1e-6), FAKE, None) == INVALID
    assert L.prox_add_rmsnorm(FAKE, FAKE, 1, 1024, 1, ctypes.c_float(-1.0), FAKE, None) == INVALID


def test_strerror_and_stage_names():
    for s in range(5):
        assert prox.strerror(s)
    assert prox.stage_names() == ["proxy_gemv_score", "stage2_select_gate_up_down", "reduce_y"]
    assert prox.lib().prox_sparse_stage_name(3) is None


def _w4(d=1024, f=3072, dtype=prox.BF16, group=128, act=prox.SILU, blob=FAKE, nbytes=1 << 40):
    return prox._W4(dtype, d, f, group, act, blob, nbytes)


def test_w4_sizes_and_rejects_bad_arguments():
    d, f = 1024, 3072
    n = prox.w4_bytes(d, f, 128)
    assert n >= 3 * f * (d // 2) + 3 * f * (d // 128) * 2
    assert prox.w4_bytes(d, f, 256) < n                  # fewer scales
    assert prox.w4_bytes(d, f, 96) == 0                   # group % 128
    assert prox.w4_bytes(d, f, 384) == 0                  # d % group
    assert prox.w4_bytes(1000, f, 128) == 0               # d % 128
    L = prox.lib()

    def dense(q, x=FAKE, B=1, y=FAKE, ws=FAKE, ws_bytes=1 << 40):
        return L.prox_ffn_dense_w4(ctypes.byref(q), x, B, y, ws, ws_bytes, None)

    def sparse(q, k_in=10, k_ff=10, ws_bytes=1 << 40):
        p = _proxy()
        return L.prox_ffn_sparse_w4(ctypes.byref(q), ctypes.byref(p), FAKE, 1, k_in, k_ff, FAKE,
                                    FAKE, None, None, FAKE, ws_bytes, None, None)

    assert L.prox_ffn_dense_w4(None, FAKE, 1, FAKE, FAKE, 1 << 40, None) == INVALID
    assert dense(_w4(blob=0)) == INVALID
    assert dense(_w4(blob=FAKE + 16)) == INVALID          # 256-byte alignment
    assert dense(_w4(dtype=5)) == INVALID
    assert dense(_w4(act=7)) == INVALID
    assert dense(_w4(group=96)) == UNSUPPORTED
    assert dense(_w4(d=1000)) == UNSUPPORTED
    assert dense(_w4(nbytes=100)) == WORKSPACE
    assert dense(_w4(), x=None) == INVALID
    assert dense(_w4(), B=65) == INVALID
    assert dense(_w4(), ws_bytes=100) == WORKSPACE
    assert sparse(_w4(), k_in=0) == INVALID
    assert sparse(_w4(), k_ff=3073) == INVALID
    assert sparse(_w4(group=96)) == UNSUPPORTED
    assert sparse(_w4(), ws_bytes=100) == WORKSPACE
    q = _w4()
    assert L.prox_unpack_w4(ctypes.byref(q), 3, FAKE, FAKE, None) == INVALID
    assert L.prox_unpack_w4(ctypes.byref(q), 0, None, FAKE, None) == INVALID
    w = _weights()
    assert L.prox_pack_w4(ctypes.byref(w), ctypes.byref(_w4(d=2048)), None) == INVALID
    assert L.prox_pack_w4(ctypes.byref(w), ctypes.byref(_w4(dtype=prox.F16)), None) == INVALID
