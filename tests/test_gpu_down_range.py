"""Extremes of s = act(g) u in the matrix-core down projection (9 rows and more of
bf16 weights), which splits s into bf16 parts: an s that overflows fp32 gives
infinities of the right sign, one beyond the largest bf16 stays finite, and tiny ones
keep their precision, as on the 8-row kernel."""
import numpy as np
import pytest
import torch

from paper_2607_27591_amd import prox
from paper_2607_27591_amd import workloads as W

pytestmark = pytest.mark.gpu

D, F, B = 4096, 96, 16
CH, I0, I1 = 37, 1234, 77   # the channel, and the inputs of rows 0 and 1


def _rounded(v):
    return W.bits_to_f32(W.to_bits(v.astype(np.float32), W.DT_BF16), W.DT_BF16)


def _call(gate, up, down, x, sparse):
    w = prox.Weights(*(prox.from_bits(W.to_bits(m, W.DT_BF16), W.DT_BF16) for m in (gate, up, down)))
    xt = prox.from_bits(W.to_bits(x, W.DT_BF16), W.DT_BF16)
    if sparse:
        y, _ = prox.ffn_sparse(w, prox.pack_proxy(w, prox.INT4, 128), xt, D, F)
    else:
        y = prox.ffn_dense(w, xt)
    torch.cuda.synchronize()
    return W.bits_to_f32(prox.to_bits(y), W.DT_BF16).reshape(x.shape)


@pytest.mark.parametrize("sparse", [False, True])
@pytest.mark.parametrize("scale,w_down", [(8.0, 1.0), (1.0, 2.0 ** -30)])
def test_large_s(scale, w_down, sparse):
    print(f"[down range] scale {scale} sparse {sparse}", flush=True)
    rng = np.random.default_rng(5)
    gate, up = (np.zeros((F, D), np.float32) for _ in range(2))
    gate[:, ::3] = rng.standard_normal((F, len(range(0, D, 3)))) * 0.02
    up[:, ::3] = gate[::-1, ::3]
    for m in (gate, up):
        m[:, [I0, I1]] = 0.0
    # s = 73 scale 2^60 x 7 2^59 = 511 scale 2^119: at scale 1 a tie between the largest
    # bf16 and infinity, finite in fp32.
    gate[CH, [I0, I1]] = 73.0 * scale, -73.0 * scale
    up[CH, [I0, I1]] = 3.5
    down = (rng.integers(0, 2, (F, D)) * 2 - 1).astype(np.float32) * np.float32(w_down)
    x = rng.laplace(size=(B, D)).astype(np.float32)
    x[:, [I0, I1]] = 0.0
    x[:2] = 0.0
    x[0, I0], x[1, I1] = 2.0 ** 60, -(2.0 ** 60)   # s > 0 and s < 0
    y = _call(gate, up, down, x, sparse)
    s = np.float64(511.0) * scale * 2.0 ** 119
    with np.errstate(over="ignore"):
        s = np.float64(np.float32(s))
        want = np.array([s * down[CH], -s * down[CH]])
    assert np.array_equal(y[:2], want.astype(np.float32) if np.isinf(s) else _rounded(want))
    # The other rows are what the 8-row kernel gives them, but for the order of fp32 sums.
    ref = np.concatenate([_call(gate, up, down, x[b:b + 7], False) for b in (2, 9)])
    assert np.isfinite(ref).all() and np.abs(y[2:] - ref).max() <= 2.0 ** -7 * np.abs(ref).max()


def test_tiny_s():
    # s of about 1e-37: its lower parts are subnormal.  One rounding to bf16 apart.
    print("[down range] tiny", flush=True)
    rng = np.random.default_rng(6)
    gate, up, down = ((rng.standard_normal((F, D)) * 0.02).astype(np.float32) for _ in range(3))
    down *= 50.0
    x = (rng.laplace(size=(B, D)) * 4e-19).astype(np.float32)
    y = _call(gate, up, down, x, False)
    ref = np.concatenate([_call(gate, up, down, x[b:b + 8], False) for b in (0, 8)])
    assert np.abs(ref).max() > 1e-37
    assert np.abs(y - ref).max() <= 2.0 ** -8 * np.abs(ref).max()
