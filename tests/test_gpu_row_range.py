"""Stage 1 of an INT4 proxy on batches whose rows differ in range: a row far larger
than the others, or one with an infinite or NaN input, leaves the other rows' scores
as they are alone.  The loud row's inputs have zero weights when it is finite, so
that its own score is 0 and the others' decide; a row that is not finite scores NaN,
which the maximum over the batch drops."""
import numpy as np
import pytest
import torch

import oracle
from paper_2607_27591_amd import prox
from paper_2607_27591_amd import workloads as W

from gpu_cases import SCORE_TOL

pytestmark = pytest.mark.gpu


def _dequantised(bits, dtype, group):
    codes, scales = oracle.quantize(bits, dtype, 4, group)
    s = np.repeat(scales.view(np.float16).astype(np.float64), group, axis=1)
    return codes.astype(np.float64) * s


@pytest.mark.parametrize("loud", ["finite", "inf", "nan"])
@pytest.mark.parametrize("d,f,batch,group,dtype", [
    (512, 96, 2, 128, W.DT_BF16), (1024, 130, 3, 128, W.DT_BF16), (4096, 64, 4, 256, W.DT_BF16),
    (8192, 70, 4, 128, W.DT_BF16), (256, 24500, 3, 128, W.DT_BF16), (2048, 96, 4, 128, W.DT_F16),
    # 16-row matrix-core kernel
    (4096, 64, 8, 128, W.DT_BF16),
    # batch kernels
    (1152, 200, 20, 128, W.DT_BF16), (4224, 130, 6, 128, W.DT_BF16), (8192, 64, 16, 8192, W.DT_BF16),
    (16384, 64, 3, 128, W.DT_BF16), (256, 24500, 40, 128, W.DT_BF16), (1152, 96, 33, 128, W.DT_F16)])
def test_rows_do_not_disturb_each_other(d, f, batch, group, dtype, loud):
    print(f"[row range] {loud} {d}x{f} B={batch} g{group} dtype {dtype}", flush=True)
    rng = np.random.default_rng(d + f + batch)
    at = np.arange(17, d, 97)   # the loud row's inputs
    w = [(rng.standard_normal((f, d)) * 0.02).astype(np.float32) for _ in range(2)]
    x = (rng.laplace(size=(batch, d)) * 2.0 ** -8).astype(np.float32)
    x[0] = 0.0
    if loud == "finite":
        for m in w:
            m[:, at] = 0.0
        x[0, at] = 2.0 ** 40 if dtype == W.DT_BF16 else 2.0 ** 15
    else:
        x[0, at] = 1.0
    bits = [W.to_bits(m, dtype) for m in w]
    x_bits = W.to_bits(x, dtype)
    if loud != "finite":   # as bit patterns: the workloads' conversion takes finite values
        value = {"inf": (0x7F80, 0x7C00), "nan": (0x7FC0, 0x7E00)}[loud]
        x_bits[0, at[len(at) // 2]] = value[0 if dtype == W.DT_BF16 else 1]
    gate, up = (prox.from_bits(b, dtype) for b in bits)
    pw = prox.Weights(gate, up, up)
    p = prox.pack_proxy(pw, prox.INT4, group)
    scores = torch.empty(f, dtype=torch.float32, device="cuda")
    in_mask = torch.empty(d, dtype=torch.uint8, device="cuda")
    k = max(at.size, int(0.6 * d))
    prox.ffn_sparse(pw, p, prox.from_bits(x_bits, dtype), k, max(1, f // 3), in_mask=in_mask, scores=scores)
    torch.cuda.synchronize()
    keep = np.flatnonzero(in_mask.cpu().numpy())
    assert keep.size == k and np.isin(at, keep).all()
    xk = W.bits_to_f32(x_bits, dtype).astype(np.float64)[1:, keep]
    g, u = (xk @ _dequantised(b, dtype, group)[:, keep].T for b in bits)
    ref = np.abs(g / (1.0 + np.exp(-g)) * u).max(axis=0)
    err = np.abs(scores.cpu().numpy().astype(np.float64) - ref).max()
    assert err <= SCORE_TOL * ref.max()
