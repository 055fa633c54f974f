"""The small-batch and batch Stage 1 where their lists can go wrong: every count of
64-input blocks per wave and of lane groups sharing them (d_model 128 to 16384, both
tile widths), row tiles of 16, 32 and 64, all inputs kept, one kept, clustered ones
(some waves keep all of their inputs, others none, and the early guess misses) and
tied magnitudes, against the oracle's selection and scores."""
import numpy as np
import pytest
import torch

import oracle
from paper_2607_27591_amd import prox
from paper_2607_27591_amd import workloads as W

from gpu_cases import SCORE_TOL

pytestmark = pytest.mark.gpu


def inputs(kind, batch, d, rng):
    x = rng.laplace(size=(batch, d)).astype(np.float32)
    if kind == "clustered":     # whole blocks large, the rest small
        x *= np.where((np.arange(d) // 64) % 5 == 0, 50.0, 0.01)
    elif kind == "first":       # large inputs only in the first rounds' blocks
        x *= np.where(np.arange(d) < max(128, d // 6), 50.0, 1.0)
    elif kind == "tied":        # few distinct magnitudes
        x = np.sign(x) * np.float32(2.0) ** np.clip(np.round(np.abs(x)), 0, 2)
    return x


@pytest.mark.parametrize("kind", ["plain", "clustered", "first", "tied"])
@pytest.mark.parametrize("d,f,batch,group,dtype", [
    (128, 70, 1, 128, W.DT_BF16), (1024, 130, 2, 256, W.DT_F16), (1152, 200, 1, 128, W.DT_BF16),
    (2176, 64, 4, 128, W.DT_BF16), (3200, 129, 3, 128, W.DT_F16), (4096, 64, 4, 128, W.DT_F16),
    (5120, 100, 1, 128, W.DT_BF16), (6272, 65, 4, 896, W.DT_BF16), (7296, 64, 2, 128, W.DT_F16),
    (8192, 130, 4, 128, W.DT_BF16), (16384, 64, 1, 128, W.DT_BF16), (16384, 70, 2, 128, W.DT_F16),
    (256, 24500, 1, 128, W.DT_BF16), (1408, 24449, 4, 128, W.DT_F16),
    # batch kernels
    (128, 70, 17, 128, W.DT_BF16), (1152, 200, 32, 128, W.DT_F16), (4096, 65, 33, 256, W.DT_BF16),
    (4224, 130, 5, 128, W.DT_F16), (8192, 64, 16, 8192, W.DT_BF16), (16384, 64, 3, 128, W.DT_F16),
    (256, 24500, 20, 128, W.DT_F16), (384, 24449, 64, 128, W.DT_BF16)])
def test_scores_and_input_mask(d, f, batch, group, dtype, kind):
    rng = np.random.default_rng(d + f + batch)
    bits = [W.to_bits((rng.standard_normal((f, d)) * 0.02).astype(np.float32), dtype) for _ in range(2)]
    gate, up = (prox.from_bits(b, dtype) for b in bits)
    w = prox.Weights(gate, up, up)
    p = prox.pack_proxy(w, prox.INT4, group)
    (cg, sg), (cu, su) = (oracle.quantize(b, dtype, 4, group) for b in bits)
    x_bits = W.to_bits(inputs(kind, batch, d, rng), dtype)
    x = prox.from_bits(x_bits, dtype)
    scores = torch.empty(f, dtype=torch.float32, device="cuda")
    in_mask = torch.empty(d, dtype=torch.uint8, device="cuda")
    for k in sorted({1, 3, d // 10, int(0.45 * d), int(0.9 * d), d}):
        print(f"[small] {kind} {d}x{f} B={batch} g{group} k_in={k}", flush=True)
        prox.ffn_sparse(w, p, x, k, max(1, f // 3), in_mask=in_mask, scores=scores)
        torch.cuda.synchronize()
        ref = oracle.ffn_sparse(x_bits, dtype, bits[0], bits[1], bits[1], k, max(1, f // 3), codes_g=cg,
                                scales_g=sg, codes_u=cu, scales_u=su, group=group)
        assert np.array_equal(np.flatnonzero(in_mask.cpu().numpy()), ref["in_idx"])
        err = np.abs(scores.cpu().numpy().astype(np.float64) - ref["score"]).max()
        assert err <= SCORE_TOL * max(ref["score"].max(), 1e-30)
