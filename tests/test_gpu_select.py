"""Channel selection on scores that its bracket finds, misses or finds tied: the
mask must be the exact top-k of the call's own scores, ties to the lower index,
whatever order the channels stand in.  d_ff at the edges of the per-thread score
counts and of the two tile widths."""
import numpy as np
import pytest
import torch

import oracle
from paper_2607_27591_amd import prox
from paper_2607_27591_amd import workloads as W

pytestmark = pytest.mark.gpu

D = 128


def channel_weights(kind, f, rng):
    w = (rng.standard_normal((2, f, D)) * 0.05).astype(np.float32)
    if kind == "ramp":        # tiles differ, so their order statistics do
        w *= np.linspace(0.05, 4.0, f, dtype=np.float32)[None, :, None]
    elif kind == "pairs":     # every score twice, half the range apart
        w[:, f // 2:2 * (f // 2)] = w[:, :f // 2]
    elif kind == "few":       # 40 distinct scores
        w = w[:, np.arange(f) % 40]
    elif kind == "zeros":     # three quarters of the scores are 0
        w[:, np.arange(f) % 4 != 1] = 0
    return w


@pytest.mark.parametrize("kind", ["plain", "ramp", "pairs", "few", "zeros"])
@pytest.mark.parametrize("f,batch", [(4096, 1), (4097, 1), (8193, 4), (12289, 1), (16385, 9), (24448, 1),
                                     (24449, 2), (28673, 1), (32769, 1), (65536, 1)])
def test_mask_is_the_top_k_of_the_scores(f, batch, kind):
    rng = np.random.default_rng(f + batch)
    g, u = (prox.from_bits(W.to_bits(m, W.DT_BF16), W.DT_BF16) for m in channel_weights(kind, f, rng))
    w = prox.Weights(g, u, u)
    p = prox.pack_proxy(w, prox.INT4, 128)
    x = prox.from_bits(W.to_bits(rng.laplace(size=(batch, D)).astype(np.float32), W.DT_BF16), W.DT_BF16)
    scores = torch.empty(f, dtype=torch.float32, device="cuda")
    for k in sorted({1, 2, f // 50, f // 16, f // 16 + 1, int(0.3 * f), f // 2, 7 * f // 8, 7 * f // 8 + 1,
                     int(0.96 * f), f - 1, f}):
        print(f"[select] {kind} f={f} B={batch} k={k}", flush=True)
        _, mask = prox.ffn_sparse(w, p, x, D // 2, k, scores=scores)
        torch.cuda.synchronize()
        kept = np.flatnonzero(mask.cpu().numpy())
        assert np.array_equal(kept, oracle.topk(scores.cpu().numpy().astype(np.float64), k))
