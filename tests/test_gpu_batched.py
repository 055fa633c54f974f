"""Matrix-core Stage 2 at the edges of its row tiles (16, 32 and 64 rows), its
256-column workgroups (d_model 4224 leaves half of one) and its 320-channel
chunks, sparse and dense, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2607_27591_amd import prox
from paper_2607_27591_amd import workloads as W

from gpu_cases import Y_TOL, check_sparse, make_case, run_sparse, y_rel_err

pytestmark = pytest.mark.gpu

CASES = [(4096, 700, 16, W.DT_BF16), (4096, 700, 17, W.DT_BF16), (4224, 520, 32, W.DT_F16),
         (4224, 1111, 33, W.DT_BF16), (8192, 260, 63, W.DT_F16), (4096, 5200, 10, W.DT_BF16),
         (4096, 5200, 20, W.DT_F16), (6144, 40, 64, W.DT_BF16)]


@pytest.mark.parametrize("d,f,batch,dtype", CASES)
def test_batched_parity(d, f, batch, dtype):
    print(f"[batched] {d}x{f} B={batch} dtype {dtype}", flush=True)
    cfg = W.small_config(d=d, f=f, batch=batch, seed=d + f + batch, dtype=dtype, in_frac=0.4, sigma_w=0.015)
    case = make_case(cfg)
    x = case.wl.x_vectors(1, batch)[0]
    check_sparse(case, x, cfg.k_in, cfg.k_ff, run_sparse(case, x, cfg.k_in, cfg.k_ff), tag=cfg.name)
    y = prox.ffn_dense(case.w, prox.from_bits(x, dtype))
    torch.cuda.synchronize()
    ref = oracle.ffn_dense(x, dtype, case.wl.w_gate, case.wl.w_up, case.wl.w_down)
    assert y_rel_err(prox.to_bits(y), ref, dtype) <= Y_TOL
    # A row alone and in the batch: the same tile arithmetic, so the same bits.
    y2 = prox.ffn_dense(case.w, prox.from_bits(np.ascontiguousarray(x[::-1]), dtype))
    torch.cuda.synchronize()
    assert np.array_equal(prox.to_bits(y2)[::-1], prox.to_bits(y))


def test_one_workspace_serves_every_batch():
    # A server allocates for its largest batch; the 8-row kernel's partial y then takes
    # more than the matrix-core path's.  Each call as on a workspace of its own.
    cfg = W.small_config(d=4096, f=700, batch=64, seed=41, in_frac=0.4, sigma_w=0.015)
    case = make_case(cfg)
    ws = prox.new_workspace(cfg.d_model, cfg.d_ff, 64)
    for batch in (64, 8, 20, 5, 3, 16, 1):
        print(f"[batched] one workspace, B={batch}", flush=True)
        x = case.wl.x_vectors(1, batch)[0]
        got, own = (run_sparse(case, x, cfg.k_in, cfg.k_ff, ws=w) for w in (ws, None))
        assert np.array_equal(got.y, own.y) and np.array_equal(got.mask, own.mask)
        xt = prox.from_bits(np.atleast_2d(x), cfg.dtype)
        got, own = (prox.to_bits(prox.ffn_dense(case.w, xt, ws=w)) for w in (ws, None))
        assert np.array_equal(got, own)
