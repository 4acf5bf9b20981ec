"""A decoder whose vocabulary is past what the token-major weight gradients address (2^20): its
plan keeps transposed copies of their operands.  Gradient and H v per parameter tensor against the
oracle's bf16 emulation, in a workspace full of NaN."""
import numpy as np
import pytest

import oracle
import workloads as W
from helpers import desc_of, relerr, tol_of

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fused,seq", [(1, 64), (0, 8)])
def test_wide_vocabulary(fused, seq):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_00793_amd import _lib as M
    from test_gpu_transformer import token_alpha
    cfg = W.SMALL["c4_small"].with_(name="wide_vocab", cfg_id=170, d_model=64, n_heads=1, d_ff=64,
                                    vocab=(1 << 20) + 5, seq=seq, rows=1, val_rows=1, n_blocks=1,
                                    fused_attention=fused)
    inp = W.make_inputs(cfg, T=1)
    n = W.n_theta(cfg)
    theta = inp["theta0"]
    v = 0.1 * W.random_direction(n, 57)
    tok = inp["train_x"][0]
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    P = M.Problem(desc_of(cfg))
    ws = P.workspace(P.mfmg_query_sizes(1).step_workspace_bytes)
    ws.fill_(255)   # every float32 and bfloat16 in it is NaN
    g, hv = torch.empty(n, device="cuda"), torch.empty(n, device="cuda")
    P.mfmg_hvp_fwd_over_rev(up(theta), up(inp["eta"]), up(tok),
                            torch.zeros(1, dtype=torch.int32, device="cuda"), 0, up(v), g, hv,
                            None, ws=ws)
    g, hv = g.cpu().numpy(), hv.cpu().numpy()
    alpha = token_alpha(cfg, theta, inp["eta"], tok)
    g_ref, _ = oracle.grad_and_loss(cfg, theta, tok, None, alpha=alpha, bf16=True)
    hv_ref = oracle.hvp_rev_rev(cfg, theta, tok, None, v, alpha=alpha, bf16=True)
    for name, off, shape in W.theta_layout(cfg):
        if len(shape) != 2:
            continue
        k = slice(off, off + int(np.prod(shape)))
        errs = relerr(g[k], g_ref[k]), relerr(hv[k], hv_ref[k])
        assert max(errs) <= tol_of(cfg), (name, errs)
