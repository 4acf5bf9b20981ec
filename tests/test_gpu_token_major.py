"""Transformer weight gradients from operands stored by token: every tile size and split-K, token
counts and vocabularies of any residue modulo 8, in a workspace full of NaN, per parameter tensor
against the oracle's bf16 emulation."""
import numpy as np
import pytest

import oracle
import workloads as W
from helpers import desc_of, relerr, tol_of

pytestmark = pytest.mark.gpu

CASES = [  # d_model, heads, d_ff, vocab, seq, rows
    (64, 4, 128, 97, 20, 1),      # 64 x 32 tiles, k = 20
    (512, 8, 512, 1602, 8, 3),    # 64 x 64 tiles for the unembedding
    (512, 8, 512, 3077, 12, 5),   # 128 x 64
    (64, 4, 128, 301, 256, 5),    # split-K
    (512, 8, 128, 97, 64, 128),   # an odd k on register-staged 128 x 128 tiles (dU^T)
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_token_major_weight_gradients(case):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_00793_amd import _lib as M
    d, heads, ff, vocab, seq, rows = case
    cfg = W.SMALL["c4_small"].with_(name="token_major", cfg_id=150, d_model=d, n_heads=heads,
                                    d_ff=ff, vocab=vocab, seq=seq, rows=rows, val_rows=1,
                                    n_blocks=1)
    inp = W.make_inputs(cfg, T=1)
    n = W.n_theta(cfg)
    theta = inp["theta0"] + 0.02 * W.random_direction(n, 56)
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
    from test_gpu_transformer import token_alpha
    alpha = token_alpha(cfg, theta, inp["eta"], tok)
    g_ref, _ = oracle.grad_and_loss(cfg, theta, tok, None, alpha=alpha, bf16=True)
    hv_ref = oracle.hvp_rev_rev(cfg, theta, tok, None, v, alpha=alpha, bf16=True)
    g, hv = g.cpu().numpy(), hv.cpu().numpy()
    for name, off, shape in W.theta_layout(cfg):
        if len(shape) != 2 or name == "emb":
            continue
        k = slice(off, off + int(np.prod(shape)))
        errs = relerr(g[k], g_ref[k]), relerr(hv[k], hv_ref[k])
        assert max(errs) <= tol_of(cfg), (name, errs)
