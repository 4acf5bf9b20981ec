"""The rounding of Adam's update where a tile is not wholly inside an output with 16-byte rows:
which of the two products of m = b1 m0 + (1 - b1) g (and of v) is fused into the sum.  A bf16
network amplifies that last bit over its steps, so it may not change with the walk a tile takes."""
import numpy as np
import pytest

import workloads as W
from helpers import desc_of

pytestmark = pytest.mark.gpu


def fma(a, b, c):
    """Rounded once (the product of two float32 is exact in 64 bits of mantissa, their sum with c
    nearly always)."""
    return (np.longdouble(a) * np.longdouble(b) + np.longdouble(c)).astype(np.float32)


# rows of 60 pad the contraction; 10 outputs have no 16-byte rows, so every tile is an edge
@pytest.mark.parametrize("rows,nout,grad_at_edges", [(64, 64, True), (60, 64, False),
                                                     (64, 10, True), (60, 10, False)])
def test_adam_edge_tiles(rows, nout, grad_at_edges):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_00793_amd import _lib as M
    cfg = W.C3.with_(name="edge", cfg_id=160, widths=(100, nout), rows=rows, val_rows=64, T=1)
    inp = W.make_inputs(cfg)
    n = W.n_theta(cfg)
    m0 = (0.01 * W.random_direction(n, 12)).astype(np.float32)
    v0 = ((0.01 * W.random_direction(n, 13)) ** 2).astype(np.float32)
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    th1, g, opt1 = (torch.empty(k, device="cuda") for k in (n, n, 2 * n))
    P = M.Problem(desc_of(cfg))
    P.mfmg_inner_step(up(inp["theta0"]), up(np.concatenate([m0, v0])), up(inp["eta"]),
                      up(inp["train_x"][0]), up(inp["train_y"][0]), 0, th1, opt1, g,
                      torch.empty(1, device="cuda"))
    g, opt1 = g.cpu().numpy(), opt1.cpu().numpy()
    b1, b2 = np.float32(cfg.adam_b1), np.float32(cfg.adam_b2)
    c1, c2 = np.float32(1) - b1, np.float32(1) - b2
    # the gradient's product rounded and the state's fused into the sum, or the other way round
    state = fma(b1, m0, c1 * g), fma(b2, v0, (c2 * g) * g)
    grad = fma(c1, g, b1 * m0), fma(c2 * g, g, b2 * v0)
    k = 100 * nout
    inner = np.arange(k) < (64 * nout if nout == 64 else 0)   # rows 0..63 of W: whole tiles
    for got, s, gr in zip((opt1[:n], opt1[n:]), state, grad):
        assert np.mean(s[:k] != gr[:k]) > 0.05   # the two orders are told apart
        want = np.where(inner, s[:k], gr[:k] if grad_at_edges else s[:k])
        assert np.mean(got[:k] == want) > 0.999
