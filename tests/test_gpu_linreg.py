"""Linear regression at the edges of its three forms (registers, staged batches, normal equations)
against the float64 oracle."""
import numpy as np
import pytest

import oracle
import workloads as W
from helpers import desc_of, relerr, to_device

pytestmark = pytest.mark.gpu

# (features, rows, validation rows, T)
CASES = [
    (64, 256, 256, 6), (64, 256, 256, 7), (60, 257, 30, 2), (1, 1, 1, 1), (31, 5, 900, 2),
    (63, 64, 64, 3), (65, 33, 40, 3), (96, 100, 7, 2), (97, 70, 257, 2), (128, 1024, 128, 2),
    (129, 90, 90, 64), (160, 61, 20, 2), (161, 130, 64, 2), (193, 65, 65, 2), (224, 64, 64, 2),
    (225, 64, 64, 2), (227, 65, 3, 2), (256, 64, 64, 16), (256, 300, 64, 34), (251, 7, 64, 3),
]


@pytest.mark.parametrize("d,rows,val_rows,T", CASES)
def test_linreg_forms(d, rows, val_rows, T):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_00793_amd import _lib as M
    cfg = W.C1.with_(name="lr", cfg_id=141, widths=(d, 1), rows=rows, val_rows=val_rows, T=T)
    inp = W.make_inputs(cfg)
    dev = to_device(inp)
    P = M.Problem(desc_of(cfg))
    ws = P.workspace(P.mfmg_query_sizes(T).workspace_bytes)
    ws.fill_(255)   # NaN
    out = torch.empty(d, device="cuda")
    loss = torch.empty(1, device="cuda")
    P.mfmg_meta_grad(dev["theta0"], None, dev["eta"], dev["xs"], dev["ys"], dev["vx"], dev["vy"],
                     out, loss, ws=ws)
    ref, V = oracle.meta_grad(cfg, inp)
    # sums of at most 1024 products and 2 T + 1 <= 69 steps in float32: 69 eps sqrt(1024) = 1.3e-4
    # in the worst order; 1e-5 leaves an order over what the forms show (5e-7 at T = 64)
    assert relerr(out.cpu().numpy(), ref) <= 1e-5
    assert abs(loss.item() - float(V)) <= 1e-5 * abs(float(V))
