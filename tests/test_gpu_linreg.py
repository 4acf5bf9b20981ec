"""Linear regression at the edges of its three forms (registers, staged batches, normal equations)
and near a fit, against the float64 oracle."""
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
    # staged for few steps: both sides of the widths, rows and steps where the rule changes
    (16, 1024, 700, 1), (64, 257, 30, 1), (63, 256, 200, 1), (100, 182, 182, 1), (180, 116, 40, 1),
    (184, 98, 98, 1), (184, 99, 98, 1), (184, 98, 98, 2), (204, 98, 10, 1), (208, 85, 85, 2),
    (224, 85, 85, 2), (224, 85, 86, 2), (224, 48, 30, 3), (190, 98, 5, 1), (225, 85, 85, 1), (252, 75, 60, 3),
    (248, 75, 60, 3),
]


def off16(t):
    """A copy of t that starts 4 bytes past a 16-byte boundary."""
    import torch
    buf = torch.empty(t.numel() + 1, device=t.device)
    buf[1:] = t.reshape(-1)
    return buf[1:].reshape(t.shape)


@pytest.mark.parametrize("d,rows,val_rows,T,aligned", [(*c, True) for c in CASES] + [
    (64, 256, 256, 6, False), (36, 100, 50, 2, False), (208, 85, 85, 1, False),
    (256, 64, 64, 2, False), (130, 90, 90, 2, False)])
def test_linreg_forms(d, rows, val_rows, T, aligned):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_00793_amd import _lib as M
    cfg = W.C1.with_(name="lr", cfg_id=141, widths=(d, 1), rows=rows, val_rows=val_rows, T=T)
    inp = W.make_inputs(cfg)
    dev = to_device(inp)
    if not aligned:
        dev["xs"], dev["vx"] = [off16(x) for x in dev["xs"]], off16(dev["vx"])
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


@pytest.mark.parametrize("mean", [0.0, 3.0, 10.0])
@pytest.mark.parametrize("d,rows,T", [(64, 700, 8), (97, 300, 2), (130, 1000, 3), (256, 1024, 4)])
def test_normal_equations_at_a_fit(d, rows, T, mean):
    """Where the gradient is small against G theta and X^T y, which it is the difference of."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_00793_amd import _lib as M
    cfg = W.C1.with_(name="fit", cfg_id=142, widths=(d, 1), rows=rows, val_rows=rows - 50, T=T)
    inp = W.make_inputs(cfg)
    w = W.random_direction(d, 58).astype(np.float32)
    w *= np.float32(np.sqrt(d)) / np.linalg.norm(w)
    rng = np.random.default_rng(59)

    def shifted(x):
        x = (x + np.float32(mean)).astype(np.float32)
        y = x.astype(np.float64) @ w + 0.1 * rng.standard_normal(len(x))
        return x, y.astype(np.float32).reshape(-1, 1)

    inp["train_x"], inp["train_y"] = map(list, zip(*[shifted(x) for x in inp["train_x"]]))
    inp["val_x"], inp["val_y"] = shifted(inp["val_x"])
    inp["theta0"] = w
    inp["eta"] = np.full(d, np.log(0.01 / (1 + mean * mean * d / 4)), dtype=np.float32)
    dev = to_device(inp)
    P = M.Problem(desc_of(cfg))
    out = torch.empty(d, device="cuda")
    loss = torch.empty(1, device="cuda")
    P.mfmg_meta_grad(dev["theta0"], None, dev["eta"], dev["xs"], dev["ys"], dev["vx"], dev["vy"],
                     out, loss)
    ref, V = oracle.meta_grad(cfg, inp)
    # float64 but for exp(eta) and the result, two units of 6e-8 each, through T <= 8 steps that
    # contract; float32 matrices show 4e-6 .. 8e-2 here, float32 residuals 4e-6 .. 7e-2
    assert relerr(out.cpu().numpy(), ref) <= 1e-6
    assert abs(loss.item() - float(V)) <= 1e-6 * abs(float(V))
