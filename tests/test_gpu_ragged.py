"""Products whose contractions are padded to whole 16-byte chunks: widths and rows of every residue
modulo 8 (bf16) and 4 (float32), on every tile size of the direct-to-LDS kernel, in a workspace full
of NaN, against the oracle."""
import numpy as np
import pytest

import oracle
import workloads as W
from helpers import desc_of, group_errors, to_device, tol_of

pytestmark = pytest.mark.gpu

# a first layer of 8 slices, whose rows and outputs both end in padding
SPLIT = ((608, 33, 130, 18), 67, 43, W.C2)

CASES = [  # widths, rows, val_rows, optimiser family
    ((65, 130, 67, 3), 60, 43, W.C5), ((61, 35, 44, 5), 121, 129, W.C5),
    ((9, 1, 7, 2), 3, 1, W.C5), ((70, 131, 6), 37, 64, W.C3), ((64, 128, 136), 65, 8, W.C5),
    ((66, 257), 127, 130, W.C5),
    # float32: 64 x 16 and 64 x 32 tiles, split-K (608), 64 x 64, 128 x 64 and 128 x 128 tiles
    ((61, 35, 44, 5), 121, 129, W.C2), ((530, 33, 130, 18), 67, 258, W.C2), SPLIT,
    ((9, 1, 7, 2), 3, 1, W.C2.with_(optimizer=W.OPT_ADAM, meta=W.META_LOGLR_PER_LAYER_WD)),
    ((1030, 1537), 197, 130, W.C2), ((1541, 2050), 133, 70, W.C2),
]


def _id(case):
    return "-".join(map(str, case[0])) + ("-f32" if case[3].precision == W.PREC_FP32 else "")


@pytest.mark.parametrize("case", CASES, ids=_id)
def test_padded_contractions(case):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_00793_amd import _lib as M
    widths, rows, val_rows, base = case
    cfg = base.with_(name="ragged", cfg_id=140, widths=widths, rows=rows, val_rows=val_rows, T=2)
    inp = W.make_inputs(cfg)
    dev = to_device(inp)
    P = M.Problem(desc_of(cfg))
    ws = P.workspace(P.mfmg_query_sizes(cfg.T).workspace_bytes)
    ws.fill_(255)   # every float32 and bfloat16 in it is NaN
    d = torch.empty(W.n_eta(cfg), device="cuda")
    P.mfmg_meta_grad(dev["theta0"], dev["opt_state0"], dev["eta"], dev["xs"], dev["ys"], dev["vx"],
                     dev["vy"], d, ws=ws)
    ref, _ = oracle.meta_grad(cfg, inp, bf16=cfg.precision == W.PREC_BF16)
    errs = group_errors(cfg, d.cpu().numpy().astype(np.float64), ref)
    assert max(errs) <= tol_of(cfg), errs


def test_split_case_splits():
    """Its plan holds the slices' sums: one feature more has none, and yet longer rows."""
    from paper_2505_00793_amd import _lib as M
    widths, rows, val_rows, base = SPLIT

    def dynamic(n_in):
        cfg = base.with_(widths=(n_in, *widths[1:]), rows=rows, val_rows=val_rows)
        return M.Problem(desc_of(cfg)).mfmg_query_sizes(2).dynamic_bytes

    assert dynamic(608) > dynamic(609)


@pytest.mark.parametrize("last", [64, 10])
def test_ragged_layer_sums_in_one_order(last):
    """A ragged first layer (k = 530) adds its products in one run whether or not another layer
    (512 -> 64 over 64 rows) plans split-K scratch: 2^27, ones and -2^27 leave the ones out."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_00793_amd import _lib as M
    cfg = W.C2.with_(name="order", cfg_id=143, widths=(530, 33, 512, last), act=W.ACT_RELU, rows=64,
                     val_rows=64, T=1)
    inp = W.make_inputs(cfg)
    theta = inp["theta0"].copy()
    layout = {name: slice(off, off + int(np.prod(shape))) for name, off, shape in W.theta_layout(cfg)}
    names = list(layout)
    theta[layout[names[0]]] = 1.0                    # W_0
    theta[layout[names[3]]] = 0.1                    # b_1 keeps the second layer's units on
    x = np.ones((64, 530), dtype=np.float32)
    x[:, 0], x[:, -1] = 2.0 ** 27, -2.0 ** 27
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    n = W.n_theta(cfg)
    th1, g = torch.empty(n, device="cuda"), torch.empty(n, device="cuda")
    P = M.Problem(desc_of(cfg))
    P.mfmg_inner_step(up(theta), None, up(inp["eta"]), up(x), up(inp["train_y"][0]), 0, th1, None, g,
                      torch.empty(1, device="cuda"))
    g = g.cpu().numpy()
    assert np.abs(g[layout[names[5]]]).max() > 0     # the gradient reaches the layers behind it
    assert np.abs(g[layout[names[2]]]).max() == 0    # dW_1 = a_0^T dZ_1 with a_0 = 0
