"""The workspace of a linear regression is that of the form its sizes take: (T + 1) d floats of
checkpoints where one workgroup walks the batches, their float64 matrices else."""
import pytest

import workloads as W
from helpers import desc_of

M = pytest.importorskip("paper_2505_00793_amd._lib")


def workspace(d, rows, T):
    cfg = W.C1.with_(widths=(d, 1), rows=rows, val_rows=rows, T=T)
    return M.Problem(desc_of(cfg)).mfmg_query_sizes(T).workspace_bytes


@pytest.mark.parametrize("d,rows,T", [(64, 256, 4), (64, 256, 6), (4, 1, 1), (256, 64, 64),
                                      (225, 64, 9), (252, 70, 9), (184, 98, 1), (208, 85, 2), (224, 85, 2)])
def test_walked_batches_need_checkpoints_only(d, rows, T):
    assert workspace(d, rows, T) == 4 * (T + 1) * d


@pytest.mark.parametrize("d", [1, 63, 64, 130, 200, 256])
@pytest.mark.parametrize("T", [7, 64])
def test_matrices_fit_the_static_scratch(d, T):
    need = workspace(d, 1024, T)
    assert 8 * (T + 1) * (d + 1) ** 2 < need <= 8 * (T + 2) * (d + 17) * (d + 3) + 4096
    assert need <= M.NOALLOC_SCRATCH_BYTES
