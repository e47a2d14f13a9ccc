"""The columns algorithm: the forward product that stores the column matrix on its way (columns_split_kernel).

Bound of a product as in test_gpu_small.py, below 1e-6 of the result's norm; the column matrix is a copy, equal to the bit."""
import pytest
import torch

import paper_1803_11385_amd as hch
from tests.test_gpu_small import _data, _levels, _reference

pytestmark = pytest.mark.gpu


def _forward(lv, X, W, spare=None):
    (n, ci), co = X.shape, W.shape[2]
    want = hch.hch_conv_workspace_bytes(lv, 0, ci, co, hch.HCH_F32, hch.HCH_WS_FWD, hch.HCH_ALGO_COLUMNS)
    if spare is not None:
        want = hch.hch_conv_workspace_bytes(lv, 0, ci, co, hch.HCH_F32, hch.HCH_WS_MIN, hch.HCH_ALGO_COLUMNS) + spare
    ws = torch.full((want + 512,), 255, dtype=torch.uint8, device="cuda")
    ws = ws[(-ws.data_ptr()) % 256:]
    tail = ws[want:].clone()
    Y = torch.full((n, co), float("nan"), device="cuda")
    hch.hch_profile_reset()
    hch.hch_profile_enable(-1, True)
    hch.hch_conv_fwd(lv, 0, hch.HCH_F32, X, W, Y, ci, co, ws[:want], hch.HCH_ALGO_COLUMNS)
    hch.hch_profile_enable(-1, False)
    names = {hch.hch_kernel_name(i) for i in range(hch.hch_kernel_count()) if hch.hch_profile_read(i)["launches"]}
    assert torch.equal(ws[want:], tail)
    col = ws[:n * 27 * ci * 4].view(torch.float32) if want >= n * 27 * ci * 4 else None
    return Y, col, names


def _columns(lv, X):
    col = torch.empty(X.shape[0] * 27 * X.shape[1], device="cuda")
    hch.hch_hash2col(lv, 0, hch.HCH_F32, X, X.shape[1], 0, X.shape[0], col)
    return col


@pytest.mark.parametrize("n", [1, 15, 16, 17, 63, 64, 65, 127, 128, 129, 1000, 24513, 40000])
@pytest.mark.parametrize("ci,co", [(4, 16), (4, 4), (8, 33), (12, 20), (16, 32), (20, 70), (32, 64), (36, 17), (64, 130), (96, 32)])
def test_forward_and_its_column_matrix(n, ci, co):
    lv = _levels(n, 64, models=1 if n < 60 else 2)
    X, W, G = _data(n, ci, co)
    Y, col, names = _forward(lv, X, W)
    assert [k for k in names if k.startswith("columns_split_kernel")] and not [k for k in names if k.startswith(("hash2col", "gemm"))], names
    assert torch.equal(col, _columns(lv, X))
    want = _reference(lv, X, W, G)[0]
    assert float((Y.double() - want).norm() / want.norm()) < 1e-6


def test_column_matrix_beyond_the_caches():
    """More than 256 MB with rows of whole 64-byte pieces: stored past the caches."""
    lv = _levels(170000, 128, models=2)
    X, W, G = _data(170000, 16, 32)
    Y, col, _ = _forward(lv, X, W)
    assert torch.equal(col, _columns(lv, X))
    want = _reference(lv, X, W, G)[0]
    assert float((Y.double() - want).norm() / want.norm()) < 1e-6


@pytest.mark.parametrize("ci,co", [(4, 16), (16, 32)])
def test_smaller_workspaces_go_in_chunks(ci, co):
    """Room for a part of the column matrix: one chunk after the other, as ever."""
    lv = _levels(3000, 64)
    X, W, G = _data(3000, ci, co)
    Y, _, names = _forward(lv, X, W, spare=0)
    assert not [k for k in names if k.startswith("columns_split")] and [k for k in names if k.startswith("hash2col")], names
    want = _reference(lv, X, W, G)[0]
    assert float((Y.double() - want).norm() / want.norm()) < 1e-6


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
@pytest.mark.parametrize("ci,co", [(4, 16), (12, 20), (32, 64)])
def test_numbers_that_are_not_finite(value, ci, co):
    """A row's reach its neighbours and no others, as they come into the column matrix; a weight's its column, in every row (the
    rows without the tap have zero times it)."""
    n, v = 300, 150
    lv = _levels(n, 32)
    X, W, _ = _data(n, ci, co)
    clean = _forward(lv, X, W)[0]
    B = X.clone()
    B[v, ci - 1] = value
    Y, col, _ = _forward(lv, B, W)
    row = lv.info(0).device_nbr27()[v]
    near = torch.zeros(n, dtype=torch.bool, device="cuda")
    near[torch.from_numpy(row[row >= 0].astype("int64")).cuda()] = True
    assert torch.equal(col.view(torch.int32), _columns(lv, B).view(torch.int32))
    assert not torch.isfinite(Y[near]).any()
    assert float((Y[~near] - clean[~near]).norm() / clean.norm()) < 1e-6
    U = W.clone()
    U[5, 1, 3] = value
    Y = _forward(lv, X, U)[0]
    assert not torch.isfinite(Y[:, 3]).any()
    others = [k for k in range(co) if k != 3]
    assert float((Y[:, others] - clean[:, others]).norm() / clean.norm()) < 1e-6
