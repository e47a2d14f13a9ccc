"""The columns algorithm: the forward product that stores the column matrix on its way (columns_split_kernel), the gradient of the
column matrix on split operands (dcol_split_kernel).

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


@pytest.mark.parametrize("n", [65, 300, 25000])
@pytest.mark.parametrize("ci,co", [(12, 40), (44, 70), (76, 33), (4, 64), (20, 16)])
def test_weights_end_where_they_end(n, ci, co):
    """Terms past the last one, up to three steps of 32, have weights of zero, whatever lies behind the weights in memory; the rows' side
    of these terms is other rows' numbers.  27 * 12, 44, 76 = 4 modulo 32: half of the eight terms of a thread are past the end."""
    lv = _levels(n, 64)
    X, W, G = _data(n, ci, co)
    inside = torch.full((W.numel() + 256 * co,), 1e6, device="cuda")
    inside[:W.numel()] = W.reshape(-1)
    Y, _, names = _forward(lv, X, inside[:W.numel()].view(W.shape))
    assert [k for k in names if k.startswith("columns_split_kernel")], names
    want = _reference(lv, X, W, G)[0]
    assert float((Y.double() - want).norm() / want.norm()) < 1e-6
    assert torch.equal(Y, _forward(lv, X, W)[0])


@pytest.mark.parametrize("n,ci,co,stream", [(170000, 16, 32, True), (155345, 16, 16, True), (155344, 16, 16, False), (90000, 32, 64, True), (87381, 32, 16, False),
                                            (60000, 48, 20, True), (110000, 24, 16, False), (40000, 96, 130, True)])
def test_column_matrix_beyond_the_caches(n, ci, co, stream):
    """More than 256 MB (288 with more than 16 channels) with rows of whole 64-byte pieces: stored past the caches."""
    lv = _levels(n, 128, models=2)
    X, W, G = _data(n, ci, co)
    Y, col, names = _forward(lv, X, W)
    assert [k.endswith("true>") for k in names if k.startswith("columns_split_kernel")] == [stream], names
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


def _data_gradient(lv, G, W):
    (n, co), ci = G.shape, W.shape[1]
    ws = torch.full((hch.hch_conv_workspace_bytes(lv, 0, ci, co, hch.HCH_F32, hch.HCH_WS_BWD_DATA, hch.HCH_ALGO_COLUMNS) + 256,), 255, dtype=torch.uint8, device="cuda")
    dX = torch.full((n, ci), float("nan"), device="cuda")
    hch.hch_profile_reset()
    hch.hch_profile_enable(-1, True)
    hch.hch_conv_bwd_data(lv, 0, hch.HCH_F32, G, W, dX, ci, co, ws[(-ws.data_ptr()) % 256:], hch.HCH_ALGO_COLUMNS)
    hch.hch_profile_enable(-1, False)
    return dX, {hch.hch_kernel_name(i) for i in range(hch.hch_kernel_count()) if hch.hch_profile_read(i)["launches"]}


@pytest.mark.parametrize("n", [1, 15, 17, 127, 128, 129, 1000, 4096, 20001])
@pytest.mark.parametrize("ci,co", [(12, 32), (16, 32), (20, 64), (32, 64), (9, 64), (16, 48), (8, 64), (12, 128), (64, 128)])
def test_data_gradient(n, ci, co):
    """Rows of 32, 64 and 128 channels, shares of the columns that end within a workgroup's; c_in of 9 and 8, 48 channels and few rows of 128: as before."""
    lv = _levels(n, 64, models=1 if n < 60 else 2)
    X, W, G = _data(n, ci, co)
    dX, names = _data_gradient(lv, G, W)
    split = ci % 4 == 0 and ci > 8 and (co in (32, 64) or co == 128 and n >= 4096)
    assert ({k for k in names if k.startswith("dcol")} == {f"dcol_split_kernel<{co // 32}>"}) if split else not [k for k in names if k.startswith("dcol")], names
    want = _reference(lv, X, W, G)[1]
    assert float((dX.double() - want).norm() / want.norm()) < (1e-6 if split else 2e-6)      # the fp32 instruction: a rounding per 4 terms


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
@pytest.mark.parametrize("n,ci,co", [(300, 12, 32), (300, 32, 64), (4100, 16, 128)])
def test_gradients_that_are_not_finite(value, n, ci, co):
    """A row's reach its neighbours' and no others; a weight's the rows that have its tap, in its channel."""
    v = n // 2
    lv = _levels(n, 32)
    _, W, G = _data(n, ci, co)
    clean = _data_gradient(lv, G, W)[0]
    nb = torch.from_numpy(lv.info(0).device_nbr27().astype("int64")).cuda()
    H = G.clone()
    H[v, co - 1] = value
    got, near = _data_gradient(lv, H, W)[0], (nb == v).any(1)
    assert not torch.isfinite(got[near]).any()
    assert float((got[~near] - clean[~near]).norm() / clean.norm()) < 1e-6
    U = W.clone()
    U[5, ci - 1, 3] = value
    got, has = _data_gradient(lv, G, U)[0], nb[:, 21] >= 0
    assert not torch.isfinite(got[has, ci - 1]).any()
    assert float((got[:, :-1] - clean[:, :-1]).norm() / clean.norm()) < 1e-6 and float((got[~has] - clean[~has]).norm() / clean.norm()) < 1e-6
