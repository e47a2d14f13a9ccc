"""Few voxels: the gathered products whose wavefronts share out the reduction (conv_small_kernel), at the edges of their tiles of 16
rows and 32 columns and on both sides of the line to conv_split_kernel, and the row order made by one workgroup per level
(pattern_small_kernel), up to its 6144 voxels and beyond.

Bound of a product: the pieces leave out at most 2^-24 of a term; a sum of K terms is rounded about K / 8 times and once per
wavefront, 0.29 * 2^-23 * sqrt(27 * 130 / 16) = 5e-7 of the result's norm: below 1e-6."""
import numpy as np
import pytest
import torch

import paper_1803_11385_amd as hch

pytestmark = pytest.mark.gpu


def _levels(n, u, levels=1, models=1, seed=0):
    rng = np.random.default_rng([n, seed])
    side = int(np.ceil((n / models) ** (1 / 3))) + 2                        # dense enough for many neighbours
    cut = np.linspace(0, n, models + 1).astype(np.int64)
    parts = []
    for a, b in zip(cut[:-1], cut[1:]):
        q = np.sort(rng.permutation(side ** 3)[:b - a])
        parts.append(np.stack([q // side ** 2, q // side % side, q % side], 1))
    return hch.hch_build_levels_device(np.ascontiguousarray(np.concatenate(parts), np.int32), cut, u, levels)


def _products(lv, X, W, G):
    n, ci, co = X.shape[0], X.shape[1], G.shape[1]
    ws = torch.full((max(hch.hch_conv_workspace_bytes(lv, 0, ci, co, hch.HCH_F32, k, hch.HCH_ALGO_FUSED)
                         for k in (hch.HCH_WS_FWD, hch.HCH_WS_BWD_DATA)) + 256,), 255, dtype=torch.uint8, device="cuda")
    ws = ws[(-ws.data_ptr()) % 256:]
    Y, dX = torch.full((n, co), float("nan"), device="cuda"), torch.full((n, ci), float("nan"), device="cuda")
    hch.hch_profile_reset()
    hch.hch_profile_enable(-1, True)
    hch.hch_conv_fwd(lv, 0, hch.HCH_F32, X, W, Y, ci, co, ws, hch.HCH_ALGO_FUSED)
    hch.hch_conv_bwd_data(lv, 0, hch.HCH_F32, G, W, dX, ci, co, ws, hch.HCH_ALGO_FUSED)
    hch.hch_profile_enable(-1, False)
    names = {hch.hch_kernel_name(i) for i in range(hch.hch_kernel_count()) if hch.hch_profile_read(i)["launches"]}
    return Y, dX, names


def _reference(lv, X, W, G):
    nb = torch.from_numpy(lv.info(0).device_nbr27().astype(np.int64)).cuda()
    X, W, G = X.double(), W.double(), G.double()

    def rows(T, k):
        return torch.where(nb[:, k:k + 1] >= 0, T[nb[:, k].clamp(min=0)], torch.zeros((), dtype=T.dtype, device="cuda"))
    return sum(rows(X, k) @ W[k] for k in range(27)), sum(rows(G, k) @ W[26 - k].T for k in range(27))


def _data(n, ci, co):
    g = torch.Generator(device="cuda")
    g.manual_seed(n + 100 * ci + co)
    return (torch.randn(s, device="cuda", generator=g) for s in ((n, ci), (27, ci, co), (n, co)))


@pytest.mark.parametrize("n", [1, 15, 16, 17, 33, 700])
@pytest.mark.parametrize("ci,co", [(3, 16), (5, 7), (8, 33), (16, 32), (31, 65), (24, 17), (64, 64), (50, 50), (130, 20)])
def test_products(n, ci, co):
    lv = _levels(n, 32)
    X, W, G = _data(n, ci, co)
    Y, dX, names = _products(lv, X, W, G)
    assert any(k.startswith("conv_small_kernel") for k in names), names
    for got, want in zip((Y, dX), _reference(lv, X, W, G)):
        assert float((got.double() - want).norm() / want.norm()) < 1e-6


@pytest.mark.parametrize("n,ci,co", [(700, 1, 4), (700, 2, 8), (3177, 1, 16), (3177, 3, 16), (12000, 2, 7)])
def test_sums_of_few_terms_are_rounded_once(n, ci, co):
    """A rounding errs by 2^-23 / sqrt(12) at the lower end of a binade, 2.25e-8 of values spread evenly over it.  Two of them, one within a
    wavefront's instruction and the result's own, are 3.2e-8 of the norm, below 4e-8; with the wavefronts' sums rounded one by one, and after
    each addition, it was 5.0e-8 to 5.9e-8."""
    lv = _levels(n, 32)
    X, W, G = _data(n, ci, co)
    Y, dX, names = _products(lv, X, W, G)
    assert "conv_small_kernel<1, false>" in names, names
    want = _reference(lv, X, W, G)[0]
    assert float((Y.double() - want).norm() / want.norm()) < 4e-8


FWD, BWD = "conv_small_kernel<2, false>", "conv_small_kernel<2, true>"


@pytest.mark.parametrize("n,ci,co,small", [
    (12109, 16, 32, {FWD, "conv_small_kernel<1, true>"}), (12110, 16, 32, {"conv_small_kernel<1, true>"}), (12695, 16, 32, {"conv_small_kernel<1, true>"}),
    (12696, 16, 32, set()), (6103, 32, 64, {FWD}), (6104, 32, 64, set()), (300, 64, 128, {FWD}), (300, 64, 129, set()), (300, 112, 72, {FWD}), (300, 128, 64, set()),
    (300, 88, 32, {FWD, BWD}), (300, 96, 32, {BWD}), (300, 32, 88, {FWD, BWD}), (300, 32, 96, {FWD}), (300, 20, 40, {FWD, BWD}), (300, 40, 50, {FWD}),
    (12109, 12, 20, {FWD}), (12110, 12, 20, set()), (7812, 24, 20, {FWD}), (7813, 24, 20, set()), (24218, 6, 7, {"conv_small_kernel<1, false>"}),
    (24219, 6, 7, set()), (16406, 6, 7, {"conv_small_kernel<1, false>", "conv_small_kernel<1, true>"}), (16407, 6, 7, {"conv_small_kernel<1, false>"}), (40000, 6, 7, set())])
def test_line_to_conv_split_kernel(n, ci, co, small):
    lv = _levels(n, 64, models=2)
    X, W, G = _data(n, ci, co)
    Y, dX, names = _products(lv, X, W, G)
    assert {k for k in names if k.startswith("conv_small")} == small
    for got, want in zip((Y, dX), _reference(lv, X, W, G)):
        assert float((got.double() - want).norm() / want.norm()) < 1e-6


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_numbers_that_are_not_finite(value):
    """They reach the voxels that have them as a neighbour and no others, which keep their values."""
    n, ci, co, v = 300, 33, 40, 150
    lv = _levels(n, 32)
    X, W, G = _data(n, ci, co)
    clean = _products(lv, X, W, G)
    X[v, 7] = G[v, 39] = value
    got = _products(lv, X, W, G)
    row = lv.info(0).device_nbr27()[v]
    near = torch.zeros(n, dtype=torch.bool, device="cuda")
    near[torch.from_numpy(row[row >= 0].astype(np.int64)).cuda()] = True
    for a, b in zip(got[:2], clean[:2]):
        assert not torch.isfinite(a[near]).any()
        assert float((a[~near] - b[~near]).norm() / b.norm()) < 1e-6


@pytest.mark.parametrize("a,b", [(1e-34, 1.0), (1.0, 1e-36), (1e-40, 1e20), (1e20, 1e-40), (1e30, 1e-30), (1e15, 1e15)])
@pytest.mark.parametrize("ci,co", [(3, 16), (33, 40)])
def test_ends_of_the_range(ci, co, a, b):
    """As test_gpu_split.py, with sums that leave the scaled range (1e15) and are repeated with the fp32 instruction, a rounding per 4 terms."""
    lv = _levels(700, 32)
    X, W, G = _data(700, ci, co)
    X, W, G = X * a, W * b, G * a
    Y, dX, names = _products(lv, X, W, G)
    assert {k.split("<")[0] for k in names} == {"conv_small_kernel"}, names
    for got, want in zip((Y, dX), _reference(lv, X, W, G)):
        assert float((got.double() - want).norm() / want.norm()) < 1e-6


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_weights_that_are_not_finite(value):
    """They reach the rows that have their tap, in their column, and no others."""
    n, ci, co = 300, 33, 40
    lv = _levels(n, 32)
    X, W, G = _data(n, ci, co)
    clean = _products(lv, X, W, G)
    W[5, 3, 7] = value
    got = _products(lv, X, W, G)
    nb = torch.from_numpy(lv.info(0).device_nbr27().astype(np.int64)).cuda()
    for a, b, tap, column in ((got[0], clean[0], 5, 7), (got[1], clean[1], 21, 3)):
        hit = torch.zeros_like(a, dtype=torch.bool)
        hit[nb[:, tap] >= 0, column] = True
        assert bool(hit.any()) and not torch.isfinite(a[hit]).any()
        assert float((a[~hit] - b[~hit]).norm() / b.norm()) < 1e-6


@pytest.mark.parametrize("n", [1, 63, 64, 65, 1024, 1025, 6143, 6144, 6145, 8191, 8192, 8193])
def test_row_order(n):
    lv = _levels(n, 64, levels=3, models=1 if n < 60 else 3, seed=1)
    for l in range(3):
        info = lv.info(l)
        valid = info.device_nbr27() >= 0
        key = np.zeros(info.n_total, np.int64)
        for k in range(1, 13, 2):
            key = key * 2 + (valid[:, k] | valid[:, 26 - k])
        order = info.device_row_order()
        assert np.array_equal(order, np.argsort(key, kind="stable"))
        mask = np.zeros(-(-info.n_total // 64) * 64, np.int64)
        mask[:info.n_total] = (valid.astype(np.int64) @ (1 << np.arange(27, dtype=np.int64)))[order]
        assert np.array_equal(info.device_tile_taps().astype(np.int64), np.bitwise_or.reduce(mask.reshape(-1, 64), axis=1))
