"""The bf16 products over the row order in workgroups of 128 rows (conv_bf16_kernel<..., 4>, conv_ragged_bf16_kernel): around the edges of
their tiles of rows, columns and channels, and on both sides of the lines to the other kernels.

Bound: products are exact; a sum of K terms is rounded about K / 8 times (8 lanes' terms an instruction, in the order of K): 0.29 * 2^-23 *
sqrt(27 * 130 / 8) = 7.3e-7 of the result's norm, below 1e-6; a single result is looked at against 30 times that."""
import pytest
import torch

import paper_1803_11385_amd as hch
from tests.test_gpu_small import _levels

pytestmark = pytest.mark.gpu


def _odd_base(t):
    """The same tensor 4 bytes past a 16-byte boundary."""
    flat = torch.empty(t.numel() + 2, dtype=t.dtype, device="cuda")
    flat[2:] = t.reshape(-1)
    return flat[2:].view(t.shape)


def _data(n, ci, co, shift=False):
    g = torch.Generator(device="cuda")
    g.manual_seed(n + 100 * ci + co)
    out = [torch.randn(s, device="cuda", generator=g).bfloat16() for s in ((n, ci), (27, ci, co), (n, co))]
    return [_odd_base(t) for t in out] if shift else out


def _products(lv, X, W, G):
    (n, ci), co = X.shape, G.shape[1]
    out, names = [], []
    for name, kind, A, m in (("hch_conv_fwd", hch.HCH_WS_FWD, X, co), ("hch_conv_bwd_data", hch.HCH_WS_BWD_DATA, G, ci)):
        ws = torch.full((hch.hch_conv_workspace_bytes(lv, 0, ci, co, hch.HCH_BF16, kind, hch.HCH_ALGO_FUSED) + 256,), 255, dtype=torch.uint8, device="cuda")
        Y = torch.full((n, m), float("nan"), device="cuda")
        hch.hch_profile_reset()
        hch.hch_profile_enable(-1, True)
        getattr(hch, name)(lv, 0, hch.HCH_BF16, A, W, Y, ci, co, ws[(-ws.data_ptr()) % 256:], hch.HCH_ALGO_FUSED)
        hch.hch_profile_enable(-1, False)
        names.append([hch.hch_kernel_name(i) for i in range(hch.hch_kernel_count()) if hch.hch_profile_read(i)["launches"]])
        out.append(Y)
    return out, names


def _wants(lv, X, W, G):
    nb = lv.info(0).device_nbr27()
    nb = torch.from_numpy(nb.astype("int64")).cuda()

    def sums(A, w):
        zero = torch.zeros((), dtype=torch.float64, device="cuda")
        return sum(torch.where(nb[:, k:k + 1] >= 0, A.double()[nb[:, k].clamp(min=0)], zero) @ w[k].double() for k in range(27))
    return sums(X, W), sums(G, W.flip(0).transpose(1, 2))


def _check(got, want):
    assert float((got.double() - want).norm() / want.norm()) < 1e-6
    assert float((got.double() - want).abs().max() / want.pow(2).mean().sqrt()) < 3e-5


@pytest.mark.parametrize("n", [1, 31, 32, 33, 127, 128, 129, 300, 700])
@pytest.mark.parametrize("ci,co", [(4, 6), (6, 18), (18, 6), (34, 66), (50, 50), (62, 30), (126, 130)])
def test_ragged_rows(n, ci, co):
    """Even numbers of channels, tails of 2 to 30; the last row's last piece ends at the end of the operand."""
    lv = _levels(n, 32)
    X, W, G = _data(n, ci, co)
    out, names = _products(lv, X, W, G)
    for k, (got, want) in enumerate(zip(out, _wants(lv, X, W, G))):
        c, m = ((ci, co), (co, ci))[k]                    # few rows: 32 columns at a time, unless the reduction is short
        assert names[k] == [f"conv_ragged_bf16_kernel<{2 if m <= 32 or 27 * c >= 512 else 4}, {'true' if k else 'false'}>"], names
        _check(got, want)


@pytest.mark.parametrize("n,ci,co", [(700, 50, 50), (700, 16, 32), (700, 34, 66), (17000, 64, 64), (17000, 62, 30)])
def test_few_rows_are_summed_in_parts(n, ci, co):
    """A rounding errs by 2.25e-8 of what it rounds (test_gpu_small.py), a chain of m of them by sqrt(m / 2) times that.  Sums of 128 terms: 16
    roundings each, 6.4e-8; up to 16 such sums added up: 6.4e-8; together 9.0e-8, below 1e-7.  One chain of 27 * 32 to 27 * 66 terms: 1.6e-7 to 2.4e-7, of 9 * 62: 1.3e-7."""
    lv = _levels(n, 64) if n < 1000 else _sheet(n)
    X, W, G = _data(n, ci, co)
    out, names = _products(lv, X, W, G)
    for k, (got, want) in enumerate(zip(out, _wants(lv, X, W, G))):
        if any("conv" in name for name in names[k]):       # (16 -> 32 stays on gemm_bf16_kernel)
            assert float((got.double() - want).norm() / want.norm()) < 1e-7, names[k]
    assert any("conv" in name for name in names[0] + names[1]), names


@pytest.mark.parametrize("ci,co", [(98, 6), (34, 66), (66, 34), (50, 50)])
def test_nothing_comes_of_what_lies_behind_the_weights(ci, co):
    """2 channels modulo 32: a thread's four rows of the last tap's last step end past the last row of the weights."""
    lv = _levels(300, 32)
    X, W, G = _data(300, ci, co)
    inside = torch.full((W.numel() + 64 * max(ci, co),), float("nan"), dtype=torch.bfloat16, device="cuda")
    inside[:W.numel()] = W.reshape(-1)
    out, names = _products(lv, X, inside[:W.numel()].view(W.shape), G)
    assert all("ragged" in k[0] for k in names), names
    for got, want, clean in zip(out, _wants(lv, X, W, G), _products(lv, X, W, G)[0]):
        _check(got, want)
        assert torch.equal(got, clean)


@pytest.mark.parametrize("ci,co", [(64, 32), (40, 24), (12, 20)])
def test_operands_off_the_16_byte_boundary(ci, co):
    lv = _levels(333, 32)
    X, W, G = _data(333, ci, co, shift=True)
    out, names = _products(lv, X, W, G)
    assert all("ragged" in k[0] for k in names), names
    for got, want in zip(out, _wants(lv, X, W, G)):
        _check(got, want)


ROWS, RAGGED = "conv_bf16", "conv_ragged_bf16"


@pytest.mark.parametrize("n,ci,co,fwd,bwd", [
    (16383, 32, 64, None, None), (16384, 32, 64, ROWS, ROWS), (16385, 64, 64, ROWS, ROWS), (700, 32, 16, None, None), (700, 16, 32, None, ROWS),
    (81919, 32, 16, None, None), (81920, 32, 16, ROWS, None), (65535, 96, 32, None, ROWS), (65536, 96, 32, ROWS, ROWS), (98303, 24, 40, None, None),
    (98304, 24, 40, RAGGED, None), (160000, 40, 24, RAGGED, RAGGED), (159999, 40, 24, None, RAGGED), (98303, 64, 64, ROWS, ROWS), (98304, 64, 64, ROWS, ROWS),
    # stretches where gemm_bf16_kernel's tiles fill a round
    (20479, 32, 32, None, ROWS), (20480, 32, 32, ROWS, ROWS), (49152, 32, 32, ROWS, ROWS), (49153, 32, 32, None, ROWS), (49153, 64, 64, ROWS, ROWS), (69121, 32, 32, ROWS, ROWS), (32768, 32, 64, ROWS, ROWS),
    (32769, 32, 64, None, ROWS), (32769, 64, 64, None, None), (16384, 64, 128, ROWS, None), (16448, 64, 128, None, None), (32769, 64, 128, ROWS, None),
    # without gemm_bf16_kernel
    (40959, 12, 20, None, None), (40960, 12, 20, RAGGED, RAGGED), (50000, 4, 16, None, None), (50000, 4, 20, None, RAGGED), (81920, 12, 12, RAGGED, RAGGED),
    (81919, 12, 12, None, None), (90000, 8, 12, None, RAGGED), (700, 2, 6, None, RAGGED), (98303, 2, 2, None, None), (98304, 2, 2, RAGGED, RAGGED),
    (65536, 2, 64, RAGGED, ROWS), (700, 32, 12, ROWS, None), (12287, 64, 12, None, None), (12288, 64, 12, ROWS, None), (6144, 64, 20, ROWS, None),
    (98304, 20, 64, RAGGED, ROWS), (98303, 20, 64, RAGGED, None)])
def test_lines_to_the_other_kernels(n, ci, co, fwd, bwd):
    lv = _sheet(n)
    X, W, G = _data(n, ci, co)
    out, names = _products(lv, X, W, G)
    for got, want, name, form in zip(out, _wants(lv, X, W, G), names, (fwd, bwd)):
        assert [k.split("_kernel")[0] for k in name if "conv" in k] == ([form] if form else []), names
        _check(got, want)


@pytest.mark.parametrize("n,waves", [(98303, 4), (98304, 8)])
def test_workgroups_of_256_rows(n, waves):
    """64 channels to 64 columns, by the names that a profiler prints."""
    _, names = _products(_sheet(n), *_data(n, 64, 64))
    assert names == [[f"conv_bf16_kernel<4, 64, {waves}, false>"], [f"conv_bf16_kernel<4, 64, {waves}, true>"]]


def _sheet(n):
    """A plane of voxels, so with up to 9 neighbours each."""
    q = torch.arange(n)
    c = torch.stack([q // 400, torch.full_like(q, 5), q % 400], 1).int().numpy()
    return hch.hch_build_levels_device(c, [0, n], 512, 1)


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
@pytest.mark.parametrize("ci,co", [(50, 34), (6, 18)])
def test_numbers_that_are_not_finite(value, ci, co):
    """A row's reach the voxels that have it as a neighbour and no others, also from the channels next to a tail's end; a weight's its column."""
    n = 500
    lv = _levels(n, 32)
    X, W, G = _data(n, ci, co)
    clean, _ = _products(lv, X, W, G)
    nb = torch.from_numpy(lv.info(0).device_nbr27().astype("int64")).cuda()
    for v in (0, n // 2, n - 1):
        B, H = X.clone(), G.clone()
        B[v, 0] = B[v, ci - 1] = H[v, 0] = H[v, co - 1] = value
        near = (nb == v).any(1)
        for got, ref in zip(_products(lv, B, W, H)[0], clean):
            assert not torch.isfinite(got[near]).any() and torch.equal(got[~near], ref[~near])
    for tap in (0, 13, 26):
        B = W.clone()
        B[tap, 0, 0] = value                               # next to the end of the tap before
        for k, (got, ref) in enumerate(zip(_products(lv, X, B, G)[0], clean)):
            assert torch.equal(got[:, 1:], ref[:, 1:])
            assert not torch.isfinite(got[nb[:, 26 - tap if k else tap] >= 0, 0]).any()
