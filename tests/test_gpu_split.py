"""The products on split operands (fp32 inputs cut into bf16 pieces, conv_split_kernel and
wgrad_split_kernel) and the finer of the two row orders, at the sizes where they can go wrong:
channel counts around the tiles of 16, 32 and 64 and with remainders of 8 and of 4, a single voxel,
one voxel around the 64- and 128-row tiles, levels with and without a fine order.

The reference is the definition in fp64 over the oracle's neighbour lists.  Bound: what the six
piece products leave out is at most 2^-24 of a product and 2^-27 in the mean square; a sum of K terms is
rounded about K / 8 times to 2^-24 of its size at the time (the instruction rounds once per 8 terms),
0.29 * 2^-23 * sqrt(K / 16) of the result in any order: 5e-7 for K <= 27 * 130 forward and in the data
gradient.  The weight gradient rounds once per 32 voxels and adds at most 256 partial sums: 4e-7.
Together below 1e-6 of the result's norm."""
import numpy as np
import pytest

import synth_shapes as S

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
hch = pytest.importorskip("paper_1803_11385_amd")

BOUND = 1e-6


def _workspace(nbytes):
    t = torch.full((max(nbytes, 256) + 256,), 255, dtype=torch.uint8, device="cuda")
    off = (-t.data_ptr()) % 256
    return t[off: off + max(nbytes, 256)]


def _ws(lv, l, ci, co):
    return _workspace(max(hch.hch_conv_workspace_bytes(lv, l, ci, co, hch.HCH_F32, k, a)
                          for k in (hch.HCH_WS_FWD, hch.HCH_WS_BWD_DATA, hch.HCH_WS_BWD_WEIGHT)
                          for a in (hch.HCH_ALGO_FUSED, hch.HCH_ALGO_FUSED_DENSE)))


def _run(lv, l, X, W, G, a=hch.HCH_ALGO_FUSED):
    n, ci = X.shape
    co = G.shape[1]
    Y = torch.full((n, co), float("nan"), device="cuda")
    dX = torch.full((n, ci), float("nan"), device="cuda")
    dW = torch.full((27, ci, co), float("nan"), device="cuda")
    hch.hch_conv_fwd(lv, l, hch.HCH_F32, X, W, Y, ci, co, _ws(lv, l, ci, co), a)
    hch.hch_conv_bwd_data(lv, l, hch.HCH_F32, G, W, dX, ci, co, _ws(lv, l, ci, co), a)
    hch.hch_conv_bwd_weight(lv, l, hch.HCH_F32, X, G, dW, ci, co, _ws(lv, l, ci, co), a)
    return Y, dX, dW


def _reference(nbr, X, W, G):
    nb = torch.from_numpy(nbr.astype(np.int64)).cuda()
    X, W, G = X.double(), W.double(), G.double()

    def rows(T, k):
        return torch.where(nb[:, k:k + 1] >= 0, T[nb[:, k].clamp(min=0)], torch.zeros((), dtype=T.dtype, device="cuda"))
    Y = sum(rows(X, k) @ W[k] for k in range(27))
    dX = sum(rows(G, k) @ W[26 - k].T for k in range(27))
    dW = torch.stack([rows(X, k).T @ G for k in range(27)])
    return Y, dX, dW


def _forms(lv, X, W, G):
    """The kernels of the forward product and the data gradient, without their arguments."""
    (n, ci), co, Y, dX = X.shape, G.shape[1], torch.empty_like(G), torch.empty_like(X)
    names = [_launched(lambda: hch.hch_conv_fwd(lv, 0, hch.HCH_F32, X, W, Y, ci, co, _ws(lv, 0, ci, co), hch.HCH_ALGO_FUSED)),
             _launched(lambda: hch.hch_conv_bwd_data(lv, 0, hch.HCH_F32, G, W, dX, ci, co, _ws(lv, 0, ci, co), hch.HCH_ALGO_FUSED))]
    return {k.split("<")[0] for some in names for k in some if not k.startswith("splitk_reduce")}


def _check(got, want):
    for g, w, what in zip(got, want, ("Y", "dX", "dW")):
        err = float((g.double() - w).norm() / w.norm())
        assert err < BOUND, f"{what}: {err:.2e}"          # NaN fails too


@pytest.fixture(scope="module")
def batch(oracle):
    coords, offs, _ = S.config_batch(2)
    return hch.hch_build_levels(coords, offs, 64, 3), oracle.build_hierarchy(coords, offs, 64, 3)


@pytest.mark.parametrize("level", [0, 1, 2])            # 126k and 39k voxels with a fine order, 10k without
@pytest.mark.parametrize("ci,co", [(3, 16), (5, 7), (16, 32), (18, 22), (24, 40), (33, 17), (50, 50), (64, 64), (96, 20), (32, 130)])
def test_products_on_split_operands(oracle, batch, level, ci, co):
    lv, olv = batch
    n = olv[level].Ntot
    g = torch.Generator(device="cuda")
    g.manual_seed(1000 * level + 10 * ci + co)
    X, W, G = (torch.randn(s, device="cuda", generator=g) for s in ((n, ci), (27, ci, co), (n, co)))
    _check(_run(lv, level, X, W, G), _reference(oracle.neighbours(olv[level]), X, W, G))


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 127, 128, 129, 1000])
@pytest.mark.parametrize("ci,co", [(33, 50), (64, 18), (64, 130), (96, 96)])
def test_small_batches_in_any_order(oracle, n, ci, co):
    """Voxels in an order of their own (not by position), in two models.  conv_split_kernel has the last two pairs of channels and the
    data gradient of 50 channels, conv_small_kernel the rest."""
    rng = np.random.default_rng(n)
    pos = rng.permutation(12 ** 3)[:n]
    coords = np.stack([pos // 144, pos // 12 % 12, pos % 12], 1).astype(np.int32)
    offs = [0, n // 3, n] if n >= 3 else [0, n]
    lv = hch.hch_build_levels(coords, offs, 16, 1)
    nbr = oracle.neighbours(oracle.build_hierarchy(coords, offs, 16, 1)[0])
    X, W, G = (torch.from_numpy(rng.standard_normal(s, dtype=np.float32)).cuda() for s in ((n, ci), (27, ci, co), (n, co)))
    _check(_run(lv, 0, X, W, G), _reference(nbr, X, W, G))
    assert _forms(lv, X, W, G) == ({"conv_split_kernel"} if ci * co > 8192 else {"conv_small_kernel", "conv_split_kernel"} if co == 50 else {"conv_small_kernel"})


@pytest.mark.parametrize("n", [24512, 24513, 24576, 24577, 24641])
@pytest.mark.parametrize("ci,co", [(32, 64), (12, 20), (33, 50)])
def test_around_the_wider_workgroups(oracle, n, ci, co):
    """From 384 tiles of 64 rows on (24 513 voxels) a workgroup has 128 rows: the last one whole, a half
    and a row of a half."""
    rng = np.random.default_rng(n)
    pos = np.sort(rng.permutation(48 ** 3)[:n])
    coords = np.stack([pos // 2304, pos // 48 % 48, pos % 48], 1).astype(np.int32)
    lv = hch.hch_build_levels(coords, [0, n], 64, 1)
    nbr = oracle.neighbours(oracle.build_hierarchy(coords, [0, n], 64, 1)[0])
    X, W, G = (torch.from_numpy(rng.standard_normal(s, dtype=np.float32)).cuda() for s in ((n, ci), (27, ci, co), (n, co)))
    _check(_run(lv, 0, X, W, G), _reference(nbr, X, W, G))


@pytest.mark.parametrize("sign", ["any", "positive"])
@pytest.mark.parametrize("ci,co", [(256, 64), (512, 64), (512, 512)])
def test_many_channels(oracle, ci, co, sign):
    """All 27 taps of up to 512 channels: up to 432 steps of 32 terms in one chain of sums.  Bound as
    above, 0.29 * 2^-23 * sqrt(27 * 512 / 16) = 1.02e-6, and neither the error nor its mean beyond those
    of the fp32 instruction (HCH_ALGO_FUSED_DENSE), whose roundings lean the same way in sums of one
    sign; 5e-9 is what the mean of random roundings can come to, 1e-6 / sqrt(27 * 256 * 64) times 3."""
    q = np.arange(16 ** 3)
    coords = np.stack([q // 256, q // 16 % 16, q % 16], 1).astype(np.int32)
    lv = hch.hch_build_levels(coords, [0, q.size], 16, 1)
    nbr = oracle.neighbours(oracle.build_hierarchy(coords, [0, q.size], 16, 1)[0])
    g = torch.Generator(device="cuda")
    g.manual_seed(ci + co)
    X, W, G = (torch.randn(s, device="cuda", generator=g) for s in ((q.size, ci), (27, ci, co), (q.size, co)))
    if sign == "positive":
        X, W, G = X.abs(), W.abs(), G.abs()
    def errors(got):
        d = [(t.double() - w, w) for t, w in zip(got, want)]
        return [(float(e.norm() / w.norm()), abs(float(e.mean() / w.pow(2).mean().sqrt()))) for e, w in d]
    want = _reference(nbr, X, W, G)
    for split, plain in zip(errors(_run(lv, 0, X, W, G)), errors(_run(lv, 0, X, W, G, hch.HCH_ALGO_FUSED_DENSE))):
        assert split[0] < 1.1e-6 and split[0] <= plain[0]
        assert split[1] <= plain[1] + 5e-9


WORST = np.array([0x3F80FFFF, 0x3F807FC0, 0x3F800001, 0x3FFFFFFF], np.uint32).view(np.float32)


@pytest.mark.parametrize("values", ["worst", "random"])
@pytest.mark.parametrize("ci,co", [(33, 50), (64, 64), (91, 92), (64, 130)])
def test_single_products(values, ci, co):
    """Voxels without neighbours and rows with one number that is not zero: every result is one
    product.  The pieces leave out at most
    2^-24 of it and it is rounded once more, to 2^-24; neither has a preferred direction: the mean
    over all products is far below one rounding.  The mantissas 0x00FFFF and 0x007FC0 are the worst
    for pieces that are cut off and for pieces that are rounded."""
    rng = np.random.default_rng(7 * ci + co)
    n = min(ci, co)
    q = np.arange(n)
    coords = np.stack([q // 256 * 4 + 1, q // 16 % 16 * 4 + 1, q % 16 * 4 + 1], 1).astype(np.int32)
    lv = hch.hch_build_levels(coords, [0, n], 64, 1)

    def draw(*shape):
        a = rng.standard_normal(shape, dtype=np.float32) if values == "random" else rng.choice(WORST, shape) * rng.choice([-1.0, 1.0], shape)
        return torch.from_numpy(a.astype(np.float32)).cuda()

    W = draw(27, ci, co)
    X, G = torch.zeros((n, ci), device="cuda"), torch.zeros((n, co), device="cuda")
    X[q, q], G[q, q] = draw(n), draw(n)
    full = draw(n, co)
    Y, dX, _ = _run(lv, 0, X, W, G)
    dW = _run(lv, 0, X, W, full)[2]
    C = W[13].double()
    x, g = X[q, q].double(), G[q, q].double()
    assert _forms(lv, X, W, G) == ({"conv_split_kernel"} if ci * co > 8192 else {"conv_small_kernel", "conv_split_kernel"} if co == 50 else {"conv_small_kernel"})
    for got, want in ((Y, x[:, None] * C[:n]), (dX, g[:, None] * C.T[:n]), (dW[13, :n], x[:, None] * full.double())):
        err = (got.double() - want) / want.abs()
        assert float(err.abs().max()) <= 2.0 ** -23
        if values == "random":               # (a dozen mantissas have a mean of their own)
            assert abs(float((err * want.sign()).mean())) < 2.0 ** -27      # 2^-25 / sqrt(1650 products), five times


@pytest.mark.parametrize("scale", [1e-30, 1e-12, 1e12])
def test_any_scale(oracle, batch, scale):
    """The same relative error for small and for large numbers."""
    lv, olv = batch
    n = olv[2].Ntot
    X, W, G = (torch.randn(s, device="cuda") for s in ((n, 50), (27, 50, 50), (n, 50)))
    X, G = X * scale, G * scale
    W = W / max(scale, 1.0)
    got, want = _run(lv, 2, X, W, G), _reference(oracle.neighbours(olv[2]), X, W, G)
    _check(got[:2], want[:2])
    if scale >= 1e-12:
        _check([got[2]], [want[2]])


@pytest.mark.parametrize("a,b", [(1e-34, 1.0), (1e-36, 1.0), (1.0, 1e-36), (1e-40, 1e20), (1e20, 1e-40), (1e30, 1e-30)])
def test_ends_of_the_range(oracle, batch, a, b):
    """Operands down to the smallest fp32 numbers (1e-40 is a few tens of thousands times the smallest),
    with products in the ordinary range or exact to 2^-149: nothing is lost, the bound is the same."""
    lv, olv = batch
    n = olv[2].Ntot
    nbr = oracle.neighbours(olv[2])
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    X, W, G = (torch.randn(s, device="cuda", generator=g) for s in ((n, 50), (27, 50, 50), (n, 50)))
    _check(_run(lv, 2, X * a, W * b, G * a)[:2], _reference(nbr, X * a, W * b, G * a)[:2])
    _check(_run(lv, 2, X * a, W, G * b)[2:], _reference(nbr, X * a, W, G * b)[2:])


@pytest.mark.parametrize("value", [float("inf"), float("nan"), 3.2e38])
def test_numbers_that_are_not_finite(oracle, batch, value):
    """One infinity, NaN or number whose products leave the range: exactly the results it takes part
    in are not finite (or as large as they come), the others keep their values."""
    lv, olv = batch
    n = olv[2].Ntot
    nbr = oracle.neighbours(olv[2])
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    # no number below 0.01, whose product with 3.2e38 would not pass for a large one
    X, W, G = (t + torch.copysign(torch.full_like(t, 0.01), t) for t in
               (torch.randn(s, device="cuda", generator=g) for s in ((n, 50), (27, 50, 50), (n, 50))))
    clean = _run(lv, 2, X, W, G)
    v = n // 2
    X[v, 7] = value
    G[v, 9] = value
    Y, dX, dW = _run(lv, 2, X, W, G)
    near = torch.zeros(n, dtype=torch.bool, device="cuda")
    near[torch.from_numpy(np.unique(nbr[v][nbr[v] >= 0]).astype(np.int64)).cuda()] = True
    for got, ref in ((Y, clean[0]), (dX, clean[1])):
        assert torch.isfinite(got[~near]).all()
        err = (got[~near].double() - ref[~near].double()).norm() / ref.double().norm()
        assert float(err) < BOUND
        big = ~torch.isfinite(got[near]) | (got[near].abs() > 1e35)      # 3.2e38 * 0.01 = 3.2e36
        assert bool(big.all())
    hit = torch.zeros((27, 50, 50), dtype=torch.bool, device="cuda")
    for k in range(27):
        if (nbr[:, k] == v).any():
            hit[k, 7, :] = True                          # X[v][7] times some row of G
        if nbr[v, k] >= 0:
            hit[k, :, 9] = True                          # some row of X times G[v][9]
    assert torch.isfinite(dW[~hit]).all()
    assert float((dW[~hit].double() - clean[2][~hit].double()).norm() / clean[2].double().norm()) < BOUND
    assert bool((~torch.isfinite(dW[hit]) | (dW[hit].abs() > 1e35)).all())


@pytest.mark.parametrize("ci,co", [(16, 32), (32, 64), (64, 64), (33, 17), (64, 18), (5, 130), (18, 22)])
def test_sums_beyond_the_scaled_range(oracle, batch, ci, co):
    """Operands of 1e15: sums of 1e30 are ordinary numbers, but scaled by 2^32 for the split products they leave
    fp32's range, so that every wavefront repeats its sums with the fp32 instruction.  That rounds
    once per 4 terms and once more per 32: 0.29 * 2^-23 * sqrt(27 * 64 * (1 / 8 + 1 / 64)) = 5.4e-7."""
    lv, olv = batch
    n, no = olv[0].Ntot, olv[1].Ntot
    nbr = oracle.neighbours(olv[0])
    g = torch.Generator(device="cuda")
    g.manual_seed(10 * ci + co)
    X, W, G = (torch.randn(s, device="cuda", generator=g) * 1e15 for s in ((n, ci), (27, ci, co), (n, co)))
    _check(_run(lv, 0, X, W, G), _reference(nbr, X, W, G))
    field = torch.empty((no, 27), dtype=torch.int32, device="cuda")
    hch.hch_field_build(lv, 0, 3, 2, 1, field, None)
    dW = torch.full((27, ci, co), float("nan"), device="cuda")
    ws = _workspace(hch.hch_sconv_workspace_bytes(lv, 0, 3, 2, ci, co, hch.HCH_F32, hch.HCH_WS_BWD_WEIGHT))
    hch.hch_sconv_bwd_weight(lv, 0, 3, 2, hch.HCH_F32, X, G[:no], dW, field, ci, co, ws)
    rows = [torch.where(field[:, k:k + 1] >= 0, X.double()[field[:, k].clamp(min=0).long()], torch.zeros((), dtype=torch.float64, device="cuda"))
            for k in range(27)]
    want = torch.stack([r.T @ G[:no].double() for r in rows])
    assert float((dW.double() - want).norm() / want.norm()) < BOUND


@pytest.mark.parametrize("ci,co", [(32, 64), (50, 50)])
def test_numbers_that_are_not_finite_cost_no_more_than_a_few_times_as_much(batch, ci, co):
    """A step that overflows (every step of loss scaling that is thrown away): all rows NaN.  The yardstick
    is the fp32 instruction over every tap, which does not care; 2.0 to 2.4 times that was
    measured (32 -> 64), 0.9 to 1.6 times (50 -> 50), against 30 to 160 times with sums one by one."""
    lv, n = batch[0], batch[0].n(1)
    X, G, W = (torch.full(s, float("nan"), device="cuda") for s in ((n, ci), (n, co), (27, ci, co)))
    Y, dX, dW, ws = torch.empty_like(G), torch.empty_like(X), torch.empty_like(W), _ws(lv, 1, ci, co)

    def best(call, algo):
        times = []
        for _ in range(5):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            call(algo)
            e1.record()
            torch.cuda.synchronize()
            times.append(e0.elapsed_time(e1))
        return min(times)
    for call in (lambda a: hch.hch_conv_fwd(lv, 1, hch.HCH_F32, X, W, Y, ci, co, ws, a),
                 lambda a: hch.hch_conv_bwd_data(lv, 1, hch.HCH_F32, G, W, dX, ci, co, ws, a),
                 lambda a: hch.hch_conv_bwd_weight(lv, 1, hch.HCH_F32, X, G, dW, ci, co, ws, a)):
        assert best(call, hch.HCH_ALGO_FUSED) < 6 * best(call, hch.HCH_ALGO_FUSED_DENSE)
    assert torch.isnan(Y).all() and torch.isnan(dX).all() and torch.isnan(dW[13]).all()


def test_weight_gradient_with_the_smallest_workspace(oracle, batch):
    """A workspace that holds fewer partial sums than the query suggests gives the same result."""
    lv, olv = batch
    n, ci, co = olv[0].Ntot, 32, 64
    X, G = torch.randn((n, ci), device="cuda"), torch.randn((n, co), device="cuda")
    full = hch.hch_conv_workspace_bytes(lv, 0, ci, co, hch.HCH_F32, hch.HCH_WS_BWD_WEIGHT, hch.HCH_ALGO_FUSED)
    want = _reference(oracle.neighbours(olv[0]), X, torch.zeros((27, ci, co), device="cuda"), G)[2]
    for part in (104, 128):
        ws = _workspace(part * 27 * ci * co * 4)
        assert ws.numel() <= full
        dW = torch.full((27, ci, co), float("nan"), device="cuda")
        hch.hch_conv_bwd_weight(lv, 0, hch.HCH_F32, X, G, dW, ci, co, ws, hch.HCH_ALGO_FUSED)
        _check([dW], [want])
    with pytest.raises(hch.HchError):
        hch.hch_conv_bwd_weight(lv, 0, hch.HCH_F32, X, G, dW, ci, co, _workspace(8 * 27 * ci * co * 4), hch.HCH_ALGO_FUSED)


@pytest.mark.parametrize("n", [1, 128, 129, 384, 385, 1000])
@pytest.mark.parametrize("ci,co", [(16, 20), (50, 50)])
def test_bf16_weight_gradient_of_few_voxels(oracle, n, ci, co):
    """One to eight blocks of 128 voxels, not in order of position."""
    rng = np.random.default_rng(n)
    pos = rng.permutation(12 ** 3)[:n]
    coords = np.stack([pos // 144, pos // 12 % 12, pos % 12], 1).astype(np.int32)
    lv = hch.hch_build_levels(coords, [0, n], 16, 1)
    nbr = oracle.neighbours(oracle.build_hierarchy(coords, [0, n], 16, 1)[0])
    X, G = (torch.from_numpy(rng.standard_normal(s, dtype=np.float32)).cuda().bfloat16() for s in ((n, ci), (n, co)))
    need = hch.hch_conv_workspace_bytes(lv, 0, ci, co, hch.HCH_BF16, hch.HCH_WS_BWD_WEIGHT, hch.HCH_ALGO_FUSED)
    dW = torch.full((27, ci, co), float("nan"), device="cuda")
    hch.hch_conv_bwd_weight(lv, 0, hch.HCH_BF16, X, G, dW, ci, co, _workspace(need), hch.HCH_ALGO_FUSED)
    _check([dW], [_reference(nbr, X, torch.zeros((27, ci, co), device="cuda"), G)[2]])


@pytest.mark.parametrize("level", [0, 2])
@pytest.mark.parametrize("ci,co", [(6, 18), (50, 50), (64, 64), (32, 130), (34, 20)])
def test_bf16_weight_gradient(oracle, batch, level, ci, co):
    """Even channel counts of any kind (wgrad_bf16_kernel; 64 -> 64 takes it on the finest level only).
    bf16 inputs, exact products, fp32 sums: the same bound."""
    lv, olv = batch
    n = olv[level].Ntot
    X, G = torch.randn((n, ci), device="cuda").bfloat16(), torch.randn((n, co), device="cuda").bfloat16()
    ws = _workspace(hch.hch_conv_workspace_bytes(lv, level, ci, co, hch.HCH_BF16, hch.HCH_WS_BWD_WEIGHT, hch.HCH_ALGO_FUSED))
    dW = torch.full((27, ci, co), float("nan"), device="cuda")
    hch.hch_conv_bwd_weight(lv, level, hch.HCH_BF16, X, G, dW, ci, co, ws, hch.HCH_ALGO_FUSED)
    want = _reference(oracle.neighbours(olv[level]), X, torch.zeros((27, ci, co), device="cuda"), G)[2]
    _check([dW], [want])


def test_index_lists_alone(oracle):
    """hch_build_index_lists rewrites the lists and leaves the row orders as they are."""
    coords, offs, _ = S.config_batch(3, batch=4, u=64)
    lv, olv = hch.hch_build_levels(coords, offs, 64, 3), oracle.build_hierarchy(coords, offs, 64, 3)
    before = [(lv.info(l).device_row_order(), lv.info(l).device_tile_taps()) for l in range(3)]
    hch.hch_build_index_lists(lv, 0, 3)
    hch.hch_build_index_lists(lv, 1, 0)
    torch.cuda.synchronize()
    for l in range(3):
        assert np.array_equal(lv.info(l).device_nbr27(), oracle.neighbours(olv[l]))
        if l:
            assert np.array_equal(lv.info(l).device_child8(), oracle.children(olv[l - 1], olv[l]))
        assert np.array_equal(lv.info(l).device_row_order(), before[l][0])
        assert np.array_equal(lv.info(l).device_tile_taps(), before[l][1])
    with pytest.raises(hch.HchError):
        hch.hch_build_index_lists(lv, 2, 2)


@pytest.mark.parametrize("F,stride,pad", [(2, 2, 0), (3, 2, 1), (5, 1, 2), (3, 4, 1), (7, 1, 3)])
@pytest.mark.parametrize("ci,co", [(18, 22), (50, 50), (6, 22), (33, 130), (32, 64)])
def test_strided_weight_gradient(batch, F, stride, pad, ci, co):
    """wgrad_split_kernel on index rows of general fields: data order, X of another level than dY, 8 to 343
    taps over several row tiles (windows of 28 taps); with more than 28 taps, rows of fewer than 16
    channels stay with gemm_f32_kernel (6 -> 22), as does little work (32 -> 64, stride 4).  Against the definition over the index rows, which
    the parity tests check bit by bit.  (7^3, stride 1: dW has millions of elements; the coarsest level.)"""
    lv = batch[0]
    l = 1 if F == 7 else 0
    lo = l + {1: 0, 2: 1, 4: 2}[stride]
    n_in, n_out, F3 = lv.n(l), lv.n(lo), F ** 3
    field = torch.empty((n_out, F3), dtype=torch.int32, device="cuda")
    hch.hch_field_build(lv, l, F, stride, pad, field, None)
    g = torch.Generator(device="cuda")
    g.manual_seed(F * 100 + ci)
    X, G = torch.randn((n_in, ci), device="cuda", generator=g), torch.randn((n_out, co), device="cuda", generator=g)
    dW = torch.full((F3, ci, co), float("nan"), device="cuda")
    ws = _workspace(hch.hch_sconv_workspace_bytes(lv, l, F, stride, ci, co, hch.HCH_F32, hch.HCH_WS_BWD_WEIGHT))
    hch.hch_sconv_bwd_weight(lv, l, F, stride, hch.HCH_F32, X, G, dW, field, ci, co, ws)
    zero = torch.zeros((), dtype=torch.float64, device="cuda")
    want = torch.stack([torch.where(field[:, k:k + 1] >= 0, X.double()[field[:, k].clamp(min=0).long()], zero).T @ G.double()
                        for k in range(F3)])
    err = float((dW.double() - want).norm() / want.norm())
    assert err < BOUND, f"{err:.2e}"
    assert float((dW.double() - want).abs().max() / want.pow(2).mean().sqrt()) < 30 * BOUND     # no element out of place


def test_weight_gradients_do_not_depend_on_what_the_workspace_has_to_spare(batch):
    """The queried size and 64 MiB more give the same bits: plain and strided weight gradients."""
    lv = batch[0]
    n, no, ci, co = lv.n(0), lv.n(1), 32, 64
    X, G = torch.randn((n, ci), device="cuda"), torch.randn((n, co), device="cuda")
    field = torch.empty((no, 27), dtype=torch.int32, device="cuda")
    hch.hch_field_build(lv, 0, 3, 2, 1, field, None)
    need = hch.hch_conv_workspace_bytes(lv, 0, ci, co, hch.HCH_F32, hch.HCH_WS_BWD_WEIGHT, hch.HCH_ALGO_FUSED)
    strided = hch.hch_sconv_workspace_bytes(lv, 0, 3, 2, ci, co, hch.HCH_F32, hch.HCH_WS_BWD_WEIGHT)
    got = []
    for spare in (0, 64 << 20):
        a, b = (torch.full((27, ci, co), float("nan"), device="cuda") for _ in range(2))
        hch.hch_conv_bwd_weight(lv, 0, hch.HCH_F32, X, G, a, ci, co, _workspace(need + spare), hch.HCH_ALGO_FUSED)
        hch.hch_sconv_bwd_weight(lv, 0, 3, 2, hch.HCH_F32, X, G[:no], b, field, ci, co, _workspace(strided + spare))
        got.append((a, b))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])


@pytest.mark.parametrize("level,wide,narrow", [(1, 16384, 20), (1, 16384, 68), (0, 4352, 68)])
def test_operands_of_two_gigabytes(oracle, batch, level, wide, narrow):
    """Feature matrices of 2 GiB and more, which 32-bit byte offsets do not reach: the products on the fp32
    instruction, rows in order and absent taps left out (128 x 32, 64 x 64 and 128 x 64 tiles), and the
    dense weight gradient.  They round once per 4 terms: 0.29 * 2^-23 * sqrt(27 * 16384 / 8) = 8.1e-6."""
    lv, olv = batch
    n = olv[level].Ntot
    assert n * wide * 4 >= 1 << 31
    nb = torch.from_numpy(oracle.neighbours(olv[level]).astype(np.int64)).cuda()
    g = torch.Generator(device="cuda")
    g.manual_seed(narrow)
    big, small = torch.randn((n, wide), device="cuda", generator=g), torch.randn((n, narrow), device="cuda", generator=g)
    a = hch.HCH_ALGO_FUSED

    def rows(T, k):
        return torch.where(nb[:, k:k + 1] >= 0, T[nb[:, k].clamp(min=0)], torch.zeros((), device="cuda")).double()

    def check(got, want):
        assert float((got.double() - want).norm() / want.norm()) < 1e-5
    W = torch.randn((27, wide, narrow), device="cuda", generator=g)
    Y = torch.full((n, narrow), float("nan"), device="cuda")
    dW = torch.full((27, wide, narrow), float("nan"), device="cuda")
    hch.hch_conv_fwd(lv, level, hch.HCH_F32, big, W, Y, wide, narrow, _ws(lv, level, wide, narrow), a)
    hch.hch_conv_bwd_weight(lv, level, hch.HCH_F32, big, small, dW, wide, narrow, _ws(lv, level, wide, narrow), a)
    want = 0.0
    for k in range(27):
        r = rows(big, k)
        want = want + r @ W[k].double()
        check(dW[k], r.T @ small.double())
        del r
    check(Y, want)
    W = torch.randn((27, narrow, wide), device="cuda", generator=g)
    dX = torch.full((n, narrow), float("nan"), device="cuda")
    hch.hch_conv_bwd_data(lv, level, hch.HCH_F32, big, W, dX, narrow, wide, _ws(lv, level, narrow, wide), a)
    check(dX, sum(rows(big, k) @ W[26 - k].double().T for k in range(27)))


@pytest.mark.parametrize("F,stride,pad", [(2, 2, 0), (3, 2, 1), (3, 4, 1), (3, 1, 1)])
@pytest.mark.parametrize("ci,co", [(18, 33), (20, 130), (33, 50), (64, 64)])
def test_products_over_general_index_rows(batch, F, stride, pad, ci, co):
    """field_split_kernel, data gradient and, within a level, forward (between levels there are too few rows here for
    it, see test_products_between_two_large_levels): 126 665 rows (the last workgroup has 201), index rows in any order,
    rows without a single tap among them, channel counts with remainders; with the queried workspace and, on the ways
    taken without room for the cut weights, with less.  An infinity reaches the rows that hold it and no others."""
    lv = batch[0]
    lo = {1: 0, 2: 1, 4: 2}[stride]
    n_in, n_out, F3 = lv.n(0), lv.n(lo), F ** 3
    field, field_t = torch.empty((n_out, F3), dtype=torch.int32, device="cuda"), torch.empty((n_in, F3), dtype=torch.int32, device="cuda")
    hch.hch_field_build(lv, 0, F, stride, pad, field, field_t)
    g = torch.Generator(device="cuda")
    g.manual_seed(F * 100 + ci)
    X, G = torch.randn((n_in, ci), device="cuda", generator=g), torch.randn((n_out, co), device="cuda", generator=g)
    W = torch.randn((F3, ci, co), device="cuda", generator=g)
    zero = torch.zeros((), dtype=torch.float64, device="cuda")
    for kind, call, A, idx, w, n in ((hch.HCH_WS_FWD, hch.hch_sconv_fwd, X, field, W, n_out),
                                     (hch.HCH_WS_BWD_DATA, hch.hch_sconv_bwd_data, G, field_t, W.transpose(1, 2), n_in)):
        idx = idx[torch.randperm(n, device="cuda", generator=g)].contiguous()
        idx[n // 3: n // 3 + 40] = -1
        want = sum(torch.where(idx[:, k:k + 1] >= 0, A.double()[idx[:, k].clamp(min=0).long()], zero) @ w[k].double() for k in range(F3))
        out = torch.full((n, w.shape[2]), float("nan"), device="cuda")
        ws = _workspace(hch.hch_sconv_workspace_bytes(lv, 0, F, stride, ci, co, hch.HCH_F32, kind))
        call(lv, 0, F, stride, hch.HCH_F32, A, W, out, idx, ci, co, ws)
        assert float((out.double() - want).norm() / want.norm()) < BOUND
        assert float((out.double() - want).abs().max() / want.pow(2).mean().sqrt()) < 30 * BOUND
        again = torch.full_like(out, float("nan"))
        call(lv, 0, F, stride, hch.HCH_F32, A, W, again, idx, ci, co, ws)
        assert torch.equal(out, again)
        v = idx[idx >= 0][20000].item()
        B = A.clone()
        B[v, 3] = float("inf")
        call(lv, 0, F, stride, hch.HCH_F32, B, W, again, idx, ci, co, ws)
        holds = (idx == v).any(1)
        # rows multiplied together with one of those are summed with the fp32 instruction: other roundings, the same bound
        assert bool((~torch.isfinite(again[holds])).all()) and bool(torch.isfinite(again[~holds]).all())
        assert float((again.double() - want)[~holds].norm() / want.norm()) < BOUND
    if stride == 1:                                     # as little as the forward product has ever asked for
        out = torch.full((n_out, co), float("nan"), device="cuda")
        hch.hch_sconv_fwd(lv, 0, F, stride, hch.HCH_F32, X, W, out, field, ci, co, _workspace(256)[:256])
        want = sum(torch.where(field[:, k:k + 1] >= 0, X.double()[field[:, k].clamp(min=0).long()], zero) @ W[k].double() for k in range(F3))
        assert float((out.double() - want).norm() / want.norm()) < 4 * BOUND          # the fp32 instruction: a rounding per 4 terms


@pytest.fixture(scope="module")
def large():
    coords, offs, _ = S.config_batch(3)
    return hch.hch_build_levels_device(coords, offs, 128, 1)


@pytest.mark.parametrize("ci,co", [(32, 64), (64, 64), (96, 34), (130, 32), (64, 20), (20, 64), (64, 130)])
def test_bf16_products_over_the_row_order(batch, large, ci, co):
    """conv_bf16_kernel: steps of 32 and of 64 channels, 32 and 64 columns and several tiles of them with remainders, a last
    workgroup and a last wavefront that are not full; products are exact, so the bound is that of the fp32 sums.  Rows that
    are not finite reach their neighbours' results and no others."""
    lv = batch[0] if ci % 64 == 0 and co > 32 else large
    n = lv.n(0)
    assert n >= (98304 if lv is batch[0] else 196608) and n % 32
    nbr = torch.from_numpy(lv.info(0).device_nbr27().astype(np.int64)).cuda()
    g = torch.Generator(device="cuda")
    g.manual_seed(ci * 1000 + co)
    X, W, G = (torch.randn(s, device="cuda", generator=g).bfloat16() for s in ((n, ci), (27, ci, co), (n, co)))
    zero = torch.zeros((), dtype=torch.float64, device="cuda")
    for name, kind, A, w, m in (("hch_conv_fwd", hch.HCH_WS_FWD, X, W, co), ("hch_conv_bwd_data", hch.HCH_WS_BWD_DATA, G, W.flip(0).transpose(1, 2), ci)):
        want = sum(torch.where(nbr[:, k:k + 1] >= 0, A.double()[nbr[:, k].clamp(min=0)], zero) @ w[k].double() for k in range(27))
        out, again = torch.full((n, m), float("nan"), device="cuda"), torch.full((n, m), float("nan"), device="cuda")
        ws = _workspace(hch.hch_conv_workspace_bytes(lv, 0, ci, co, hch.HCH_BF16, kind, hch.HCH_ALGO_FUSED))
        call = lambda B, Y: getattr(hch, name)(lv, 0, hch.HCH_BF16, B, W, Y, ci, co, ws, hch.HCH_ALGO_FUSED)
        call(A, out)
        assert float((out.double() - want).norm() / want.norm()) < BOUND
        assert float((out.double() - want).abs().max() / want.pow(2).mean().sqrt()) < 30 * BOUND
        B = A.clone()
        v = n // 2
        B[v, 1] = float("nan")
        call(B, again)
        near = (nbr == v).any(1)
        assert bool(torch.isnan(again[near]).all()) and torch.equal(again[~near], out[~near])


def _launched(call):
    """Names of the kernels that `call` launches."""
    hch.hch_profile_reset()
    hch.hch_profile_enable(-1, True)
    try:
        call()
        torch.cuda.synchronize()
    finally:
        hch.hch_profile_enable(-1, False)
    return {hch.hch_kernel_name(i) for i in range(hch.hch_kernel_count()) if hch.hch_profile_read(i)["launches"]}


def _gathered(A, idx, w):
    zero = torch.zeros((), dtype=torch.float64, device="cuda")
    return sum(torch.where(idx[:, k:k + 1] >= 0, A.double()[idx[:, k].clamp(min=0).long()], zero) @ w[k].double() for k in range(idx.shape[1]))


def _sconv(lv, kind, F, stride, A, W, n, idx, ci, co):
    out = torch.full((n, co if kind == hch.HCH_WS_FWD else ci), float("nan"), device="cuda")
    call = hch.hch_sconv_fwd if kind == hch.HCH_WS_FWD else hch.hch_sconv_bwd_data
    ws = _workspace(hch.hch_sconv_workspace_bytes(lv, 0, F, stride, ci, co, hch.HCH_F32, kind))
    names = _launched(lambda: call(lv, 0, F, stride, hch.HCH_F32, A, W, out, idx, ci, co, ws))
    return out, names


@pytest.fixture(scope="module")
def halves():
    coords, offs, _ = S.config_batch(4)
    return hch.hch_build_levels_device(coords, offs, 256, 2)


@pytest.mark.parametrize("F,pad,ci,co,fwd,bwd", [(3, 1, 16, 32, "2, false", "1, true"), (3, 1, 50, 13, "1, false", "4, true"),
                                                (3, 1, 7, 50, None, "1, true"), (3, 1, 32, 16, "1, false", "2, true"),
                                                (2, 0, 64, 20, "2, false", None), (2, 0, 18, 40, None, "2, true"),
                                                (2, 0, 32, 64, "4, false", "2, true")])
def test_products_between_two_large_levels(halves, F, pad, ci, co, fwd, bwd):
    """field_split_kernel between two levels, the forward product with more rows in X than in the result and the data
    gradient with fewer: 16, 32 and 64 columns to a workgroup, 27 and 8 taps, channels with remainders.  None: the product
    goes another way."""
    lv = halves
    n_in, n_out = lv.n(0), lv.n(1)
    assert n_in >= 262144 and n_out >= 98304
    field, field_t = (torch.empty((n, F ** 3), dtype=torch.int32, device="cuda") for n in (n_out, n_in))
    hch.hch_field_build(lv, 0, F, 2, pad, field, field_t)
    g = torch.Generator(device="cuda")
    g.manual_seed(F * 100 + ci)
    X, G, W = (torch.randn(s, device="cuda", generator=g) for s in ((n_in, ci), (n_out, co), (F ** 3, ci, co)))
    for kind, A, idx, w, n, form in ((hch.HCH_WS_FWD, X, field, W, n_out, fwd), (hch.HCH_WS_BWD_DATA, G, field_t, W.transpose(1, 2), n_in, bwd)):
        out, names = _sconv(lv, kind, F, 2, A, W, n, idx, ci, co)
        assert [x for x in names if x.startswith("field_split")] == ([f"field_split_kernel<{form}>"] if form else []), names
        want = _gathered(A, idx, w)
        # the other ways are the fp32 instruction: a rounding per 4 terms
        assert float((out.double() - want).norm() / want.norm()) < (BOUND if form else 4 * BOUND)
        assert float((out.double() - want).abs().max() / want.pow(2).mean().sqrt()) < (30 if form else 120) * BOUND


@pytest.fixture(scope="module")
def fields(batch):
    """Index rows of 3^3 fields of level 0: within it (forward) and from level 1 (data gradient of stride 2)."""
    lv = batch[0]
    within, between = (torch.empty((lv.n(0), 27), dtype=torch.int32, device="cuda") for _ in range(2))
    hch.hch_field_build(lv, 0, 3, 1, 1, within, None)
    hch.hch_field_build(lv, 0, 3, 2, 1, None, between)
    return within, between


def _both_products(lv, fields, X, G, W):
    """Forward within level 0 and data gradient from level 1, each with its exact result and its index rows."""
    ci, co = W.shape[1:]
    for kind, stride, A, idx, w in ((hch.HCH_WS_FWD, 1, X, fields[0], W), (hch.HCH_WS_BWD_DATA, 2, G, fields[1], W.transpose(1, 2))):
        out, names = _sconv(lv, kind, 3, stride, A, W, lv.n(0), idx, ci, co)
        assert any(x.startswith("field_split_kernel") for x in names), names
        yield out, A, idx, w


@pytest.mark.parametrize("a,b", [(1e-30, 1.0), (1e30, 1e-30), (1e-36, 1.0), (1.0, 1e-36), (1e-40, 1e20), (1e20, 1e-40), (1e15, 1e15)])
def test_ends_of_the_range_over_general_index_rows(batch, fields, a, b):
    """As test_ends_of_the_range and, with 1e15, test_sums_beyond_the_scaled_range, for field_split_kernel."""
    lv = batch[0]
    g = torch.Generator(device="cuda")
    g.manual_seed(11)
    X, G, W = (torch.randn(s, device="cuda", generator=g) for s in ((lv.n(0), 50), (lv.n(1), 50), (27, 50, 50)))
    for out, A, idx, w in _both_products(lv, fields, X * a, G * a, W * b):
        want = _gathered(A, idx, w)
        assert float((out.double() - want).norm() / want.norm()) < BOUND


@pytest.mark.parametrize("value", [float("inf"), float("nan"), 3.2e38])
def test_weights_that_are_not_finite_over_general_index_rows(batch, fields, value):
    """One weight: exactly the results that it takes part in are not finite (or as large as they come)."""
    lv = batch[0]
    g = torch.Generator(device="cuda")
    g.manual_seed(12)
    X, G, W = (t + torch.copysign(torch.full_like(t, 0.01), t) for t in
               (torch.randn(s, device="cuda", generator=g) for s in ((lv.n(0), 50), (lv.n(1), 50), (27, 50, 50))))
    B = W.clone()
    B[4, 7, 9] = value
    for (out, A, idx, w), column in zip(_both_products(lv, fields, X, G, B), (9, 7)):
        want = _gathered(A, idx, w.where(torch.isfinite(w) & (w.abs() < 1e38), torch.zeros_like(w)))
        hit = torch.zeros_like(out, dtype=torch.bool)
        hit[idx[:, 4] >= 0, column] = True
        assert bool(hit.any()) and bool(torch.isfinite(out[~hit]).all())
        assert float((out.double() - want)[~hit].norm() / want.norm()) < BOUND
        assert bool((~torch.isfinite(out[hit]) | (out[hit].abs() > 1e35)).all())


@pytest.mark.parametrize("ci,co,fwd,bwd", [(32, 32, "2, 32, 4, false", "2, 32, 4, true"), (96, 20, "2, 32, 4, false", None), (20, 96, None, "2, 32, 4, true"),
                                          (64, 64, "4, 64, 8, false", "4, 64, 8, true")])
def test_bf16_weights_that_are_not_finite(large, ci, co, fwd, bwd):
    """The forms of conv_bf16_kernel with steps of 32 channels and 32 columns (and one other): an infinite weight reaches the
    rows that have its tap, in its column.  (Rows without the tap have 0 * inf there or leave the tap out, as their tile
    has it: not looked at.)  Everything else is as with a finite weight, to the bit."""
    lv, n = large, large.n(0)
    assert n >= 196608
    nbr = torch.from_numpy(lv.info(0).device_nbr27()).cuda()
    g = torch.Generator(device="cuda")
    g.manual_seed(ci * 1000 + co)
    X, G, W = (torch.randn(s, device="cuda", generator=g).bfloat16() for s in ((n, ci), (n, co), (27, ci, co)))
    B = W.clone()
    B[4, 7, 9] = float("inf")
    for name, kind, A, w, tap, row, column, form in (("hch_conv_fwd", hch.HCH_WS_FWD, X, W, 4, 7, 9, fwd),
                                                     ("hch_conv_bwd_data", hch.HCH_WS_BWD_DATA, G, W.flip(0).transpose(1, 2), 22, 9, 7, bwd)):
        ws = _workspace(hch.hch_conv_workspace_bytes(lv, 0, ci, co, hch.HCH_BF16, kind, hch.HCH_ALGO_FUSED))
        outs = [torch.full((n, w.shape[2]), float("nan"), device="cuda") for _ in range(2)]
        for weights, out in zip((W, B), outs):
            names = _launched(lambda: getattr(hch, name)(lv, 0, hch.HCH_BF16, A, weights, out, ci, co, ws, hch.HCH_ALGO_FUSED))
            assert [x for x in names if x.startswith("conv_bf16")] == ([f"conv_bf16_kernel<{form}>"] if form else []), names
        want = _gathered(A, nbr, w)
        assert float((outs[0].double() - want).norm() / want.norm()) < BOUND
        has = nbr[:, tap] >= 0
        x = A[nbr[has, tap].long(), row].float()
        assert torch.equal(outs[1][has, column][x != 0], (torch.sign(x) * float("inf"))[x != 0])
        others = [c for c in range(w.shape[2]) if c != column]
        assert torch.equal(outs[1][:, others], outs[0][:, others])


@pytest.fixture(scope="module")
def scattered():
    pos = np.sort(np.random.default_rng(75).permutation(64 ** 3)[:75000])
    return hch.hch_build_levels_device(np.stack([pos // 4096, pos // 64 % 64, pos % 64], 1).astype(np.int32), [0, 75000], 64, 1)


@pytest.mark.parametrize("levels,F,stride,pad,ci,co,kind,split",
                         [("scattered", 3, 1, 1, 20, 64, "fwd", False), ("scattered", 3, 1, 1, 24, 128, "fwd", True),
                          ("scattered", 3, 1, 1, 18, 64, "fwd", True), ("scattered", 3, 1, 1, 20, 64, "fwd unaligned", True),
                          ("scattered", 3, 1, 1, 64, 20, "bwd", False), ("scattered", 3, 1, 1, 62, 20, "bwd", True),
                          ("halves", 1, 1, 0, 64, 64, "fwd", False), ("halves", 1, 1, 0, 32, 128, "bwd", False),
                          ("halves", 2, 2, 0, 128, 64, "fwd", False), ("halves", 2, 2, 0, 64, 64, "fwd", True),
                          ("halves", 2, 2, 0, 8, 32, "bwd", False), ("halves", 3, 2, 1, 8, 32, "bwd", True)])
def test_where_general_index_rows_go(request, levels, F, stride, pad, ci, co, kind, split):
    """Shapes on both sides of the lines of field_split_ok, with their results: one tap, rounds of workgroups that fill the chip or
    hardly more than a half of it, operands beyond the last-level cache, few columns; without the vector path of
    gemm_f32_kernel (channels, alignment) all of them on split operands."""
    lv = request.getfixturevalue(levels)
    n_in, n_out = lv.n(0), lv.n(stride // 2)
    forward = kind.startswith("fwd")
    idx = torch.empty((n_out if forward else n_in, F ** 3), dtype=torch.int32, device="cuda")
    hch.hch_field_build(lv, 0, F, stride, pad, *((idx, None) if forward else (None, idx)))
    g = torch.Generator(device="cuda")
    g.manual_seed(ci * 1000 + co)
    A, W = (torch.randn(s, device="cuda", generator=g) for s in ((n_in, ci) if forward else (n_out, co), (F ** 3, ci, co)))
    if kind.endswith("unaligned"):
        A = torch.empty(A.numel() + 1, device="cuda")[1:].view(A.shape).copy_(A)
    out, names = _sconv(lv, hch.HCH_WS_FWD if forward else hch.HCH_WS_BWD_DATA, F, stride, A, W, idx.shape[0], idx, ci, co)
    assert any(x.startswith("field_split_kernel") for x in names) == split, names
    want = _gathered(A, idx, W if forward else W.transpose(1, 2))
    # the fp32 instruction: a rounding per 4 terms
    assert float((out.double() - want).norm() / want.norm()) < (BOUND if split else 4 * BOUND)


def _sphere_shells(radius, half):
    """Two shells of a sphere of 2 * half voxels."""
    g = np.arange(256) - 128
    parts = [np.argwhere(np.abs(np.sqrt((g[:, None, None] + a) ** 2 + (g[None, :, None] + 0.2) ** 2 + (g[None, None, :] + 0.3) ** 2) - radius) < half)
             for a in (0.0, 0.1)]
    return hch.hch_build_levels_device(np.concatenate(parts).astype(np.int32), [0, len(parts[0]), len(parts[0]) + len(parts[1])], 256, 1)


@pytest.fixture(scope="module")
def shells():
    sets = {(n, tap_major): _sphere_shells(*shape) for n, shape in ((14, (85, 0.7)), (18, (72, 0.99)), (21, (58, 1.5))) for tap_major in (False, True)}
    for (_, tap_major), lv in sets.items():
        if tap_major:
            hch.hch_build_tap_major(lv, 0)
    return sets


@pytest.mark.parametrize("neighbours,tap_major,ci,co,fwd,bwd", [(14, False, 64, 64, True, True), (14, True, 64, 64, False, False),
                                                               (14, False, 64, 32, False, True), (18, False, 64, 64, False, False),
                                                               (18, False, 32, 64, True, False), (18, True, 96, 96, True, True),
                                                               (18, False, 32, 32, False, False), (21, False, 32, 64, False, False)])
def test_bf16_products_of_thick_shells(shells, neighbours, tap_major, ci, co, fwd, bwd):
    """Levels whose voxels have 14, 18 and 21 neighbours, on both sides of the lines of conv_bf16_ok, with the results."""
    lv = shells[neighbours, tap_major]
    n = lv.n(0)
    assert n >= 196608 and neighbours - 0.5 < lv.info(0).nbr_valid / n < neighbours + (0 if neighbours == 18 else 0.5)
    nbr = torch.from_numpy(lv.info(0).device_nbr27()).cuda()
    g = torch.Generator(device="cuda")
    g.manual_seed(ci * 1000 + co)
    X, G, W = (torch.randn(s, device="cuda", generator=g).bfloat16() for s in ((n, ci), (n, co), (27, ci, co)))
    for name, kind, A, w, over_order in (("hch_conv_fwd", hch.HCH_WS_FWD, X, W, fwd), ("hch_conv_bwd_data", hch.HCH_WS_BWD_DATA, G, W.flip(0).transpose(1, 2), bwd)):
        out = torch.full((n, w.shape[2]), float("nan"), device="cuda")
        ws = _workspace(hch.hch_conv_workspace_bytes(lv, 0, ci, co, hch.HCH_BF16, kind, hch.HCH_ALGO_FUSED))
        names = _launched(lambda: getattr(hch, name)(lv, 0, hch.HCH_BF16, A, W, out, ci, co, ws, hch.HCH_ALGO_FUSED))
        assert any(x.startswith("conv_bf16_kernel") for x in names) == over_order, names
        want = _gathered(A, nbr, w)
        assert float((out.double() - want).norm() / want.norm()) < BOUND


@pytest.mark.parametrize("F,pad,ci,co", [(3, 1, 16, 32), (2, 0, 64, 64), (3, 1, 64, 4), (3, 1, 1, 256)])
def test_workspace_of_strided_data_gradients(halves, F, pad, ci, co):
    """What goes without the gradient of the column matrix asks for the cut weights only, 6 bytes a weight with channels
    padded to 8 and columns to 16, works in that and is refused with less; what goes through it asks for it.  The old
    answer is taken as before."""
    lv = halves
    n_in, n_out = lv.n(0), lv.n(1)
    column = n_out * F ** 3 * ci * 4
    need = hch.hch_sconv_workspace_bytes(lv, 0, F, 2, ci, co, hch.HCH_F32, hch.HCH_WS_BWD_DATA)
    split = (ci, co) not in ((64, 4), (1, 256))            # 27 * 4 terms are too few; a column is
    assert need == -(-(F ** 3 * (-(-co // 8) * 8) * (-(-ci // 16) * 16) * 6 if split else column) // 256) * 256
    field_t = torch.empty((n_in, F ** 3), dtype=torch.int32, device="cuda")
    hch.hch_field_build(lv, 0, F, 2, pad, None, field_t)
    g = torch.Generator(device="cuda")
    g.manual_seed(ci)
    G, W = (torch.randn(s, device="cuda", generator=g) for s in ((n_out, co), (F ** 3, ci, co)))
    want = _gathered(G, field_t, W.transpose(1, 2))
    outs = []
    for size in {need, max(need, column)}:
        outs.append(torch.full((n_in, ci), float("nan"), device="cuda"))
        hch.hch_sconv_bwd_data(lv, 0, F, 2, hch.HCH_F32, G, W, outs[-1], field_t, ci, co, _workspace(size))
        assert float((outs[-1].double() - want).norm() / want.norm()) < 4 * BOUND
    assert all(torch.equal(o, outs[0]) for o in outs)
    with pytest.raises(hch.HchError) as e:
        hch.hch_sconv_bwd_data(lv, 0, F, 2, hch.HCH_F32, G, W, outs[0], field_t, ci, co, _workspace(need)[:need - 256])
    assert e.value.status == 6
