"""Index rows of general fields (field_kernel) where the rows are shared by several workgroups: every split
of the planes, one and two rows of workgroups per voxel tile, both forms of the transposed rows,
voxel counts around the tiles of 64 and of 32.  Bit-exact against the oracle and the inverse
relation; and what long rows of few voxels cost."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
hch = pytest.importorskip("paper_1803_11385_amd")


def _shapes(n, u, seed):
    rng = np.random.default_rng(seed)
    lin = np.sort(rng.permutation(u ** 3)[:n])
    coords = np.stack([lin // (u * u), lin // u % u, lin % u], 1).astype(np.int32)
    return coords, ([0, n // 3, n] if n >= 3 else [0, n])


@pytest.mark.parametrize("n", [1, 31, 33, 64, 65, 200, 3000])
@pytest.mark.parametrize("F,stride,pad", [(1, 1, 0), (3, 1, 1), (5, 1, 2), (7, 1, 3), (3, 2, 1), (6, 2, 2), (7, 2, 6), (3, 4, 1), (7, 4, 3), (7, 8, 0)])
def test_rows_shared_by_workgroups(oracle, n, F, stride, pad):
    coords, offs = _shapes(n, 32, 100 * F + n)
    levels = 1 + int(np.log2(stride))
    lv = hch.hch_build_levels_device(coords, offs, 32, levels)
    olv = oracle.build_hierarchy(coords, offs, 32, levels)
    Li, Lo = olv[0], olv[-1]
    field = torch.full((Lo.Ntot, F ** 3), -7, dtype=torch.int32, device="cuda")
    field_t = torch.full((Li.Ntot, F ** 3), -7, dtype=torch.int32, device="cuda")
    hch.hch_field_build(lv, 0, F, stride, pad, field, field_t)
    want = oracle.field_indices(Li, Lo, F, stride, pad)
    assert np.array_equal(field.cpu().numpy(), want)
    want_t = np.full((Li.Ntot, F ** 3), -1, np.int32)
    o, row = np.nonzero(want >= 0)
    want_t[want[o, row], row] = o
    assert np.array_equal(field_t.cpu().numpy(), want_t)


def test_long_rows_of_few_voxels():
    """7^3 rows of 3000 voxels against 3^3 rows: 13 us against 9.5, both about one launch; with one workgroup
    for all 343 rows of 64 voxels they took 65."""
    coords, offs = _shapes(3000, 64, 1)
    lv = hch.hch_build_levels_device(coords, offs, 64, 1)

    def best(F):
        f, times = torch.empty((3000, F ** 3), dtype=torch.int32, device="cuda"), []
        for _ in range(10):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for _ in range(4):
                hch.hch_field_build(lv, 0, F, 1, (F - 1) // 2, f, None)
            e1.record()
            torch.cuda.synchronize()
            times.append(e0.elapsed_time(e1))
        return min(times)
    assert best(7) < 4 * best(3)
