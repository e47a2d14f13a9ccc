"""Tables built by a workgroup each (psh_build_kernel) and by launches over memory (psh_place_kernel), on both sides of the lines
between them: every table is a perfect hash that Eq.1 reads, the sides are those that the sizes fix."""
import numpy as np
import pytest
import torch

import paper_1803_11385_amd as hch

pytestmark = pytest.mark.gpu


def _voxels(u, n, rng):
    q = np.sort(rng.permutation(u ** 3)[:n])
    return np.stack([q // (u * u), q // u % u, q % u], 1).astype(np.int32)


# models' sizes; the side of the largest table
@pytest.mark.parametrize("u, sizes, side", [
    (8, [1], 2), (8, [7], 2), (8, [8, 511], 8),                                # the smallest, and the fullest a side allows
    (64, [12 ** 3 - 1, 100, 5], 12), (64, [13 ** 3 - 1] * 3, 13),
    (64, [32768, 3], 33), (64, [32769, 3], 33),                                # one table most of the work: 32 768 voxels
    (128, [63 ** 3, 63 ** 3 + 5], 64), (128, [64 ** 3 - 1] * 2, 64),           # rows of 64 bits; offset cells beyond LDS
    (128, [64 ** 3, 64 ** 3], 65),                                             # rows beyond 64 bits
    (32, [300 + 7 * k for k in range(300)], 14)])                              # more tables than CUs
def test_tables(u, sizes, side):
    rng = np.random.default_rng(u + len(sizes) + sum(sizes))
    parts = [_voxels(u, n, rng) for n in sizes]
    coords, offs = np.concatenate(parts), np.concatenate([[0], np.cumsum(sizes)])
    levels = 2
    lv = hch.hch_build_levels_device(np.ascontiguousarray(coords), offs, u, levels)
    torch.cuda.synchronize()
    for l in range(levels):
        info = lv.info(l)
        H, T, Phi, V, pos = (f() for f in (info.device_H, info.device_T, info.device_Phi, info.device_V, info.device_coords))
        assert np.array_equal(info.H_host(), H) and np.array_equal(info.T_host(), T) and np.array_equal(info.Phi_host(), Phi)
        assert np.array_equal(info.coords_host(), pos)
        if l == 0:
            assert int(np.max(info.mbar)) == side and np.array_equal(pos, coords)
        for v in range(len(sizes)):
            a, b = int(info.N[v]), int(info.N[v + 1])
            m, r, n = int(info.mbar[v]), int(info.rbar[v]), b - a
            assert m ** 3 > n >= (m - 1) ** 3 and 6 * r ** 3 >= n and np.gcd(r, m) == 1 and info.attempts[v] >= 1
            h, t = H[info.M[v]:info.M[v + 1]], T[info.M[v]:info.M[v + 1]].astype(np.int64)
            phi, p = Phi[info.R[v]:info.R[v + 1]].astype(np.int64), pos[a:b].astype(np.int64)
            s = (p % m + phi[((p[:, 0] % r) * r + p[:, 1] % r) * r + p[:, 2] % r]) % m
            slot = (s[:, 0] * m + s[:, 1]) * m + s[:, 2]
            assert phi.shape[0] == r ** 3 and phi.max(initial=0) < m
            assert np.array_equal(h[slot], np.arange(n)) and np.array_equal(t[slot], p)
            assert int((h >= 0).sum()) == n and np.all(t[h < 0] == 0xFFFF) and np.all(V[info.M[v]:info.M[v + 1]] == v)
