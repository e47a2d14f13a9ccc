"""The row order of few voxels, made by one workgroup per level (pattern_small_kernel): up to its 8192 voxels and beyond."""
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


@pytest.mark.parametrize("n", [1, 63, 64, 65, 1024, 1025, 8191, 8192, 8193])
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
