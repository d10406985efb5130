"""The mixture on given neighbours over its slice sizes (4096 to 32768 entries a workgroup, a workgroup a row)
against the formula in double precision: rows that end inside a slice, rows off a 16-byte boundary, one and several
neighbours a thread, absent neighbours, and neighbours of several sets."""
import numpy as np
import pytest
import torch

import paper_2405_19325_amd as knn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,V,r", [
    (1, 1, 3), (2, 4095, 1024), (300, 4096, 1000), (3, 4097, 1025), (28, 32001, 64),      # 4096 entries a slice
    (33, 32000, 1024), (40, 32767, 2000),                                                 # 8192
    (100, 32000, 1000), (64, 65533, 2049),                                            # 16384
    (128, 50257, 1024), (120, 65536, 1030),                                               # 32768
    (257, 8193, 64), (130, 40001, 1500), (129, 65537, 4096), (3, 1 << 21, 100),                               # a workgroup a row
])
def test_slices_against_the_oracle(rows, V, r):
    rng = np.random.default_rng(rows * 7 + V + r)
    n = np.array([4200, 4096])
    ko, qo = np.concatenate([[0], np.cumsum(n)]), np.array([0, (rows + 1) // 2, rows])
    of_set = (np.arange(rows) >= qo[1]).astype(np.int64)
    ids = np.stack([rng.permutation(n[s])[:r] for s in of_set]).astype(np.int32)
    ids[:, 1::17] = -1  # absent
    dists = rng.uniform(10, 40, (rows, r)).astype(np.float32)
    vals = np.minimum(rng.zipf(1.3, int(ko[-1])) - 1, V - 1).astype(np.int32)
    vals[::3] = rng.integers(0, V, vals[::3].shape)
    p_lm = rng.random((rows, V), dtype=np.float32)
    p_lm /= p_lm.sum(1, keepdims=True)
    dev = [torch.as_tensor(x, device="cuda") for x in (ids, dists, vals, ko, qo, p_lm)]
    out = knn.mix(*dev, 0.3, 0.4).cpu().numpy()
    mixed, lam = knn.mix_rrc(*dev, 0.3, 0.3, 0.1)
    mixed, lam = mixed.cpu().numpy(), lam.cpu().numpy()
    for b in range(rows):
        w = np.where(ids[b] >= 0, np.exp(-0.3 * (dists[b].astype(np.float64) - dists[b][ids[b] >= 0].min())), 0.0)
        p_knn = np.bincount(vals[ko[of_set[b]] + np.maximum(ids[b], 0)], w / w.sum(), V)
        # sums of at most r fp32 terms of a total of 1: r * 2^-24, and the exponent's argument (up to 9) rounded
        bound = r * 2.0 ** -24 + 9 * 2.0 ** -23
        assert np.abs(out[b] - (0.4 * p_lm[b] + 0.6 * p_knn)).max() <= bound
        there = dists[b][ids[b] >= 0].astype(np.float64)
        want = 1 / (1 + np.exp(-(there.min() / there.max() - 0.3) / 0.1))
        assert abs(lam[b] - want) <= 1e-5
        assert np.abs(mixed[b] - (lam[b] * p_lm[b] + (1 - np.float64(lam[b])) * p_knn)).max() <= bound
