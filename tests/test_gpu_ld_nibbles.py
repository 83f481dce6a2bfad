"""The nibble operand of the fp4 LD tile: every pair's sums at the edges of its
64-variant groups, 64-sample steps and 2,048-sample (32-word) layout blocks,
with and without a sample list, and on both sides of the cohort size up to which
the fp4 sums are exact (the int8 tile takes more)."""
import numpy as np
import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu

pg = pytest.importorskip("paper_1410_4803_amd")

from ldcheck import compare_records as _compare

MFMA, FORCE = 2, 3 | (1 << 8)


def _codes(V, n, seed):
    """All four codes, 20% missing."""
    r = np.random.default_rng(seed)
    return r.choice(np.array([0, 1, 2, 3], np.uint8), size=(V, n), p=[.3, .2, .2, .3])


def _pack(codes):
    V, n = codes.shape
    p = np.zeros((V, 4 * ((n + 3) // 4)), np.uint8)
    p[:, :n] = codes
    p = p.reshape(V, -1, 4)
    return np.ascontiguousarray(p[:, :, 0] | p[:, :, 1] << 2 | p[:, :, 2] << 4 | p[:, :, 3] << 6)


def _check(codes, W, path, r2_min=0.0, idx=None):
    V, n = codes.shape
    c = pg.Cohort.from_numpy(_pack(codes), n)
    ours = oracle.unpack(_pack(codes), n, V)
    sel = ours if idx is None else np.ascontiguousarray(ours[:, idx])
    d_idx = None if idx is None else torch.from_numpy(idx.astype(np.int32)).cuda()
    ref = oracle.ld_window(sel, W, r2_min)
    out, n_out = pg.ld_window(c, W, r2_min, capacity=V * W, path=path, sample_idx=d_idx)
    return _compare(pg.records_to_numpy(out, int(n_out.item())), ref, r2_min)


@pytest.mark.parametrize("path", [MFMA, FORCE])
@pytest.mark.parametrize("V,n,W", [(2, 64, 1), (63, 63, 62), (64, 65, 40), (65, 255, 64),
                                   (129, 257, 128), (200, 2048, 65), (130, 2049, 129),
                                   (70, 4095, 33)])
def test_nibble_edges(V, n, W, path):
    assert _check(_codes(V, n, V + n), W, path) > 0


@pytest.mark.parametrize("path", [MFMA, FORCE])
@pytest.mark.parametrize("V,n,m", [(65, 300, 64), (129, 2500, 2049)])
def test_nibble_sample_list(V, n, m, path):
    idx = np.random.default_rng(m).permutation(n)[:m]
    assert _check(_codes(V, n, m), 64, path, idx=idx) > 0


@pytest.mark.parametrize("n", [(1 << 24) // 9 - 1, (1 << 24) // 9])
def test_largest_exact_sums(n):
    """Nearly all calls homozygous A2: the largest products throughout."""
    codes = np.full((3, n), 3, np.uint8)
    r = np.random.default_rng(n)
    base = r.random(n) < 0.001
    for v in range(3):
        codes[v, base & (r.random(n) < 0.9)] = v
    for path in (MFMA, FORCE):
        assert _check(codes, 2, path) > 0
