"""Tiles of the correction path without missing calls (128 x 128 variants, one
Gram): edges of groups and tiles, windows that end inside them, panels where
only some groups miss calls, thresholds that every pair reaches, and a cohort
whose sums exceed the 24-bit products of the quick test."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

pg = pytest.importorskip("paper_1410_4803_amd")

from ldcheck import compare_records as _compare

SPARSE, FORCE = 3, 3 | (1 << 8)


def _bed(n, V, seed, missing=()):
    bed = synth.mosaic(n, V, founders=6, switch=0.03, miss=0.0, seed=seed)
    for v, k in missing:   # one missing call: variant v, sample k
        byte = int(bed[v, k // 4])
        bed[v, k // 4] = (byte & (255 ^ 3 << 2 * (k % 4))) | (1 << 2 * (k % 4))
    return bed


def _check(bed, n, V, W, r2_min, path):
    codes = oracle.unpack(bed, n, V)
    got = pg.ld_records(pg.Cohort.from_numpy(bed, n), W, r2_min, path=path)
    ref = oracle.ld_window(codes, W, r2_min)
    return _compare(got, ref, r2_min), len(ref)


@pytest.mark.parametrize("path", [SPARSE, FORCE])
@pytest.mark.parametrize("n,V,W", [(100, 2, 1), (64, 63, 62), (65, 64, 63), (300, 65, 64),
                                   (257, 128, 127), (500, 129, 30), (513, 192, 65),
                                   (90, 193, 192), (1025, 400, 128), (130, 700, 129)])
@pytest.mark.parametrize("r2_min", [-np.inf, 0.0, 0.3])
def test_complete_tiles(n, V, W, r2_min, path):
    got, want = _check(_bed(n, V, n + V), n, V, W, r2_min, path)
    assert got == want and (V == 2 or want > 0)


@pytest.mark.parametrize("missing", [[(0, 0)], [(63, 5), (127, 199)], [(200, 0), (201, 1)],
                                     [(449, 77)]])
def test_mixed_groups(missing):
    n, V, W = 200, 450, 150
    got, want = _check(_bed(n, V, 9, missing), n, V, W, 0.1, FORCE)
    assert got == want > 0


@pytest.mark.parametrize("n", [32767, 32768, 40000])
def test_wide_sums(n):
    got, want = _check(_bed(n, 70, n), n, 70, 69, 0.2, FORCE)
    assert got == want > 0
