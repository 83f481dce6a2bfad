"""The relationship matrix where a marker's increments are small: alleles seen
once or three times, samples that have calls at rare markers only, and markers
all but at p = 1/2 with a sample that is heterozygous throughout.

The int8 path rounds such a marker's class factors to a multiple of 2^-69 or
finer (error at most 2^-70; x <= 2 and m <= 1 bring in at most three of them),
other markers' to 2^-53.  The up to five digit passes and 64 ranges are added in
double, each addition rounding a partial sum of at most D = sum of |x F1| +
|m F2|, and the division rounds once more.  The reference is numpy's extended
precision (2^-64) on a few of the samples, with the frequencies of all."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

pg = pytest.importorskip("paper_1410_4803_amd")

U = 2.0 ** -53


def _bed(x):
    """x: (V, n) minor allele counts, -1 missing."""
    code = np.where(x < 0, 1, np.where(x > 0, x + 1, 0)).astype(np.uint8)
    code = np.pad(code, ((0, 0), (0, -x.shape[1] % 4))).reshape(x.shape[0], -1, 4)
    return np.ascontiguousarray(code[:, :, 0] | code[:, :, 1] << 2 | code[:, :, 2] << 4 |
                                code[:, :, 3] << 6)


def _check(x, some, fine):
    """fine: which markers' factors are held to 2^-69 or finer."""
    V, n = x.shape
    A, N = pg.grm_matrix(pg.Cohort.from_numpy(_bed(x), n), layout="full")
    torch.cuda.synchronize()
    A, N = A.cpu().numpy()[np.ix_(some, some)], N.cpu().numpy()[np.ix_(some, some)]
    L = np.longdouble
    m = x >= 0
    p = np.where(m, x, 0).sum(1).astype(L) / (2 * m.sum(1))
    assert np.all((p > 0) & (p < 1))
    p = p[:, None]
    m = m[:, some]
    x = np.where(m, x[:, some], 0)
    f1 = np.where(m, (x - 2 * p) / (2 * p * (1 - p)), 0)
    f2 = -2 * p * f1
    S = x.T.astype(L) @ f1 + m.T.astype(L) @ f2
    D = x.T.astype(L) @ abs(f1) + m.T.astype(L) @ abs(f2)
    unit = np.where(fine, 2.0 ** -70, 2.0 ** -54)
    r = (2 * m * unit[:, None]).T @ m.astype(float) + (m * unit[:, None]).T @ m.astype(float)
    Nr = m.T.astype(np.int64) @ m.astype(np.int64)
    assert np.array_equal(N, Nr)
    ref = S / Nr
    bound = (r + 69 * U * np.maximum(D, D.T)) / Nr + U * abs(ref)
    err = abs(A - ref)
    assert np.all(err <= bound), (err / bound).max()
    return err


# singletons and markers seen three times; 10 and 8 digits of F1, both tile shapes
@pytest.mark.parametrize("n,V,copies", [(10000, 1000, 1), (10000, 1000, 3), (3000, 900, 1),
                                        (600, 1000, 1), (600, 1000, 2)])
def test_rare_alleles_only(n, V, copies):
    rng = np.random.default_rng(n + copies)
    x = np.zeros((V, n), np.int8)
    for c in range(copies):
        x[np.arange(V), 40 + (rng.integers(0, n - 40, V) + c) % (n - 40)] += 1
    x[0, 3] = 1                                # one of the samples has a copy
    some = np.arange(24)
    err = _check(x, some, np.ones(V, bool))
    # a pair without a copy, V increments of 2p/(1-p): the rounding bound of a
    # double dot product of length V
    i, j = 10, 11
    p = x.sum(1) / (2.0 * n)
    assert err[i, j] <= V * U * (2 * p / (1 - p)).sum() / V


@pytest.mark.parametrize("n,V,rare", [(1000, 1600, 700), (2000, 2049, 64), (2000, 2049, 1)])
def test_rare_alleles_among_common_ones(n, V, rare):
    """Samples 0-9 have calls at the rare markers only, which lie in chunks of
    their own and across the boundaries of chunks."""
    rng = np.random.default_rng(rare)
    x = rng.binomial(2, rng.uniform(0.05, 0.45, (V, 1)), (V, n)).astype(np.int8)
    at = 61 + np.arange(rare) if rare > 1 else np.array([V - 1])
    x[at] = 0
    x[at, rng.integers(20, n, rare)] = 1
    keep = np.zeros(V, bool)
    keep[at] = True
    x[~keep, :10] = -1
    fine = np.zeros(V, bool)
    for c in range(0, V, 64):                  # a chunk's markers are held alike
        fine[c:c + 64] = keep[c:c + 64].any()
    _check(x, np.arange(30), fine)


@pytest.mark.parametrize("n", [800, 4000])
def test_markers_near_one_half(n):
    """p = 1/2 - 1/(2n): a sample that is heterozygous everywhere."""
    rng = np.random.default_rng(n)
    V = 900
    x = np.ones((V, n), np.int8)
    x[:, 20:] = 2 * rng.permuted(np.tile(np.arange(n - 20) % 2, (V, 1)), axis=1)
    x[np.arange(V), 20 + (x[:, 20:] == 2).argmax(1)] = 1
    assert np.all(x.sum(1) == n - 1)
    _check(x, np.arange(40), np.ones(V, bool))
