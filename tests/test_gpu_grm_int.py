"""Relationship matrix on the int8 matrix cores: N bit-exact, and A against
the same sums in extended precision, within the bound of the digit split.

Each class factor is rounded once to a multiple of 2^-53 (error at most
2^-54), and enters with x <= 2 or m <= 1: at most 3 * 2^-54 per marker.  The
three or four digit passes and the variant ranges are added in double, each
addition rounding a partial sum of at most D = sum of |x F1| + |m F2|; with at
most 64 ranges that is (4 + 64) roundings of 2^-53 D.  The division rounds
once more.  numpy's extended precision (2^-64) is exact at this scale."""
import numpy as np
import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu

pg = pytest.importorskip("paper_1410_4803_amd")

U = 2.0 ** -53


def _reference(codes):
    """A, N and the bound, from unpacked (variant, sample) codes."""
    L = np.longdouble
    m = codes != 1
    x = np.where(codes > 1, codes - 1, 0) * m
    n, a = 2 * m.sum(1), x.sum(1)
    flip = 2 * a > n
    x = np.where(flip[:, None], 2 * m - x, x)
    a = np.where(flip, n - a, a)
    used = a > 0
    m, x, n, a = m[used], x[used], n[used].astype(L), a[used].astype(L)
    p = (a / n)[:, None]
    w = 1 / (2 * p * (1 - p))
    f1 = np.where(m, w * (x - 2 * p), 0)
    f2 = -2 * p * f1
    S = x.T.astype(L) @ f1 + m.T.astype(L) @ f2
    D = x.T.astype(float) @ np.abs(f1).astype(float) + m.T.astype(float) @ np.abs(f2).astype(float)
    D = np.maximum(D, D.T)
    N = m.T.astype(np.int64) @ m.astype(np.int64)
    with np.errstate(invalid="ignore", divide="ignore"):
        A = S / N
        bound = (3 * U / 2 * N + 68 * U * D) / np.maximum(N, 1) + U * np.abs(A)
    return A, N, bound


def _check(codes, layout, path="auto"):
    V, n = codes.shape
    bed = np.zeros((V, (n + 3) // 4), dtype=np.uint8)
    for k in range(n):
        bed[:, k // 4] |= codes[:, k].astype(np.uint8) << (2 * (k % 4))
    A, N = pg.grm_matrix(pg.Cohort.from_numpy(bed, n), layout=layout, path=path)
    torch.cuda.synchronize()
    A, N = A.cpu().numpy(), N.cpu().numpy().view(np.uint32)
    Ar, Nr, bound = _reference(codes)
    if layout == "full":
        assert np.array_equal(A, A.T, equal_nan=True)
    else:
        i = np.triu_indices(n, 1)
        Ar, Nr, bound = Ar[i], Nr[i], bound[i]
    assert np.array_equal(N, Nr)
    ok = Nr > 0
    assert np.all(np.isnan(A[~ok]))
    err = np.abs(A[ok] - Ar[ok]).astype(float)
    assert np.all(err <= bound[ok].astype(float)), (err / bound[ok].astype(float)).max()


def _hwe(n, V, q, miss, seed):
    return oracle.unpack(synth.hwe(n, V, q, miss, seed=seed), n, V)


# around the 32-sample blocks and 256 x 64 tiles; V around the chunks of 64,
# the operand's 256, and the counters' 128 samples; ranges of few chunks
@pytest.mark.parametrize("layout", ["full", "tri"])
@pytest.mark.parametrize("n,V", [(2, 800), (31, 801), (33, 832), (64, 1023), (65, 1025),
                                 (127, 1088), (129, 2049), (255, 1280), (257, 1500)])
def test_grm_int_edges(n, V, layout):
    _check(_hwe(n, V, (0.01, 0.5), 0.02, n + V), layout)


# 7, 8 and 9 digits of F1: no rare allele, the usual, alleles seen once in 600
@pytest.mark.parametrize("n,q,miss", [(200, (0.42, 0.5), 0.0), (200, (0.02, 0.98), 0.05),
                                      (600, (0.0005, 0.01), 0.0)])
def test_grm_int_digits(n, q, miss):
    codes = _hwe(n, 900, q, miss, 11)
    if n == 600:
        codes[:5] = 0
        codes[:5, 7] = 2                     # one copy among 1,200 alleles
    _check(codes, "full")


def test_grm_int_undefined_and_empty():
    codes = _hwe(90, 1000, (0.05, 0.5), 0.03, 12)
    codes[3], codes[4], codes[5] = 0, 3, 1
    codes[:, 9] = 1
    codes[:, 40] = 1
    _check(codes, "full")


@pytest.mark.parametrize("n,V", [(1537, 3500), (4500, 700)])
def test_grm_int_large_tiles(n, V):
    """512 x 32 tiles: one partial round of split tiles, and whole rounds
    followed by a split one; sampled pairs against the oracle."""
    bed = synth.hwe(n, V, (0.01, 0.5), 0.02, seed=n)
    A, N = pg.grm_matrix(pg.Cohort.from_numpy(bed, n), layout="full")
    torch.cuda.synchronize()
    A, N = A.cpu().numpy(), N.cpu().numpy().view(np.uint32)
    assert np.array_equal(A, A.T) and np.array_equal(N, N.T)
    codes = np.ascontiguousarray(oracle.unpack(bed, n, V).T)
    rng = np.random.default_rng(5)
    pi = np.concatenate([rng.integers(0, n, 3000), np.arange(n), np.full(n, n - 1)])
    pj = np.concatenate([rng.integers(0, n, 3000), np.arange(n), np.arange(n)])
    Ar, Nr, Sr = oracle.grm_pairs(codes, pi, pj)
    assert np.array_equal(N[pi, pj], Nr)
    bound = ((2 * V + 32) * U * Sr + 4 * U * np.abs(Ar) * Nr) / Nr
    assert np.all(np.abs(A[pi, pj] - Ar) <= bound)
