"""The nibble operand of LD is laid out only where the window reads it often
enough, and while it is a small part of the card: other calls keep the workspace
of the tiles that work on the 2-bit words alone."""
import ctypes

import pytest

from paper_1410_4803_amd import _native as N

GIB = 1 << 30


def _bytes(n, V, W, path, prune=False):
    g = N.Genotypes(0x1000, n, V, 0, None)
    b = ctypes.c_size_t(0)
    lib = N.load()
    rc = (lib.pg_prune_workspace_bytes(ctypes.byref(g), 0, 0, 0, W, path, ctypes.byref(b))
          if prune else
          lib.pg_ld_workspace_bytes(ctypes.byref(g), 0, 0, 0, W, path, ctypes.byref(b)))
    assert rc == 0
    return b.value


def _words(n, V):
    return -(-V // 64) * 64 * (-(-n // 256) * 16) * 4


@pytest.mark.parametrize("path", [N.PG_PATH_AUTO, N.PG_PATH_MFMA])
def test_a_biobank_chromosome_fits_the_card(path):
    n, V = 487409, 500000
    panel = V * ((n + 3) // 4)
    assert panel + _bytes(n, V, 1000, path) < 256 * GIB
    assert panel + _bytes(n, V, 500, path, prune=True) < 256 * GIB


def test_largest_nibble_operand():
    """32 GiB of nibbles are 16 GiB of words: 131,072 samples x 524,288 variants."""
    n, V = 131072, 524288
    assert _words(n, V) == 16 * GIB
    W = 4000
    assert _bytes(n, V, W, N.PG_PATH_MFMA) > 3 * 16 * GIB
    for n, V in ((131072, 524289), (131073, 524288)):
        assert _bytes(n, V, W, N.PG_PATH_MFMA) < 1.1 * _words(n, V)


@pytest.mark.parametrize("n,V,W,nibbles", [(3000, 400000, 1, True), (3001, 200000, 74, False),
                                           (3001, 200000, 75, True), (20000, 50000, 499, False),
                                           (20000, 50000, 500, True), (20000, 20000, 311, False),
                                           (20000, 20000, 312, True), (20000, 3000, 1, True)])
def test_narrow_windows_over_many_samples(n, V, W, nibbles):
    got = _bytes(n, V, W, N.PG_PATH_MFMA) / _words(n, V)
    assert (got > 3) == nibbles and (nibbles or got < 1.6)


def test_a_batch_shares_the_limit():
    """Three problems of 12 GiB of nibbles each: two get theirs."""
    n, V = 131072, 196608
    lib = N.load()
    sizes = []
    for k in (1, 2, 3):
        probs = (N.Problem * k)()
        for p in probs:
            p.kind = N.PG_KIND_LD
            p.g = N.Genotypes(0x1000, n, V, 0, None)
            p.window, p.r2_min, p.capacity = 4000, 0.5, 16
            p.out = p.n_out = 0x1000
        plan, b = ctypes.c_void_p(), ctypes.c_size_t(0)
        assert lib.pg_batch_plan(probs, k, ctypes.byref(plan)) == 0, N.last_error()
        assert lib.pg_batch_workspace_bytes(plan, ctypes.byref(b)) == 0
        lib.pg_plan_free(plan)
        sizes.append(b.value)
    assert sizes[0] > 18 * GIB
    assert sizes[1] - sizes[0] > 18 * GIB
    assert sizes[2] - sizes[1] < 7 * GIB
