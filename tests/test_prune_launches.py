"""How many launches the greedy pruning pass enqueues: the rounds that a full
list of pairs may need, fewer for short panels and narrow windows, and none
where the sequential kernel has at most three passes.  The host side alone runs,
against stand-ins of the HIP calls."""
import os

import pytest

import fakehip
from paper_1410_4803_amd import _native

CHILD = r"""
import ctypes, sys
sys.path.insert(0, sys.argv[4])
from paper_1410_4803_amd import _native as N
lib = N.load()
V, W, S = int(sys.argv[1]), int(sys.argv[2]), int(sys.argv[3])
g = N.Genotypes(4096, 300, V, 0, None)
n = ctypes.c_size_t(0)
lib.pg_prune_workspace_bytes(ctypes.byref(g), 0, 0, 0, W, N.PG_PATH_MFMA, ctypes.byref(n))
p = ctypes.c_void_p(4096)
rc = lib.pg_ld_prune(ctypes.byref(g), None, 0, 0, 0, W, S, 0.5, p, p, N.PG_PATH_MFMA, p, n.value,
                     None)
fake = ctypes.CDLL(None)
sys.stdout.flush()
fake.printf(b"rc %d last %d\n", rc, fake.hipGetLastError())
fake.fflush(None)
"""

FIXED = 3            # the LD operand, the allele counts, the pairs
SEQUENTIAL = 3       # drop sides, cell counts, the pass
AROUND = 4           # clear, list, the last pairs, the flags


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    return fakehip.build(tmp_path_factory.mktemp("fake"))


@pytest.mark.parametrize("V,W,S,rounds", [(4000, 50, 5, None), (6600, 50, 5, 14),
                                          (16000, 50, 5, 21), (30000, 50, 5, 26),
                                          (6600, 200, 20, 26), (88025, 700, 70, 26)])
def test_rounds_by_size(fake, V, W, S, rounds):
    root = os.path.dirname(os.path.dirname(os.path.abspath(_native.__file__)))
    calls = fakehip.launches(fake, "", CHILD, V, W, S, root)
    extra = 0 if rounds is None else AROUND + rounds
    assert calls == ["plain"] * (FIXED + SEQUENTIAL + extra)
