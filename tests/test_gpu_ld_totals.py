"""Allele and missing-call counts that the LD layout takes along: blocks of 512
samples and 64 variants, 1,024 variants a block of the sum, without and with a
sample list.  The pruning drop side (the allele counts) and the correction
path's own records (the totals) both depend on every count."""
import numpy as np
import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu

pg = pytest.importorskip("paper_1410_4803_amd")

from ldcheck import compare_records as _compare

FORCE = 3 | (1 << 8)


@pytest.mark.parametrize("path", ["mfma", FORCE])
@pytest.mark.parametrize("n,V,m", [(511, 63, 0), (512, 64, 0), (513, 65, 0), (3, 1025, 0),
                                   (1030, 1024, 0), (2100, 300, 1025), (600, 129, 37)])
def test_counts(n, V, m, path):
    bed = synth.mosaic(n, V, founders=5, switch=0.03, miss=0.03, seed=n + V)
    codes = oracle.unpack(bed, n, V)
    d_idx = None
    if m:
        idx = np.random.default_rng(m).permutation(n)[:m].astype(np.int32)
        codes = np.ascontiguousarray(codes[:, idx])
        d_idx = torch.from_numpy(idx).cuda()
    c = pg.Cohort.from_numpy(bed, n)
    for W, S, t in [(50, 7, 0.2), (V, 1, 0.05)]:
        W = min(W, V)
        keep, n_kept = pg.ld_prune(c, W, min(S, W), t, sample_idx=d_idx, path=path)
        ref = oracle.ld_prune(codes, W, min(S, W), t)
        assert np.array_equal(keep.cpu().numpy(), ref)
        assert int(n_kept.item()) == int(ref.sum())
    W = min(70, V - 1)
    got = pg.ld_records(c, W, 0.1, sample_idx=d_idx, path=path)
    assert _compare(got, oracle.ld_window(codes, W, 0.1), 0.1) > 0
