"""Sample-major layout in its two block shapes: cohorts on both sides of the
line between them (256 blocks of 512 samples x 256 variants), with ragged edges,
rows off the dword grid and masks; IBS counts equal the oracle's."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

pg = pytest.importorskip("paper_1410_4803_amd")


@pytest.mark.parametrize("n,V,masked", [(1, 1, False), (127, 255, True), (129, 257, False),
                                        (513, 4081, True), (60, 65000, False), (60, 65537, True)])
def test_layout_blocks(n, V, masked):
    bed = synth.hwe(n, V, (0.05, 0.5), 0.02, seed=n + V, garbage_pad=True)
    mask = synth.missing_mask(n, V, 0.02, seed=V) if masked else None
    got = pg.ibs_matrix(pg.Cohort.from_numpy(bed, n, mask), layout="full", path="mfma")
    ref = oracle.ibs_matrix(oracle.unpack(bed, n, V, mask), full=True)
    for g, r in zip(got, ref):
        assert np.array_equal(g.cpu().numpy().view(np.uint32).reshape(r.shape), r)
