"""IBS calls whose planned tail ranges pay, pay in a smaller number, and do not
pay for parking their sums: each leaves the same counts, equal to the popcount
path's, in the planned workspace."""
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu

pg = pytest.importorskip("paper_1410_4803_amd")


@pytest.mark.parametrize("n,V", [(4100, 1024), (4100, 10000), (4548, 2560), (4548, 1023),
                                 (6000, 5000), (6000, 20000)])
def test_tail_use(n, V):
    c = pg.Cohort.from_numpy(synth.hwe(n, V, (0.05, 0.5), 0.02, seed=n + V), n)
    for layout in ("tri", "full"):
        got = pg.ibs_matrix(c, layout=layout, path="mfma")
        want = pg.ibs_matrix(c, layout=layout, path="popc")
        assert all(torch.equal(g, w) for g, w in zip(got, want))
        del got, want
