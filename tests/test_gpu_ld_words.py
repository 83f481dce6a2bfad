"""LD without the nibble operand (cohorts whose sums do not fit its fp4 form,
1,864,135 samples and more, and narrow windows over many samples): the fp4 tile
on the 2-bit words, the correction path beside it, pruning and batches, over more
than one tile of variants."""
import numpy as np
import pytest
import torch

import oracle
from ldcheck import compare_records

pytestmark = pytest.mark.gpu

pg = pytest.importorskip("paper_1410_4803_amd")

N = (1 << 24) // 9
MFMA, FORCE, POPC = 2, 3 | (1 << 8), "popc"


def _bed(V, n, missing, seed):
    rng = np.random.default_rng(seed)
    code = rng.integers(0, 4 if missing else 3, (V, -(-n // 4), 4), dtype=np.uint8)
    if not missing:
        code += code > 0                       # 0, 2, 3
        code[:, ::97, 1] = 1                   # 0.26% missing, shared
    # neighbours in linkage
    code[1::2, ::3] = code[0::2, ::3][: code[1::2].shape[0]]
    return np.ascontiguousarray(code[:, :, 0] | code[:, :, 1] << 2 | code[:, :, 2] << 4 |
                                code[:, :, 3] << 6)


def _records(cohort, W, r2_min, path, idx=None):
    out, n_out = pg.ld_window(cohort, W, r2_min, capacity=cohort.n_variants * W, path=path,
                              sample_idx=idx)
    return pg.records_to_numpy(out, int(n_out.item()))


@pytest.mark.parametrize("V,W,n", [(2, 1, N), (65, 64, N + 1), (70, 33, N + 255)])
def test_words_against_the_oracle(V, W, n):
    bed = _bed(V, n, True, V)
    got = _records(pg.Cohort.from_numpy(bed, n), W, 0.0, MFMA)
    assert compare_records(got, oracle.ld_window(oracle.unpack(bed, n, V), W, 0.0), 0.0) > 0


@pytest.mark.parametrize("missing", [True, False])
@pytest.mark.parametrize("path", [MFMA, FORCE])
def test_words_against_bit_planes(path, missing):
    V, n = 195, N + 77
    c = pg.Cohort.from_numpy(_bed(V, n, missing, 5), n)
    for W, r2_min in ((194, -np.inf), (100, 0.01)):
        got = _records(c, W, r2_min, path)
        assert len(got) > 0
        assert got.tobytes() == _records(c, W, r2_min, POPC).tobytes()


def test_words_with_a_sample_list():
    V, n = 66, N + 1000
    c = pg.Cohort.from_numpy(_bed(V, n, True, 6), n)
    idx = torch.randperm(n, generator=torch.Generator().manual_seed(1))[:N + 3].to(torch.int32).cuda()
    got = _records(c, 65, 0.0, MFMA, idx)
    assert len(got) > 0 and got.tobytes() == _records(c, 65, 0.0, POPC, idx).tobytes()


def test_words_in_a_batch():
    V, n = 131, N
    c = pg.Cohort.from_numpy(_bed(V, n, True, 7), n)
    small = pg.Cohort.from_numpy(_bed(40, 500, True, 8), 500)
    probs = [pg.LdProblem(c, window=100, r2_min=0.0, capacity=V * 100, path="mfma"),
             pg.LdProblem(small, window=30, r2_min=0.0, capacity=2000, path="mfma")]
    batch = pg.Batch(probs)
    batch.launch()
    torch.cuda.synchronize()
    for p in probs:
        got = pg.records_to_numpy(p.out, int(p.n_out.item()))
        assert len(got) > 0
        assert got.tobytes() == _records(p.cohort, p.window, 0.0, MFMA).tobytes()


@pytest.mark.parametrize("n,V,W", [(3001, 23000, 45), (5003, 14001, 20), (10000, 7000, 1),
                                   (20011, 3500, 130)])
def test_narrow_windows(n, V, W):
    """Operands from 16 MiB on."""
    c = pg.Cohort.from_numpy(_bed(V, n, True, W), n)
    assert pg.ld_workspace_bytes(c, W, path=MFMA) < 1.6 * V * n / 4
    for r2_min in (0.0, 0.05):   # linked neighbours: about 0.1
        got = _records(c, W, r2_min, MFMA)
        assert len(got) > 0 and got.tobytes() == _records(c, W, r2_min, POPC).tobytes()
    idx = torch.randperm(n, generator=torch.Generator().manual_seed(2)).to(torch.int32).cuda()
    got = _records(c, W, 0.0, MFMA, idx)
    assert len(got) > 0 and got.tobytes() == _records(c, W, 0.0, POPC, idx).tobytes()
    keep, n_kept = pg.ld_prune(c, W + 1, max(1, W // 10), 0.05, path="mfma")
    ref, n_ref = pg.ld_prune(c, W + 1, max(1, W // 10), 0.05, path="popc")
    assert torch.equal(keep, ref) and torch.equal(n_kept, n_ref)
