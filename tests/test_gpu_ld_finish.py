"""Row offsets and emission of LD records around the sizes where the scan
changes (4 and 4,096 rows, one block's 32,768), and batches whose LD problems
share one scan and one emission launch, with one too long to share the scan."""
import numpy as np
import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu

pg = pytest.importorskip("paper_1410_4803_amd")

from ldcheck import compare_records as _compare


def _ref(n, V, W, r2_min, seed, idx=None):
    bed = synth.mosaic(n, V, founders=6, switch=0.05, miss=0.02, seed=seed)
    codes = oracle.unpack(bed, n, V)
    sel = codes if idx is None else np.ascontiguousarray(codes[:, idx])
    return pg.Cohort.from_numpy(bed, n), oracle.ld_window(sel, W, r2_min)


@pytest.mark.parametrize("V", [2, 3, 5, 63, 4095, 4096, 4097, 32767, 32768, 32769, 70001])
def test_scan_sizes(V):
    c, ref = _ref(24, V, 5, 0.4, V)
    got = pg.ld_records(c, 5, 0.4, path="mfma")
    assert _compare(got, ref, 0.4) == len(ref)


def test_batch_shared_finish():
    spec = [(24, 131073, 3, "mfma", None), (40, 40000, 4, "mfma", None), (33, 65, 64, "popc", None),
            (50, 3, 1, "mfma", None), (70, 500, 70, "mfma", 41), (24, 140000, 2, "popc", None)]
    problems, refs = [], []
    for k, (n, V, W, path, m) in enumerate(spec):
        idx = None if m is None else np.random.default_rng(k).permutation(n)[:m]
        c, ref = _ref(n, V, W, 0.4, 50 + k, idx)
        d_idx = None if idx is None else torch.from_numpy(idx.astype(np.int32)).cuda()
        problems.append(pg.LdProblem(c, window=W, r2_min=0.4, capacity=V * W, path=path,
                                     sample_idx=d_idx))
        refs.append(ref)
    c, ref = _ref(64, 900, 20, 0.4, 90)
    out = torch.zeros(7, 64, dtype=torch.uint8, device="cuda")
    n_out = torch.zeros(1, dtype=torch.int64, device="cuda")
    problems.append(pg.LdProblem(c, window=20, r2_min=0.4, capacity=7, out=out, n_out=n_out))
    batch = pg.Batch(problems[:-1])
    cut = pg.Batch([problems[-1], problems[1]])
    for _ in range(2):
        batch.launch()
        for got, r in zip(batch.results(), refs):
            assert _compare(got, r, 0.4) == len(r)
        cut.launch()
        torch.cuda.synchronize()
        assert int(n_out.item()) == len(ref) > 7
        assert _compare(pg.records_to_numpy(out, 7), ref[:7], 0.4) == 7
