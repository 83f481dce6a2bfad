"""The greedy pruning pass in rounds: chains of pairs that wait for each
other (one pair decided per round), short enough for the one block that
finishes and too long for it (the sequential kernels take over), lists that
overflow, and list sizes around what the last block holds; flags equal the
oracle's bit for bit."""
import numpy as np
import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu

pg = pytest.importorskip("paper_1410_4803_amd")


def _check(bed, n, V, W, S, t):
    codes = oracle.unpack(bed, n, V)
    ref = oracle.ld_prune(codes, W, S, t)
    c = pg.Cohort.from_numpy(bed, n)
    for _ in range(2):
        keep, n_kept = pg.ld_prune(c, W, S, t)
        torch.cuda.synchronize()
        got = keep.cpu().numpy()
        assert np.array_equal(got, ref)
        assert int(n_kept.item()) == int(ref.sum())
    return ref


def _chain(n, V, shift, width):
    """Variant i heterozygous on a circular block of samples that moves by
    `shift`: equal allele frequencies, r2 above 0.4 for neighbours (and
    variants a whole turn apart)."""
    codes = np.zeros((V, n), dtype=np.uint8)
    k = np.arange(width)
    for v in range(V):
        codes[v, (v * shift + k) % n] = 2
    bed = np.zeros((V, (n + 3) // 4), dtype=np.uint8)
    for s in range(n):
        bed[:, s // 4] |= codes[:, s] << (2 * (s % 4))
    return bed


@pytest.mark.parametrize("V,W,S", [(3000, 60, 5), (8193, 100, 10), (12000, 60, 60)])
def test_prune_rounds_chain(V, W, S):
    n = 400
    ref = _check(_chain(n, V, 5, 20), n, V, W, S, 0.4)
    assert 0 < ref.sum() < V


def test_prune_rounds_short_chains():
    """300 chains of 40 pairs: about 40 rounds, 12,000 pairs, the last 8,192
    of them in one block."""
    n, runs, length = 400, 300, 41
    one = _chain(n, length, 5, 20)
    gap = synth.hwe(n, 60, (0.3, 0.5), 0.0, seed=9)
    bed = np.concatenate([np.concatenate([one, gap]) for _ in range(runs)])
    _check(bed, n, bed.shape[0], 60, 20, 0.4)


@pytest.mark.parametrize("V,F,t", [(2000, 4, 0.05), (20000, 3, 0.05), (20000, 8, 0.2)])
def test_prune_rounds_dense(V, F, t):
    n = 120
    bed = synth.mosaic(n, V, F, 0.01, 0.001, 0.0, 0.0, seed=V + F)
    _check(bed, n, V, 50, 5, t)


@pytest.mark.parametrize("W,S", [(2, 1), (17, 4), (18, 18), (64, 1), (1025, 33)])
def test_prune_rounds_windows(W, S):
    n, V = 90, 9000
    bed = synth.mosaic(n, V, 6, 0.02, 0.001, 0.0, 0.02, seed=W)
    _check(bed, n, V, W, S, 0.3)


def test_prune_rounds_capture():
    """The launches are plain kernel nodes: three replays of a captured call,
    with other work between them, give the eager flags."""
    n, V = 200, 12000
    bed = synth.mosaic(n, V, 8, 0.01, 0.001, 0.0, 0.0, seed=5)
    c = pg.Cohort.from_numpy(bed, n)
    ref, n_ref = pg.ld_prune(c, 50, 5, 0.3)
    ws = torch.empty(pg.prune_workspace_bytes(c, 50), dtype=torch.uint8, device="cuda")
    keep, n_kept = torch.zeros_like(ref), torch.zeros_like(n_ref)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        pg.ld_prune(c, 50, 5, 0.3, keep=keep, n_kept=n_kept, workspace=ws)
    for _ in range(3):
        keep.zero_()
        ws.fill_(255)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(keep, ref) and torch.equal(n_kept, n_ref)
