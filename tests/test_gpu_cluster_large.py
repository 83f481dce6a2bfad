"""The two forms of complete linkage against each other: the rounds of mutually
nearest pairs (an eager call) and one pair at a time (a captured one) at the size
where the rounds are used most, and one pair at a time over every kind of input
on both sides of 3,200 samples, where it changes from one block's loop to two
launches per merge."""
import numpy as np
import pytest
import torch

import oracle
from test_gpu_cluster_rounds import KINDS, _counts

pytestmark = pytest.mark.gpu

pg = pytest.importorskip("paper_1410_4803_amd")


def _captured(dev, m, replays=2):
    out = torch.zeros((m - 1, 16), dtype=torch.uint8, device="cuda")
    ws = torch.empty(pg.cluster_workspace_bytes(m), dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        pg.ibs_cluster(dev[0], dev[1], None, dev[2], out=out, workspace=ws)
    for _ in range(replays):
        out.zero_()
        ws.fill_(255)
        graph.replay()
        torch.cuda.synchronize()
        yield pg.merges_to_numpy(out, m)


def _on_gpu(kind, m):
    """The inputs of _counts, made on the GPU."""
    N = 4096
    i = torch.arange(m, device="cuda", dtype=torch.int32)
    if kind == "random":
        g = torch.Generator(device="cuda").manual_seed(m)
        w = torch.randint(0, 2 * N, (m, m), generator=g, device="cuda", dtype=torch.int32)
    else:                                  # few pairs at a time in a far crowd
        w = 1000 + torch.minimum(i[:, None], i[None]) % 4096
        w[i[:-1].long(), i[1:].long()] = 3 + i[:-1] // 20
    w = torch.triu(w, 1)
    w = w + w.T
    return [(w // 2).contiguous(), (w % 2).contiguous(), torch.full_like(w, N)]


@pytest.mark.parametrize("kind", ["random", "few"])
def test_rounds_equal_one_pair_at_a_time_at_10000(kind):
    m = 10007
    dev = _on_gpu(kind, m)
    got = pg.merges_to_numpy(pg.ibs_cluster(dev[0], dev[1], None, dev[2]), m)
    for ref in _captured(dev, m, replays=1):
        for f in ("a", "b", "height"):
            assert np.array_equal(got[f], ref[f]), f


@pytest.mark.parametrize("m", [333, 3217])
@pytest.mark.parametrize("kind", KINDS)
def test_one_pair_at_a_time(kind, m):
    counts = _counts(kind, m)
    dev = [torch.from_numpy(x.view(np.int32)).cuda() for x in counts]
    if m < 1000:
        ref = oracle.cluster_complete(oracle.ibs_distance(*counts))
    else:
        ref = pg.merges_to_numpy(pg.ibs_cluster(dev[0], dev[1], None, dev[2]), m)
    for got in _captured(dev, m):
        for f in ("a", "b", "height"):
            assert np.array_equal(got[f], ref[f]), f
