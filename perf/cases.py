"""The work this package is measured by: one pass of each public entry point at
the sizes its users have, from a 500-sample cohort to a biobank chromosome.

A case is a dict of plain values.  Panels are drawn on the GPU from the seed
alone: Hardy-Weinberg panels (independent variants) and founder mosaics
(samples copy segments of a few founders, which gives the linkage and the
relatedness that pruning, clustering and LD queries meet), both with missing
calls at the rate of a cleaned array panel.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1410_4803_amd as pg

DEV = "cuda"


def listed() -> list:
    return [
        # a pilot cohort's pairwise IBS counts: latency and launches count
        dict(name="ibs_small", kind="ibs", panel="hwe", n=500, V=5000, miss=0.01, layout="tri",
             counts="u32", mask=0.0),
        # one request of a server: a sample subset of a resident cohort over a
        # region, 16-bit counts for the copy to the client
        dict(name="ibs_request", kind="request", panel="hwe", n=6011, V=40009, miss=0.01, m=1733,
             begin=1237, length=10121),
        # the IBS matrix of a whole cohort over a chromosome panel
        dict(name="ibs_large", kind="ibs", panel="mosaic", founders=20, n=10000, V=100000,
             miss=0.02, layout="full", counts="u32", mask=0.0),
        # LD of close neighbours in a small cohort, with calls masked by quality control
        dict(name="ld_small", kind="ld", panel="mosaic", founders=20, n=503, V=20011, miss=0.01,
             mask=0.005, window=50, r2_min=0.2),
        # a chromosome's LD windows in a cohort with 1% missing calls
        dict(name="ld_large", kind="ld", panel="mosaic", founders=20, n=5000, V=500000, miss=0.01,
             mask=0.0, window=1000, r2_min=0.2),
        # --indep-pairwise over wide windows of an imputed panel (no missing calls)
        dict(name="prune_large", kind="prune", panel="mosaic", founders=8, n=10000, V=88025,
             miss=0.0, window=700, step=70, r2_max=0.7),
        # the relationship matrix of a pilot cohort and of a whole one, on pruned panels
        dict(name="grm_small", kind="grm", panel="hwe", n=1000, V=76124, miss=0.01,
             layout="full"),
        dict(name="grm_large", kind="grm", panel="mosaic", founders=8, n=10000, V=71307, miss=0.01,
             layout="full"),
        # complete-linkage clustering of the same two cohorts, from their IBS counts
        dict(name="cluster_small", kind="cluster", panel="hwe", n=1000, V=76124, miss=0.01),
        dict(name="cluster_large", kind="cluster", panel="mosaic", founders=8, n=10000, V=71307,
             miss=0.01),
        # the IBD report of a cohort, one line per pair, from its IBS counts
        dict(name="ibd_report", kind="report", panel="mosaic", founders=20, n=10000, V=71307,
             miss=0.01, layout="tri"),
        # a queue of mixed IBS and LD problems over several cohorts, captured once and replayed
        dict(name="batch", kind="batch", count=16, n_min=200, n_max=5000, V_min=2000, V_max=20000,
             miss=0.01, shapes=1003),
    ]


def _log(rng, lo: int, hi: int) -> int:
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng) -> dict:
    kind = rng.choice(["ibs", "request", "ld", "ld", "prune", "grm", "cluster", "report", "batch"])
    panel = dict(panel="hwe") if rng.random() < 0.5 else dict(panel="mosaic",
                                                              founders=rng.choice([8, 10, 20]))
    miss = rng.choice([0.0, 0.002, 0.005, 0.01, 0.02])
    if kind == "ibs":
        V = _log(rng, 1000, 100000)
        return dict(kind=kind, **panel, n=_log(rng, 64, 10000), V=V, miss=miss,
                    layout=rng.choice(["tri", "full"]),
                    counts=rng.choice(["u16", "u32"]) if V < 65536 else "u32",
                    mask=rng.choice([0.0, 0.0, 0.005]))
    if kind == "request":
        n, V = _log(rng, 1000, 12000), _log(rng, 20000, 100000)
        length = rng.randint(1000, 20000)
        return dict(kind=kind, panel="hwe", n=n, V=V, miss=miss, m=rng.randint(100, min(5000, n)),
                    begin=rng.randint(0, V - length), length=length)
    if kind == "ld":
        n, W = _log(rng, 200, 20000), _log(rng, 20, 1000)
        most = min(500000, 5000 * 500000 // n, 5000 * 500000 * 1000 // (n * W))
        return dict(kind=kind, panel="mosaic", founders=rng.choice([8, 10, 20]), n=n,
                    V=_log(rng, 2000, most), miss=miss, mask=rng.choice([0.0, 0.0, 0.005]),
                    window=W, r2_min=0.2)
    if kind == "prune":
        W, S, t = rng.choice([(50, 5, 0.5), (50, 5, 0.2), (200, 20, 0.5), (700, 70, 0.7)])
        return dict(kind=kind, panel="mosaic", founders=rng.choice([8, 10, 20]),
                    n=_log(rng, 500, 10000), V=_log(rng, 5000, 88025), miss=miss, window=W, step=S,
                    r2_max=t)
    if kind == "grm":
        return dict(kind=kind, **panel, n=_log(rng, 100, 10000), V=_log(rng, 1000, 71307),
                    miss=miss, layout=rng.choice(["tri", "full"]))
    if kind == "cluster":
        return dict(kind=kind, **panel, n=_log(rng, 200, 10000), V=_log(rng, 2000, 71307),
                    miss=miss)
    if kind == "report":
        return dict(kind=kind, **panel, n=_log(rng, 200, 10000), V=_log(rng, 2000, 71307),
                    miss=miss, layout=rng.choice(["tri", "full"]))
    return dict(kind=kind, count=rng.randint(4, 16), n_min=200, n_max=5000, V_min=2000,
                V_max=20000, miss=miss, shapes=rng.randint(1, 1 << 20))


# --- panels ------------------------------------------------------------------

def _generator(seed: int) -> torch.Generator:
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _dosage_hwe(g, n, rows):
    """A2 allele counts of `rows` independent variants, A2 frequency 1 - q, q ~ U[0.01, 0.5]."""
    q = 0.01 + 0.49 * torch.rand(rows, 1, generator=g, device=DEV)
    r = torch.rand(rows, n, generator=g, device=DEV)
    return (r >= q * q).to(torch.uint8) + (r >= q * (2 - q)).to(torch.uint8)


class _Mosaic:
    """Haplotypes that copy one of `founders` founders for 100 variants at a
    time (each haplotype with its own offset), with one flip in a thousand."""
    SEG = 100

    def __init__(self, g, n, V, founders):
        self.g, self.F, self.H, self.at = g, founders, 2 * n, 0
        self.offset = torch.randint(self.SEG, (1, self.H), generator=g, device=DEV,
                                    dtype=torch.int32)
        self.copied = torch.randint(founders, (V // self.SEG + 2, self.H), generator=g, device=DEV,
                                    dtype=torch.int32)

    def dosage(self, rows):
        g, F = self.g, self.F
        # every variant is polymorphic among the founders: 1 .. F-1 carriers
        carriers = torch.randint(1, F, (rows, 1), generator=g, device=DEV)
        order = torch.rand(rows, F, generator=g, device=DEV).argsort(1).argsort(1)
        allele = (order < carriers).to(torch.uint8)
        v = torch.arange(self.at, self.at + rows, device=DEV, dtype=torch.int32)[:, None]
        founder = self.copied.gather(0, ((v + self.offset) // self.SEG).long())
        hap = allele.gather(1, founder.long())
        hap ^= (torch.rand(rows, self.H, generator=g, device=DEV) < 0.001).to(torch.uint8)
        self.at += rows
        return hap[:, 0::2] + hap[:, 1::2]


def _codes(case: dict, seed: int):
    """The panel's 2-bit codes in pieces of variants: (rows, n) uint8 tensors."""
    n, V, miss = case["n"], case["V"], case["miss"]
    g = _generator(seed)
    source = _Mosaic(g, n, V, case["founders"]) if case["panel"] == "mosaic" else None
    step = max(64, (1 << 26) // n)
    for v in range(0, V, step):
        rows = min(step, V - v)
        d = source.dosage(rows) if source else _dosage_hwe(g, n, rows)
        code = d + (d > 0).to(torch.uint8)          # 0, 1, 2 A2 alleles -> codes 0, 2, 3
        if miss:
            code[torch.rand(rows, n, generator=g, device=DEV) < miss] = 1
        yield code


def _bed(case: dict, seed: int) -> torch.Tensor:
    n, V = case["n"], case["V"]
    bed = torch.empty(V, (n + 3) // 4, dtype=torch.uint8, device=DEV)
    at = 0
    for code in _codes(case, seed):
        c = torch.nn.functional.pad(code, (0, -n % 4)).view(code.shape[0], -1, 4)
        bed[at:at + code.shape[0]] = c[:, :, 0] | c[:, :, 1] << 2 | c[:, :, 2] << 4 | c[:, :, 3] << 6
        at += code.shape[0]
    return bed


def _mask(case: dict, seed: int):
    """Calls masked by quality control: V rows of ceil(n/64) words."""
    rate = case.get("mask", 0.0)
    if not rate:
        return None
    n, V = case["n"], case["V"]
    g = _generator(seed ^ 0x5bd1e995)
    out = torch.empty(V, (n + 63) // 64, dtype=torch.int64, device=DEV)
    bit = torch.arange(64, device=DEV)
    step = max(64, (1 << 24) // n)
    for v in range(0, V, step):
        rows = min(step, V - v)
        hit = torch.rand(rows, out.shape[1], 64, generator=g, device=DEV) < rate
        out[v:v + rows] = (hit.long() << bit).sum(2)
    return out


def _masked(code, mask, v):
    """The codes with the masked calls of rows v, v+1, ... set to missing."""
    if mask is None:
        return code
    bits = mask[v:v + code.shape[0], :, None] >> torch.arange(64, device=DEV) & 1
    return torch.where(bits.flatten(1)[:, :code.shape[1]].bool(), torch.ones_like(code), code)


def _cohort(case: dict, seed: int) -> pg.Cohort:
    n, V = case["n"], case["V"]
    return pg.Cohort(_bed(case, seed), n, V, (n + 3) // 4, _mask(case, seed))


def _subset(case: dict, seed: int) -> torch.Tensor:
    g = _generator(seed + 1)
    return torch.randperm(case["n"], generator=g, device=DEV)[:case["m"]].sort()[0].to(torch.int32)


def _batch_shapes(case: dict) -> list:
    """Every second problem an IBS triangle, the others LD windows of 500."""
    rng = np.random.Generator(np.random.PCG64(case["shapes"]))
    shapes = []
    for k in range(case["count"]):
        n, V = (int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))
                for a, b in ((case["n_min"], case["n_max"]), (case["V_min"], case["V_max"])))
        shapes.append(dict(kind="ld" if k % 2 else "ibs", panel="mosaic", founders=20, n=n, V=V,
                           miss=case["miss"]))
    return shapes


def _records(rows: int):
    """A record buffer and its count, as a caller that repeats LD queries keeps them."""
    return (torch.zeros(rows, 64, dtype=torch.uint8, device=DEV),
            torch.zeros(1, dtype=torch.int64, device=DEV))


# --- one pass ----------------------------------------------------------------

def prepare(case: dict, seed: int) -> dict:
    kind = case["kind"]
    if kind == "batch":
        problems = []
        for k, s in enumerate(_batch_shapes(case)):
            c = _cohort(s, seed * 1000 + k)
            if s["kind"] == "ibs":
                problems.append(pg.IbsProblem(c, layout="tri"))
            else:
                out, n_out = _records(4 * s["V"])
                problems.append(pg.LdProblem(c, window=500, r2_min=0.2, capacity=4 * s["V"],
                                             out=out, n_out=n_out))
        batch = pg.Batch(problems)
        batch.capture()
        return dict(case=case, batch=batch, problems=problems)
    state = dict(case=case, cohort=_cohort(case, seed))
    if kind == "request":
        state["idx"] = _subset(case, seed)
    elif kind == "ld":
        state["out"], state["n_out"] = _records(max(1024, 4 * case["V"]))
    elif kind in ("cluster", "report"):
        state["counts"] = pg.ibs_matrix(state["cohort"], layout=case.get("layout", "full"))
    return state


def run(state: dict):
    case = state["case"]
    kind = case["kind"]
    if kind == "batch":
        state["batch"].replay()
        return [list(p.out) if isinstance(p, pg.IbsProblem) else [p.out, p.n_out]
                for p in state["problems"]]
    cohort = state["cohort"]
    if kind == "ibs":
        return list(pg.ibs_matrix(cohort, layout=case["layout"], counts=case["counts"]))
    if kind == "request":
        return list(pg.ibs_matrix(cohort, sample_idx=state["idx"],
                                  v_range=(case["begin"], case["begin"] + case["length"]),
                                  layout="tri", counts="u16"))
    if kind == "ld":
        return list(pg.ld_window(cohort, case["window"], case["r2_min"],
                                 capacity=state["out"].shape[0], out=state["out"],
                                 n_out=state["n_out"]))
    if kind == "prune":
        return list(pg.ld_prune(cohort, case["window"], case["step"], case["r2_max"]))
    if kind == "grm":
        return list(pg.grm_matrix(cohort, layout=case["layout"]))
    if kind == "cluster":
        return pg.ibs_cluster(*state["counts"])
    ibs0, ibs1, _, nonmiss = state["counts"]
    return list(pg.ibs_genome(cohort, ibs0, ibs1, nonmiss))


# --- what one pass cannot do without -----------------------------------------

def _entries(m: int, layout: str) -> int:
    return m * m if layout == "full" else m * (m - 1) // 2


def _panel_bytes(case: dict, V: int) -> float:
    words = 8 * ((case["n"] + 63) // 64) if case.get("mask") else 0
    return V * ((case["n"] + 3) // 4 + words)


def work(case: dict) -> dict:
    """Bytes: the panel read once, the results written once.  Operations: a
    multiply-add of each genotype pair in each product that the statistic
    takes: four for the IBS counts, six for the LD sums with missing calls (one
    without), one for the relationship matrix."""
    kind = case["kind"]
    if kind == "batch":
        b = f = 0.0
        for s in _batch_shapes(case):
            w = work({**s, **(dict(window=500) if s["kind"] == "ld" else
                              dict(layout="tri", counts="u32"))})
            b, f = b + w["bytes"], f + w["flops"]
        return dict(bytes=b, flops=f)
    n, V = case["n"], case["V"]
    if kind == "ibs":
        width = 2 if case["counts"] == "u16" else 4
        return dict(bytes=_panel_bytes(case, V) + 4 * width * _entries(n, case["layout"]),
                    flops=8.0 * _entries(n, "tri") * V)
    if kind == "request":
        m, L = case["m"], case["length"]
        return dict(bytes=L * ((m + 3) // 4) + 4 * m + 8.0 * _entries(m, "tri"),
                    flops=8.0 * _entries(m, "tri") * L)
    if kind in ("ld", "prune"):
        W = min(case["window"] if kind == "ld" else case["window"] - 1, V - 1)
        pairs = W * V - W * (W + 1) // 2
        ops = 12.0 if case["miss"] or case.get("mask") else 2.0
        return dict(bytes=_panel_bytes(case, V) + V, flops=ops * pairs * n)
    if kind == "grm":
        return dict(bytes=_panel_bytes(case, V) + 12.0 * _entries(n, case["layout"]),
                    flops=2.0 * n * (n + 1) / 2 * V)
    if kind == "cluster":
        # the counts once, the distances once, one comparison of each distance
        return dict(bytes=12.0 * n * n + 8.0 * n * n, flops=3.0 * n * n)
    e = _entries(n, case["layout"])
    return dict(bytes=_panel_bytes(case, V) + 44.0 * e, flops=20.0 * e)


# --- the same results in 64 bits ---------------------------------------------

def _features(case: dict, seed: int):
    """(first variant, calls as float64 dosages, presence) per piece of the panel."""
    mask, v = _mask(case, seed), 0
    for code in _codes(case, seed):
        code = _masked(code, mask, v)
        v += code.shape[0]
        there = code != 1
        yield torch.where(code > 1, code - 1, torch.zeros_like(code)).double(), there


def _layout(x: torch.Tensor, layout: str) -> torch.Tensor:
    if layout == "full":
        return x
    i = torch.arange(x.shape[0], device=x.device)
    return x[i[:, None] < i[None, :]]


def exact(case: dict, seed: int):
    """The relationship matrix by a float64 product of standardised dosages,
    and the IBD report from float64 moments.  The other kinds return whole
    numbers and records."""
    if case["kind"] == "grm":
        n = case["n"]
        S = torch.zeros(n, n, dtype=torch.float64, device=DEV)
        N = torch.zeros(n, n, dtype=torch.float64, device=DEV)
        for x, there in _features(case, seed):
            for x, there in zip(x.split(8192), there.split(8192)):
                p = x.sum(1, keepdim=True) / (2.0 * there.sum(1, keepdim=True))
                used = (p > 0) & (p < 1)
                z = torch.where(there & used, (x - 2 * p) / (2 * p * (1 - p)).sqrt(), 0.0)
                S.addmm_(z.t().contiguous(), z)
                t = (there & used).float()
                N += (t.t().contiguous() @ t).double()
        return [_layout(S / N, case["layout"]), None]
    if case["kind"] == "report":
        n = case["n"]
        sums, count = torch.zeros(3, dtype=torch.float64, device=DEV), 0
        ibs0, ibs1, nonmiss = (torch.zeros(n, n, dtype=torch.float64, device=DEV)
                               for _ in range(3))
        for x, there in _features(case, seed):
            # counts below 2^24 are exact in a float32 product of 0 and 1
            m, het, a2 = (f.float().t().contiguous() for f in (there, x == 1, x == 2))
            a1 = m - het - a2
            nonmiss += (m @ m.t()).double()
            ibs1 += (het @ (a1 + a2).t()).double()
            ibs0 += (a1 @ a2.t()).double()
            t = 2.0 * there.sum(1).double()
            x = x.sum(1)
            ok = t >= 4
            x, t = x[ok], t[ok]
            y = t - x
            four, three = t * (t - 1) * (t - 2) * (t - 3), t * (t - 1) * (t - 2)
            e00 = 2 * x * (x - 1) * y * (y - 1) / four
            e10 = 4 * (x * (x - 1) * (x - 2) * y + x * y * (y - 1) * (y - 2)) / four
            e11 = 2 * (x * (x - 1) * y + x * y * (y - 1)) / three
            sums += torch.stack([e00.sum(), e10.sum(), e11.sum()])
            count += int(ok.sum())
        e00, e10, e11 = (sums / count).tolist()
        ibs0, ibs1, nonmiss = (_layout(t, case["layout"])
                               for t in (ibs0 + ibs0.t(), ibs1 + ibs1.t(), nonmiss))
        z0 = (ibs0 / nonmiss / e00).clamp(max=1.0)
        z1 = ((ibs1 / nonmiss - z0 * e10) / e11).clamp(min=0.0).minimum(1 - z0)
        z2 = 1 - z0 - z1
        return [z0, z1, z2, z1 / 2 + z2]
    return None
