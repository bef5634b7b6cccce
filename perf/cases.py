"""What the performance of this framework is measured on: the work its users have it do.

A program that uses the framework keeps an index over a coded database (codebooks and one-byte
sub-codes), receives batches of queries and calls `icq_search`; one that follows the paper's
threshold policy step by step uses the staged calls or `icq_search_running`; one that builds a
database from vectors encodes them.  Sizes are those of this repository's workloads (a tiny set,
10^6 items at d = 128 and d = 960, 10^7 clustered items, 10^8 items) and, for the drawn cases,
the ranges between and around them with odd sizes, odd dimensions and short codebooks.

Inputs are drawn on the GPU from the seed: codebooks N(0, sigma_k^2) with sigma_k = ratio^k,
uniform (or cluster-wise repeated) sub-codes, queries = reconstruction of a random item plus 5 %
noise, thresholds = a sampled quantile of the crude distance, as the repository's workloads have it.
"""
import math

import torch

from paper_1912_08756_amd import binding as icq


def listed():
    return [
        # the tiny workload: a small database behind an interactive service, one hundred queries; launches count
        dict(name="search_tiny", kind="search", N=10_000, Q=100, d=32, K=4, Kf=1, m=256, topk=10, ratio=0.5, keep=0.004, codes="uniform"),
        # one user's query on a database of a million items: latency
        dict(name="search_single", kind="search", N=1_000_000, Q=1, d=128, K=8, Kf=2, m=256, topk=100, ratio=0.5, keep=0.01, codes="uniform"),
        # evaluation or batch retrieval: ten thousand queries at once, 64-bit codes
        dict(name="search_bulk", kind="search", N=1_000_000, Q=10_000, d=128, K=8, Kf=2, m=256, topk=100, ratio=0.5, keep=0.01, codes="uniform"),
        # image descriptors of 960 dimensions, 128-bit codes: the tables weigh as much as the search
        dict(name="search_wide", kind="search", N=1_000_000, Q=1_000, d=960, K=16, Kf=4, m=256, topk=100, ratio=0.8, keep=0.01, codes="uniform"),
        # data in clusters (bursts of survivors, ties), a service's batch of 256 queries
        dict(name="search_clustered", kind="search", N=10_000_000, Q=256, d=96, K=8, Kf=2, m=256, topk=100, ratio=0.5, keep=0.01, codes="clustered"),
        # the largest database, a batch of 128 queries: the headline workload's call
        dict(name="search_large", kind="search", N=100_000_000, Q=128, d=96, K=16, Kf=4, m=256, topk=100, ratio=0.8, keep=0.01, codes="uniform"),
        # the same database, one query by itself
        dict(name="search_large_single", kind="search", N=100_000_000, Q=1, d=96, K=16, Kf=4, m=256, topk=100, ratio=0.8, keep=0.01, codes="uniform"),
        # nothing is a round number: dimension, codebooks, codewords, items, queries, result length
        dict(name="search_ragged", kind="search", N=777_777, Q=37, d=99, K=11, Kf=3, m=200, topk=47, ratio=0.7, keep=0.01, codes="uniform"),
        # the paper's policy through the staged calls: tables, thresholds from the first items, both stages, operation counts
        dict(name="staged_policy", kind="staged", N=250_001, Q=199, d=100, K=8, Kf=2, m=256, topk=20, ratio=0.5, keep=0.0, codes="uniform"),
        # the paper's running threshold refreshed per tile, tiles growing fourfold
        dict(name="running_tiles", kind="running", N=10_000_000, Q=128, d=96, K=16, Kf=4, m=256, topk=100, ratio=0.8, keep=0.0, codes="uniform"),
        # a million vectors encoded into 64-bit codes
        dict(name="encode", kind="encode", N=1_000_000, d=128, K=8, m=256, ratio=0.5, sweeps=0),
        # an odd number of vectors into 128-bit codes, refined by two sweeps
        dict(name="encode_refined", kind="encode", N=262_147, d=96, K=16, m=256, ratio=0.8, sweeps=2),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: the kinds above, sizes spread over the ranges between the repository's workloads."""
    m = 256 if rng.random() < 0.7 else rng.randint(64, 255)
    what = rng.choice(["tiny", "bulk", "bulk", "clustered", "wide", "large", "large", "staged", "running", "encode", "encode"])
    if what == "encode":
        K, d, sweeps = rng.choice([4, 7, 8, 16]), _log(rng, 24, 960), rng.choice([0, 0, 1, 2])
        most = min(1_000_000, 4.0e11 / (2.0 * K * 256 * d * (1 + sweeps)))
        return dict(kind="encode", N=_log(rng, 1000, max(2000, most)), d=d, K=K, m=m, ratio=rng.choice([0.5, 0.7, 0.8]), sweeps=sweeps)
    c = dict(kind="search", m=m, keep=0.01, codes="uniform", topk=rng.choice([10, 20, 50, 100, 100, rng.randint(1, 200)]))
    if what == "tiny":
        c.update(N=_log(rng, 2_000, 100_000), Q=_log(rng, 1, 1000), d=_log(rng, 16, 128), K=4, Kf=1, ratio=0.5)
    elif what == "bulk":
        c.update(N=_log(rng, 100_000, 4_000_000), K=rng.choice([6, 8, 8, 12]), Kf=2, d=_log(rng, 32, 256), ratio=0.5)
        c.update(Q=_log(rng, 1, min(10_000, 1.0e10 / c["N"])))
    elif what == "clustered":
        c.update(N=_log(rng, 1_000_000, 20_000_000), K=8, Kf=2, d=_log(rng, 32, 256), ratio=0.5, codes="clustered")
        c.update(Q=_log(rng, 1, min(1_000, 4.0e9 / c["N"])))
    elif what == "wide":
        c.update(N=_log(rng, 100_000, 4_000_000), K=16, Kf=rng.choice([3, 4, 4]), d=_log(rng, 128, 960), ratio=0.8)
        c.update(Q=_log(rng, 1, min(1_000, 1.0e9 / c["N"])))
    elif what == "large":
        c.update(N=_log(rng, 4_000_000, 100_000_000), K=rng.choice([12, 16, 16]), Kf=rng.choice([3, 4, 4]), d=_log(rng, 32, 256), ratio=0.8)
        c.update(Q=_log(rng, 1, min(256, 1.2e10 / c["N"])))
    elif what == "staged":
        c.update(kind="staged", keep=0.0, N=_log(rng, 20_000, 1_000_000), K=rng.choice([4, 8, 8]), Kf=2, d=_log(rng, 32, 256), ratio=0.5)
        c.update(Q=_log(rng, 1, min(1_000, 1.0e8 / c["N"])), topk=min(c["topk"], 100))
    else:
        c.update(kind="running", keep=0.0, N=_log(rng, 200_000, 20_000_000), K=rng.choice([12, 16]), Kf=rng.choice([3, 4]), d=_log(rng, 32, 256), ratio=0.8)
        c.update(Q=_log(rng, 1, 256))
    return c


# ---- inputs

def _codebooks(c, g):
    cb = torch.randn((c["K"], c["m"], c["d"]), device="cuda", generator=g)
    s = torch.tensor([c["ratio"] ** k for k in range(c["K"])], device="cuda")
    return cb.mul_(s[:, None, None])


def _codes(c, g):
    K, N, m = c["K"], c["N"], c["m"]
    codes = torch.randint(0, m, (K, N), dtype=torch.uint8, device="cuda", generator=g)
    if c["codes"] == "clustered":       # an item keeps its cluster's fast sub-codes with probability 0.9
        centres = torch.randint(0, m, (c["Kf"], 1000), dtype=torch.uint8, device="cuda", generator=g)
        pick = torch.randint(0, 1000, (N,), device="cuda", generator=g)
        for k in range(c["Kf"]):
            keep = torch.rand((N,), device="cuda", generator=g) < 0.9
            codes[k] = torch.where(keep, centres[k][pick], codes[k])
    return codes


def _queries(c, cb, codes, g):
    src = torch.randint(0, c["N"], (c["Q"],), device="cuda", generator=g)
    x = torch.zeros((c["Q"], c["d"]), device="cuda")
    for k in range(c["K"]):
        x += cb[k][codes[k, src].long()]
    rms = math.sqrt(sum(c["ratio"] ** (2 * k) for k in range(c["K"])) * c["d"])
    x += (0.05 * rms / math.sqrt(c["d"])) * torch.randn(x.shape, device="cuda", generator=g)
    return x.contiguous()


def _thresholds(c, cb, codes, queries, g):
    """The `keep` quantile of the crude distance over a sample of the items, per query."""
    n = min(c["N"], 16384 if c["Q"] <= 1024 else 4096)
    at = torch.randint(0, c["N"], (n,), device="cuda", generator=g)
    kth = max(1, math.ceil(c["keep"] * n))
    out = []
    for q in queries.split(512):
        P = torch.zeros((q.shape[0], n), device="cuda")
        for k in range(c["Kf"]):
            t = (q * q).sum(1, keepdim=True) - 2.0 * (q @ cb[k].T) + (cb[k] * cb[k]).sum(1)
            P += t.index_select(1, codes[k, at].long())
        out.append(torch.kthvalue(P, kth, dim=1).values)
    return torch.cat(out).contiguous()


def _empty(shape, dtype):
    return torch.zeros(shape, dtype=dtype, device="cuda")


def prepare(case, seed):
    c = case
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    cb = _codebooks(c, g)
    s = {"kind": c["kind"]}
    if c["kind"] == "encode":
        # vectors of a Gaussian mixture: 1000 centres (reconstructions), within-cluster deviation of the middle codebooks
        K, N, d = c["K"], c["N"], c["d"]
        centres = torch.zeros((1000, d), device="cuda")
        for k in range(K):
            centres += cb[k][torch.randint(0, c["m"], (1000,), device="cuda", generator=g)]
        x = torch.randn((N, d), device="cuda", generator=g).mul_(c["ratio"] ** (K // 4))
        x += centres[torch.randint(0, 1000, (N,), device="cuda", generator=g)]
        index = icq.icq_index_create(cb, _empty((K, 0), torch.uint8), 1)
        s.update(index=index, x=x, codes=_empty((K, N), torch.uint8), sweeps=c["sweeps"],
                 ws=_empty((icq.icq_encode_workspace_bytes(index, N),), torch.uint8))
        return s

    Q, K, N, topk = c["Q"], c["K"], c["N"], c["topk"]
    codes = _codes(c, g)
    queries = _queries(c, cb, codes, g)
    s.update(queries=queries, topk=topk, ids=_empty((Q, topk), torch.int32), dist=_empty((Q, topk), torch.float32),
             count=_empty((Q,), torch.int32))
    if c["kind"] == "running":
        bases, size, at = [], 8192, 0
        while at < N:
            bases.append(at)
            at, size = at + size, size * 4
        if len(bases) > 1 and N - bases[-1] < 8192:      # a last sliver joins the tile before it
            bases.pop()
        ends = bases[1:] + [N]
        tiles = [icq.icq_index_create(cb, codes[:, a:b].contiguous(), c["Kf"]) for a, b in zip(bases, ends)]
        cap = N // 8 + 32768
        s.update(tiles=tiles, bases=bases, cap=cap, sigma=_sigma(c),
                 ws=torch.empty(icq.icq_running_workspace_bytes(tiles, Q, cap, topk), dtype=torch.uint8, device="cuda"))
        return s
    index = icq.icq_index_create(cb, codes, c["Kf"])
    if c["kind"] == "staged":
        cap = N                                          # a list never overflows
        s.update(index=index, sigma=_sigma(c), sample=4096, lut=_empty((Q, K, 256), torch.float32), thr=_empty((Q,), torch.float32),
                 cand_ids=_empty((Q, cap), torch.int32), cand_part=_empty((Q, cap), torch.float32),
                 ops=_empty((Q,), torch.int64), summary=_empty((4,), torch.float64))
    else:
        cap = min(N, max(4096, N // 20))
        s.update(index=index, cap=cap, thr=_thresholds(c, cb, codes, queries, g))
    s["ws"] = torch.empty(icq.icq_workspace_bytes(index, Q, cap, topk), dtype=torch.uint8, device="cuda")
    return s


def _sigma(c):
    """The margin of the paper's policy: the variance the slow codebooks cover."""
    v = c["d"] * sum(c["ratio"] ** (2 * k) for k in range(c["Kf"], c["K"]))
    return torch.full((c["Q"],), v, dtype=torch.float32, device="cuda")


# ---- one pass

def run(s):
    if s["kind"] == "search":
        icq.icq_search(s["index"], s["queries"], s["thr"], s["cap"], s["topk"], s["ids"], s["dist"], s["count"], s["ws"])
        return {"ids": s["ids"], "dist": s["dist"], "survivors": s["count"]}
    if s["kind"] == "staged":
        # the candidate lists themselves come in no particular order; what is read from them is returned
        icq.icq_build_lut(s["index"], s["queries"], s["lut"])
        icq.icq_sample_thresholds(s["index"], s["lut"], s["sigma"], s["topk"], s["sample"], s["thr"])
        icq.icq_scan_fast(s["index"], s["lut"], s["thr"], s["cand_ids"], s["cand_part"], s["count"], s["ws"])
        icq.icq_refine(s["index"], s["lut"], s["cand_ids"], s["cand_part"], s["count"], s["topk"], s["ids"], s["dist"], s["ws"])
        icq.icq_op_counts(s["index"], s["count"], s["ops"], s["summary"])
        return {"lut": s["lut"], "thresholds": s["thr"], "ids": s["ids"], "dist": s["dist"], "survivors": s["count"],
                "ops": s["ops"], "summary": s["summary"]}
    if s["kind"] == "running":
        icq.icq_search_running(s["tiles"], s["bases"], s["queries"], s["sigma"], s["cap"], s["topk"], s["ids"], s["dist"],
                               s["count"], s["ws"])
        return {"ids": s["ids"], "dist": s["dist"], "refined": s["count"]}
    icq.icq_encode(s["index"], s["x"], s["codes"], s["ws"])
    if s["sweeps"]:
        icq.icq_encode_refine(s["index"], s["x"], s["codes"], s["sweeps"], None, s["ws"])
    return {"codes": s["codes"]}


# ---- what a pass cannot do without

def work(case):
    c = case
    K, m, d, N = c["K"], c["m"], c["d"], c["N"]
    tables = 4.0 * K * m * d                             # the codebooks
    if c["kind"] == "encode":
        return {"bytes": tables + 4.0 * N * d + float(N) * K, "flops": 2.0 * N * K * m * d * (1 + c["sweeps"])}
    Q, Kf, topk = c["Q"], c["Kf"], c["topk"]
    out = 8.0 * Q * topk + 4.0 * Q
    flops = 2.0 * Q * K * m * d
    # crude distances: one per item and query, or one per tuple of fast sub-codes where items share it
    crude = min(float(N), 256.0 ** Kf)
    share = {"search": c["keep"], "staged": 0.06, "running": 0.004}[c["kind"]]
    refined = share * Q * N
    read = 4.0 * Q * d + tables + (float(Kf) * N if Kf > 2 else 0.0) + min(float(N), refined) * K
    if c["kind"] == "staged":
        out += 4.0 * Q * K * 256 + 8.0 * refined         # the tables and the candidate lists are outputs of their calls
    return {"bytes": read + out, "flops": flops + Q * crude * Kf + refined * (K - Kf)}


def tolerance(case):
    if case["kind"] == "encode":
        return {"rel": 0.0, "differ": 1e-3}              # sub-codes: near ties of 32-bit scores, and what follows from them
    # distances are sums of K 32-bit terms; ids may differ where two distances tie within that
    return {"rel": 1e-5, "max": 2e-4, "differ": 2e-3}
