"""GPU parity: the HIP path (through the C ABI) against the CPU oracle, element
by element on the same seeded inputs.  Bar: candidate lists equal as sets except
entries whose crude distance lies within 1e-4*(|t|+1) of the threshold; distances
within 1e-4*(|d|+1); top-k sets equal except at ties within that tolerance;
storage round trip bit-exact."""
import numpy as np
import pytest

from helpers import check_candidates, check_topk, thresholds_kth, thresholds_quantile, tiled_loop_analysis, tol
from oracle import icq_oracle as orc
from paper_1912_08756_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    from paper_1912_08756_amd import binding
    assert torch.cuda.is_available(), "these tests need the MI355X"
    binding.load()
    return torch, binding


def _dev(torch, a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _u32(t):
    return t.cpu().numpy().view(np.uint32)


class Gpu:
    """Thin test driver around the binding for one workload."""

    def __init__(self, gpu, cfg, mode=0):
        self.torch, self.b = gpu
        torch = self.torch
        self.cfg = cfg
        self.cb = _dev(torch, cfg["codebooks"])
        self.codes = _dev(torch, cfg["codes"])
        self.queries = _dev(torch, cfg["queries"])
        self.index = self.b.icq_index_create(self.cb, self.codes, cfg["Kf"])
        self.b.icq_index_set_scan_mode(self.index, mode)    # 0 auto, 1 streamed, 2 grouped
        self.K, self.Q, self.N = cfg["K"], cfg["queries"].shape[0], cfg["codes"].shape[1]

    def workspace(self, Q, cap, topk, nbytes=None):
        n = self.b.icq_workspace_bytes(self.index, Q, cap, topk) if nbytes is None else nbytes
        return self.torch.empty(n, dtype=self.torch.uint8, device="cuda")

    def lut(self):
        torch = self.torch
        lut = torch.empty((self.Q, self.K, 256), dtype=torch.float32, device="cuda")
        self.b.icq_build_lut(self.index, self.queries, lut)
        return lut

    def scan(self, lut, thr, cap, want_partial=True):
        torch = self.torch
        Q = lut.shape[0]
        ids = torch.full((Q, cap), -1, dtype=torch.int32, device="cuda")
        part = torch.full((Q, cap), float("nan"), dtype=torch.float32, device="cuda") if want_partial else None
        cnt = torch.full((Q,), 12345, dtype=torch.int32, device="cuda")
        ws = self.workspace(Q, cap, 1)
        self.b.icq_scan_fast(self.index, lut, _dev(torch, thr), ids, part, cnt, ws)
        torch.cuda.synchronize()
        return ids, part, cnt

    def refine(self, lut, ids, part, cnt, topk):   # part may be None: full K-term sum
        torch = self.torch
        Q, cap = ids.shape
        out_ids = torch.empty((Q, topk), dtype=torch.int32, device="cuda")
        out_dist = torch.empty((Q, topk), dtype=torch.float32, device="cuda")
        ws = self.workspace(Q, cap, topk)
        self.b.icq_refine(self.index, lut, ids, part, cnt, topk, out_ids, out_dist, ws)
        torch.cuda.synchronize()
        return _u32(out_ids), out_dist.cpu().numpy()

    def search(self, thr, cap, topk, ws_bytes=None, queries=None):
        torch = self.torch
        qs = self.queries if queries is None else queries
        Q = qs.shape[0]
        out_ids = torch.empty((Q, topk), dtype=torch.int32, device="cuda")
        out_dist = torch.empty((Q, topk), dtype=torch.float32, device="cuda")
        surv = torch.empty((Q,), dtype=torch.int32, device="cuda")
        ws = self.workspace(Q, cap, topk, ws_bytes)
        self.b.icq_search(self.index, qs, _dev(torch, thr), cap, topk, out_ids, out_dist, surv, ws)
        torch.cuda.synchronize()
        return _u32(out_ids), out_dist.cpu().numpy(), _u32(surv)


def oracle_all(cfg, topk=None):
    """Oracle tables, crude distances and full distances of EVERY item (exhaustive
    sums), so that band cases can be judged whatever the GPU decided."""
    T = orc.lut(cfg["codebooks"], cfg["queries"])
    P = orc.partial(T, cfg["codes"], cfg["Kf"])
    _, _, D = orc.adc_exhaustive(T, cfg["codes"], 1, want_all=True)
    return T, P, D


def small(name, N, Q, **kw):
    return synth.make(name, N=N, Q=Q, **kw)


# ------------------------------------------------------------------ storage layout
@pytest.mark.parametrize("K,Kf,N", [(4, 1, 10_007), (8, 2, 4096), (16, 4, 70_001), (3, 3, 513),
                                      (7, 2, 1), (20, 4, 9_999)])
def test_storage_round_trip_is_bit_exact(gpu, K, Kf, N):
    torch, b = gpu
    cfg = synth.make("C0", N=N, Q=1, K=K, Kf=Kf, sigma=("geom", 0.7))
    g = Gpu(gpu, cfg)
    for from_items in (0, 1, 2) if Kf <= 4 else (0, 1):      # 2: the layout grouped by fast sub-codes
        out = torch.zeros((K, N), dtype=torch.uint8, device="cuda")
        b.icq_index_export_codes(g.index, from_items, out)
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy(), cfg["codes"])


# ------------------------------------------------------------------ lookup tables
@pytest.mark.parametrize("name,Q,over", [
    ("C0", 100, {}), ("C1", 130, {}), ("C2", 70, {}), ("C3", 65, {}),
    ("C0", 5, dict(d=7)), ("C0", 64, dict(d=33, m=100)), ("C1", 1, dict(d=200, K=3, Kf=1, sigma=("geom", 0.5))),
    # more than four blocks per compute unit: the kernel form without read-ahead, with and without 16-byte query loads
    ("C1", 4100, {}), ("C0", 8200, dict(d=33))])
def test_build_lut_matches_oracle(gpu, name, Q, over):
    cfg = synth.make(name, N=1000, Q=Q, **over)
    g = Gpu(gpu, cfg)
    lut = g.lut().cpu().numpy().astype(np.float64)
    T = orc.lut(cfg["codebooks"], cfg["queries"])
    m = cfg["m"]
    err = np.abs(lut[:, :, :m] - T)
    assert (err <= tol(T)).all(), "table entry off by %g" % err.max()
    assert np.isposinf(lut[:, :, m:]).all()


# ------------------------------------------------------------------ stage 1
SCAN_CASES = [
    # name, N, Q, overrides, threshold rule
    ("C0", 10_000, 100, {}, ("kth", 20, 1.5)),            # lanes = queries, Kf = 1
    ("C1", 50_003, 130, {}, ("q", 0.01)),                 # lanes = queries, Kf = 2, ragged tail
    ("C1", 5_000, 3, {}, ("q", 0.02)),                    # streaming kernel, two query groups
    ("C1", 40_007, 1, {}, ("q", 0.01)),                   # streaming kernel, one query, Kf = 2
    ("C4", 70_001, 2, dict(K=6), ("q", 0.01)),            # streaming kernel, Kf = 4, two queries
    ("C4", 33_000, 1, dict(K=5), ("q", 0.3)),             # streaming kernel, many survivors: flushes
    ("C0", 9_000, 4, {}, ("q", 0.01)),                    # streaming kernel, Kf = 1
    ("C2", 9_000, 2, dict(d=32, Kf=3), ("q", 0.01)),      # streaming kernel, Kf = 3
    ("C2", 20_001, 70, dict(d=64), ("q", 0.01)),          # Kf = 4
    ("C3", 60_000, 64, {}, ("q", 0.01)),                  # clustered codes: ties and bursts
    ("C4", 30_000, 9, dict(Kf=6), ("q", 0.05)),           # Kf = 6
    ("C1", 700, 8, {}, ("q", 0.5)),                       # tiny N, half survive
]


def _thr(P, rule):
    if rule[0] == "kth":
        return thresholds_kth(P, rule[1], rule[2])
    return thresholds_quantile(P, rule[1])


@pytest.mark.parametrize("mode", [1, 2], ids=["streamed", "grouped"])
@pytest.mark.parametrize("name,N,Q,over,rule", SCAN_CASES)
def test_scan_fast_candidates_match_oracle(gpu, name, N, Q, over, rule, mode):
    cfg = small(name, N, Q, **over)
    if mode == 2 and cfg["Kf"] > 4:
        pytest.skip("grouping exists for Kf <= 4 only")
    g = Gpu(gpu, cfg, mode)
    T, P, D = oracle_all(cfg)
    thr = _thr(P, rule)
    cap = int((P < thr[:, None].astype(np.float64)).sum(axis=1).max() * 1.2) + 64
    lut = g.lut()
    ids, part, cnt = g.scan(lut, thr, cap)
    ids, part, cnt = _u32(ids), part.cpu().numpy(), _u32(cnt)
    for q in range(Q):
        assert cnt[q] <= cap
        check_candidates(P[q], thr[q], ids[q], part[q], cnt[q], cap)
    # determinism of the candidate sets
    ids2, _, cnt2 = g.scan(lut, thr, cap)
    ids2, cnt2 = _u32(ids2), _u32(cnt2)
    assert np.array_equal(cnt, cnt2)
    for q in range(Q):
        assert np.array_equal(np.sort(ids[q][:cnt[q]]), np.sort(ids2[q][:cnt2[q]]))


@pytest.mark.parametrize("mode", [1, 2], ids=["streamed", "grouped"])
@pytest.mark.parametrize("Q", [2, 70])
def test_scan_fast_special_thresholds_and_overflow(gpu, Q, mode):
    cfg = small("C1", 3000, Q)
    g = Gpu(gpu, cfg, mode)
    T, P, D = oracle_all(cfg)
    N = 3000
    lut = g.lut()
    # +inf keeps everything
    inf = np.full(Q, np.inf, dtype=np.float32)
    ids, part, cnt = g.scan(lut, inf, N)
    ids, cnt = _u32(ids), _u32(cnt)
    assert (cnt == N).all()
    for q in range(Q):
        assert np.array_equal(np.sort(ids[q]), np.arange(N, dtype=np.uint32))
    # -inf and NaN keep nothing
    for v in (-np.inf, np.nan):
        _, _, cnt = g.scan(lut, np.full(Q, v, dtype=np.float32), 8)
        assert (_u32(cnt) == 0).all()
    # overflow: true count reported, the cap entries written are genuine survivors
    thr = thresholds_quantile(P, 0.1)
    cap = 50
    ids, part, cnt = g.scan(lut, thr, cap)
    ids, part, cnt = _u32(ids), part.cpu().numpy(), _u32(cnt)
    for q in range(Q):
        exact = int((P[q] < np.float64(thr[q])).sum())
        assert abs(int(cnt[q]) - exact) <= 3 and cnt[q] > cap
        check_candidates(P[q], thr[q], ids[q], part[q], cnt[q], cap)


@pytest.mark.parametrize("Q,Kf,m,N", [
    (140, 2, 256, 70_001),     # every tuple below the threshold: a wavefront's buffer fills and is expanded more than once
    (3, 2, 3, 40_003),         # nine tuples of 4445 items: windows of survivors far longer than a step
    (2, 1, 256, 270_001), (70, 1, 2, 70_000), (29, 1, 256, 20_001), (1030, 1, 100, 2_000),     # 64, 15, 4 blocks per query, one
])
def test_scan_fast_grouped_lists_at_the_edges_of_its_buffers(gpu, Q, Kf, m, N):
    """Grouped lists against the item-by-item lists (same additions): equal as sets, crude distances bit for bit."""
    cfg = small("C1", N, Q, d=16, Kf=Kf, m=m)
    lists = []
    for mode in (1, 2):
        g = Gpu(gpu, cfg, mode)
        lut = g.lut()
        sums = np.sort(sum(lut.cpu().numpy()[:, k, cfg["codes"][k]] for k in range(Kf)), axis=1)
        thr = np.where(np.arange(Q) % 2 == 0, np.inf, sums[:, N // 2]).astype(np.float32)
        ids, part, cnt = g.scan(lut, thr, N)
        ids, part, cnt = _u32(ids), part.cpu().numpy(), _u32(cnt)
        order = np.argsort(np.where(np.arange(N) < cnt[:, None], ids, 0xFFFFFFFF), axis=1, kind="stable")
        lists.append((cnt, [(ids[q][order[q, :cnt[q]]], part[q][order[q, :cnt[q]]]) for q in range(Q)]))
    assert np.array_equal(lists[0][0], lists[1][0]) and (lists[0][0][::2] == N).all()
    for a, b in zip(lists[0][1], lists[1][1]):
        assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])


# ------------------------------------------------------------------ stage 2 + list
@pytest.mark.parametrize("name,N,Q,over,rule,topk", [
    ("C0", 10_000, 100, {}, ("kth", 20, 1.5), 10),
    ("C1", 50_003, 66, {}, ("q", 0.01), 100),
    ("C2", 20_001, 5, dict(d=64), ("q", 0.3), 100),       # long lists, few queries: sliced + merged
    ("C4", 30_000, 9, dict(Kf=6, K=7), ("q", 0.05), 1000),  # one slow codebook, long result
    ("C1", 4_000, 10, dict(Kf=8), ("q", 0.05), 7),        # Kf == K: stage 2 adds nothing
])
def test_refine_matches_oracle(gpu, name, N, Q, over, rule, topk):
    cfg = small(name, N, Q, **over)
    g = Gpu(gpu, cfg, 1)
    T, P, D = oracle_all(cfg)
    thr = _thr(P, rule)
    cap = int((P < thr[:, None].astype(np.float64)).sum(axis=1).max() * 1.2) + 64
    lut = g.lut()
    ids, part, cnt = g.scan(lut, thr, cap)
    out_ids, out_dist = g.refine(lut, ids, part, cnt, topk)
    for q in range(Q):
        check_topk(P[q], D[q], thr[q], topk, out_ids[q], out_dist[q])
    # without crude distances: ids only from stage 1, whole sum in stage 2, identical bits
    ids2, none, cnt2 = g.scan(lut, thr, cap, want_partial=False)
    assert none is None and np.array_equal(_u32(cnt2), _u32(cnt))
    out_ids2, out_dist2 = g.refine(lut, ids2, None, cnt2, topk)
    assert np.array_equal(out_ids2, out_ids) and np.array_equal(out_dist2, out_dist)


@pytest.mark.parametrize("Q,n,topk,values", [
    (1, 8192, 100, "real"), (1, 8193, 100, "real"),        # one load of a block's registers, and one key more
    (2, 131_073, 20, "real"), (1, 300_001, 512, "real"),   # several parts per query, joined
    (3, 40_961, 256, "real"), (21, 40_961, 10, "few"), (2, 131_073, 257, "real"), (22, 131_073, 9, "real"),    # one key more than
    (2, 40_960, 30, "real"), (2, 131_072, 400, "few"),     # a block takes alone, and just as many
    (3, 20_000, 512, "few"), (2, 140_000, 64, "few"),      # masses of equal distances: the ids decide
    (600, 700, 256, "real"), (5, 1000, 257, "few"),        # block sizes, at their longest results
    (600, 1024, 512, "real"), (513, 1025, 300, "few"), (600, 4097, 512, "real"), (530, 1000, 100, "few"),
    (4, 300, 1, "real"), (40, 257, 300, "real"),           # shortest result; fewer keys than the result holds
    (530, 5_000, 30, "few"), (2, 20_000, 150, "few threads"),      # 512 threads; 100 of 1024 threads hold the 1954 smallest
])
def test_refine_lists_are_the_exact_smallest_keys(gpu, Q, n, topk, values):
    """The list of every query = the first topk of its candidates ordered by (D, id), D the fp32 sum in codebook
    order: exact, since the sums are formed from the given tables in that order on both sides."""
    torch, _ = gpu
    rng = np.random.default_rng(Q * 1000 + topk)
    K, m, d, N = 4, 256, 8, n + 50
    cfg = dict(K=K, Kf=2, codebooks=rng.standard_normal((K, m, d)).astype(np.float32),
               codes=rng.integers(0, m, (K, N), dtype=np.uint8), queries=np.zeros((Q, d), np.float32))
    g = Gpu(gpu, cfg)
    lut = rng.random((Q, K, 256), dtype=np.float32) if values == "real" else \
        rng.integers(0, 2 if values == "few" else 50, (Q, K, 256)).astype(np.float32)
    ids = np.stack([rng.permutation(N)[:n] for _ in range(Q)]).astype(np.int32)
    if values == "few threads":
        for q in range(Q):
            D = sum(lut[q, k, cfg["codes"][k, ids[q]]] for k in range(K))
            at = np.argsort(np.arange(n) % 1024 >= 100, kind="stable")
            ids[q, at] = ids[q, np.lexsort((ids[q], D))]
    cnt = np.array([n if q % 4 == 0 else n // (q % 4 + 1) * (q % 7 != 3) for q in range(Q)], np.int32)
    out_ids, out_dist = g.refine(_dev(torch, lut), _dev(torch, ids), None, _dev(torch, cnt), topk)
    for q in range(Q):
        mine = ids[q, :cnt[q]]
        D = lut[q, 0, cfg["codes"][0, mine]]
        for k in range(1, K):
            D = D + lut[q, k, cfg["codes"][k, mine]]
        order = np.lexsort((mine, D))[:topk]
        kept = order.size
        assert np.array_equal(out_ids[q, :kept], mine[order].astype(np.uint32)) and np.array_equal(out_dist[q, :kept], D[order])
        assert (out_ids[q, kept:] == 0xFFFFFFFF).all() and np.isinf(out_dist[q, kept:]).all()


@pytest.mark.parametrize("topk,m", [(100, 256), (400, 256), (20, 3)])
def test_search_whose_first_selection_is_joined_from_parts(gpu, topk, m):
    """More than 131072 keys per query before the first selection of the hit-bit form, which leaves its result in place of the
    keys for the rest of the search: lists exact by (D, id), D the fp32 sums of the library's own tables."""
    torch, b = gpu
    Q, K, Kf, d, N = 3, 4, 3, 8, 130 * 2 * 32768 + 777
    g = torch.Generator(device="cuda"); g.manual_seed(topk)
    cb = torch.randn((K, m, d), device="cuda", generator=g)
    codes = torch.randint(0, m, (K, N), dtype=torch.uint8, device="cuda", generator=g)
    queries = torch.randn((Q, d), device="cuda", generator=g)
    index = b.icq_index_create(cb, codes, Kf)
    lut = torch.empty((Q, K, 256), device="cuda")
    b.icq_build_lut(index, queries, lut)
    ids, dist = torch.full((Q, topk), -7, dtype=torch.int32, device="cuda"), torch.zeros((Q, topk), device="cuda")
    count = torch.full((Q,), -7, dtype=torch.int32, device="cuda")
    ws = torch.empty(b.icq_workspace_bytes(index, Q, N, topk), dtype=torch.uint8, device="cuda")
    for _ in range(2):
        b.icq_search(index, queries, torch.full((Q,), np.inf, device="cuda"), N, topk, ids, dist, count, ws)
        assert (count == N).all()
        for q in range(Q):
            D = lut[q, 0][codes[0].long()]
            for k in range(1, K):
                D = D + lut[q, k][codes[k].long()]
            want = torch.sort(D, stable=True)
            assert torch.equal(ids[q].long(), want.indices[:topk]) and torch.equal(dist[q], want.values[:topk])


@pytest.mark.parametrize("Q,topk", [(500, 256), (260, 1), (180, 47), (130, 256), (100, 30)])     # 2, 2, 3, 4, 6 lists per query
def test_grouped_lists_joined_from_several_blocks(gpu, Q, topk):
    """The same lists, bit for bit, as from the item-by-item form; none, one, few and all items survive; with ties."""
    torch, b = gpu
    K, Kf, d, N, m = 6, 2, 8, 40_000, 200
    g = torch.Generator(device="cuda"); g.manual_seed(Q)
    cb = torch.randn((K, m, d), device="cuda", generator=g)
    codes = torch.randint(0, m, (K, N), dtype=torch.uint8, device="cuda", generator=g)
    codes[:, N // 2:] = codes[:, :N // 2]
    queries = torch.randn((Q, d), device="cuda", generator=g)
    index = b.icq_index_create(cb, codes, Kf)
    lut = torch.empty((Q, K, 256), device="cuda")
    b.icq_build_lut(index, queries, lut)
    P = torch.sort(lut[:, 0][:, codes[0].long()] + lut[:, 1][:, codes[1].long()], dim=1).values
    rank = torch.tensor([0, 2, topk // 2 * 2, topk + 40, 4000, N - 1], device="cuda")[torch.arange(Q, device="cuda") % 6]
    thr = P.gather(1, rank[:, None])[:, 0].contiguous()
    thr[5::12] = np.inf
    out = []
    for mode in (b.ICQ_SCAN_GROUPED, b.ICQ_SCAN_STREAMED):
        b.icq_index_set_scan_mode(index, mode)
        ids, dist = torch.full((Q, topk), -7, dtype=torch.int32, device="cuda"), torch.zeros((Q, topk), device="cuda")
        count = torch.full((Q,), -7, dtype=torch.int32, device="cuda")
        ws = torch.empty(b.icq_workspace_bytes(index, Q, N, topk), dtype=torch.uint8, device="cuda")
        b.icq_search(index, queries, thr, N, topk, ids, dist, count, ws)
        out.append((ids, dist, count))
    assert all(torch.equal(x, y) for x, y in zip(*out))
    assert (out[0][2][0::6] == 0).all() and (out[0][0][0::6] == -1).all() and (out[0][2][5::12] == N).all()


# ------------------------------------------------------------------ whole path
def _check_search(g, cfg, T, P, D, thr, topk, cap, min_equal=0.9):
    out_ids, out_dist, surv = g.search(thr, cap, topk)
    o_ids, o_dist, o_cnt = orc.search(T, cfg["codes"], cfg["Kf"], thr, topk)
    n_equal = n_eligible = 0
    for q in range(g.Q):
        if np.isnan(thr[q]):
            assert surv[q] == 0 and (out_ids[q] == 0xFFFFFFFF).all() and np.isinf(out_dist[q]).all()
            continue
        band = np.nonzero((P[q] >= thr[q] - tol(thr[q])) & (P[q] <= thr[q] + tol(thr[q])))[0] \
            if np.isfinite(thr[q]) else np.zeros(0, dtype=np.int64)
        assert abs(int(surv[q]) - int(o_cnt[q])) <= band.size
        check_topk(P[q], D[q], thr[q], topk, out_ids[q], out_dist[q])
        if not (np.isin(o_ids[q], band).any() or np.isin(out_ids[q], band).any()):
            n_eligible += 1
            n_equal += np.array_equal(out_ids[q], o_ids[q])
    # where no threshold-band item reaches the list, the lists are identical up to near-ties
    assert n_equal >= min_equal * n_eligible
    return out_ids, out_dist, surv


@pytest.mark.parametrize("name,N,Q,over,rule", [
    ("C0", None, None, {}, ("kth", 20, 1.5)),             # the tiny config, complete
    ("C1", 200_003, 130, {}, ("q", 0.01)),
    ("C2", 50_001, 70, {}, ("q", 0.01)),                  # d = 960, Kf = 4
    ("C3", 100_000, 256, {}, ("q", 0.01)),
    ("C4", 120_000, 128, {}, ("q", 0.01)),
    ("C1", 2_000, 1, {}, ("q", 0.01)),                    # one query
    ("C1", 300, 33, {}, ("kth", 3, 1.0)),                 # fewer survivors than topk
    ("C0", 70_000, 40, {}, ("q", 0.02)),                  # Kf = 1: 256 groups of ~270 items
])
@pytest.mark.parametrize("mode", [1, 2], ids=["streamed", "grouped"])
def test_search_matches_oracle(gpu, name, N, Q, over, rule, mode):
    cfg = small(name, N, Q, **over)
    if mode == 2 and cfg["Kf"] > 4:
        pytest.skip("grouping exists for Kf <= 4 only")
    g = Gpu(gpu, cfg, mode)
    T, P, D = oracle_all(cfg)
    thr = _thr(P, rule)
    exact = (P < thr[:, None].astype(np.float64)).sum(axis=1)
    _check_search(g, cfg, T, P, D, thr, cfg["topk"], int(exact.max() * 1.2) + 64)


# With grouping, record width <= 16 bytes and topk <= 256 the grouped kernel keeps the
# nearest-neighbour lists on chip (no candidate list in memory).  From 1024 queries on a block
# owns its query; with fewer, up to 8 blocks share a query's surviving tuples and a merge kernel
# joins their lists.  The cases below run both forms.
@pytest.mark.parametrize("name,N,Q,over,rule,topk", [
    ("C1", 70_000, 600, {}, ("q", 0.01), 100),              # about one item per fast-code tuple
    ("C1", 40_000, 512, {}, ("q", 0.02), 128),              # fewer items than tuples
    ("C0", 70_000, 520, {}, ("q", 0.02), 10),               # Kf = 1: 256 tuples of ~270 items, 4-byte records
    ("C3", 150_000, 512, {}, ("q", 0.01), 100),             # clustered codes: a few huge tuples, bursts
    ("C2", 60_000, 512, dict(d=32, Kf=2), ("q", 0.01), 100),  # K = 16: 16-byte records
    ("C1", 60_000, 512, {}, ("q", 0.25), 100),              # many surviving tuples: several passes per query
    ("C1", 3_000, 512, {}, ("kth", 3, 1.0), 100),           # fewer survivors than topk
    ("C1", 50_000, 512, {}, ("q", 0.03), 256),              # longest on-chip list: final order by the register sort
    ("C1", 70_000, 1100, {}, ("q", 0.01), 100),             # one block per query
    ("C1", 70_000, 24, {}, ("q", 0.01), 100),               # 8 blocks per query
    ("C3", 150_000, 150, {}, ("q", 0.01), 100),             # 4 blocks per query, clustered codes
    ("C3", 150_000, 75, {}, ("q", 0.01), 100),              # 7 blocks per query, clustered codes
    ("C1", 60_000, 300, {}, ("q", 0.25), 100),              # 2 blocks per query, several passes each
    ("C1", 3_000, 40, {}, ("kth", 3, 1.0), 100),            # 8 blocks, fewer survivors than topk, some blocks with none
    ("C1", 50_000, 130, {}, ("q", 0.03), 256),              # 4 blocks, 256 keys each into the merge
    ("C2", 60_000, 90, dict(d=32, Kf=2), ("q", 0.01), 100), # 6 blocks, 16-byte records
])
def test_search_with_lists_kept_on_chip(gpu, name, N, Q, over, rule, topk):
    cfg = small(name, N, Q, **over)
    g = Gpu(gpu, cfg, 2)
    T, P, D = oracle_all(cfg)
    thr = _thr(P, rule)
    thr[5] = np.inf
    thr[11] = np.nan
    ids2, dist2, surv2 = _check_search(g, cfg, T, P, D, thr, topk, N)
    # the item-by-item form agrees to the bit, and so do the leading rows of lists too long to keep
    # on chip (300: one key per survivor to the select kernel; 513: position lists and the generic
    # stage-2 kernel)
    ids1, dist1, surv1 = Gpu(gpu, cfg, 1).search(thr, N, topk)
    assert np.array_equal(surv2, surv1) and np.array_equal(ids2, ids1) and np.array_equal(dist2, dist1)
    for longer in (300, 513):
        ids3, dist3, surv3 = g.search(thr, N, longer)
        assert np.array_equal(surv3, surv2) and np.array_equal(ids3[:, :topk], ids2)
        assert np.array_equal(dist3[:, :topk], dist2)


def test_search_with_queries_that_are_codewords(gpu):
    """Queries equal to a codeword of a slow codebook: the table entry of that codeword is
    ||q||^2 - 2<q,c> + ||c||^2 = 0 up to rounding, on either side of zero.  The grouped kernel
    prunes tuples by its list's bound only when no table entry is negative; with such queries
    some blocks run with the pruning and some without (about 135 of the 600 queries get a negative
    entry, 48 an exact zero), and both must give the oracle's lists."""
    cfg = small("C1", 70_000, 600)
    rng = np.random.default_rng(11)
    K, m = cfg["K"], cfg["codebooks"].shape[1]
    for q in range(0, 600, 2):
        cfg["queries"][q] = cfg["codebooks"][rng.integers(2, K), rng.integers(0, m)]
    g = Gpu(gpu, cfg, 2)
    T, P, D = oracle_all(cfg)
    thr = thresholds_quantile(P, 0.02)
    _check_search(g, cfg, T, P, D, thr, 100, 70_000)
    ids1, dist1, surv1 = Gpu(gpu, cfg, 1).search(thr, 70_000, 100)
    ids2, dist2, surv2 = g.search(thr, 70_000, 100)
    assert np.array_equal(surv2, surv1) and np.array_equal(ids2, ids1) and np.array_equal(dist2, dist1)


def test_search_infinite_threshold_is_exhaustive_adc(gpu):
    cfg = small("C1", 20_000, 20)
    g = Gpu(gpu, cfg)
    T, P, D = oracle_all(cfg)
    inf = np.full(20, np.inf, dtype=np.float32)
    out_ids, out_dist, surv = g.search(inf, 20_000, 100)
    e_ids, e_dist = orc.adc_exhaustive(T, cfg["codes"], 100)
    assert (surv == 20_000).all()
    for q in range(20):
        check_topk(P[q], D[q], np.inf, 100, out_ids[q], out_dist[q])
    assert (out_ids == e_ids).mean() > 0.98


def test_search_grouped_with_many_surviving_tuples(gpu):
    """Thresholds that let far more fast-code tuples through than the grouped kernel buffers
    at once (several passes per query), an infinite and a NaN threshold among them."""
    cfg = small("C1", 150_000, 12)
    g = Gpu(gpu, cfg, 2)
    T, P, D = oracle_all(cfg)
    thr = thresholds_quantile(P, 0.2)
    thr[3] = np.inf
    thr[7] = np.nan
    thr[9] = np.float32(np.sort(P[9])[5000])
    N, topk = 150_000, 100
    out_ids, out_dist, surv = g.search(thr, N, topk)
    for q in range(12):
        if q == 7:
            assert surv[q] == 0 and (out_ids[q] == 0xFFFFFFFF).all() and np.isinf(out_dist[q]).all()
            continue
        band = np.count_nonzero((P[q] >= thr[q] - tol(thr[q])) & (P[q] <= thr[q] + tol(thr[q]))) if np.isfinite(thr[q]) else 0
        exact = int((P[q] < np.float64(thr[q])).sum())
        assert abs(int(surv[q]) - exact) <= band
        check_topk(P[q], D[q], thr[q], topk, out_ids[q], out_dist[q])
    # same lists from the item-by-item form
    g1 = Gpu(gpu, cfg, 1)
    ids1, dist1, surv1 = g1.search(thr, N, topk)
    assert np.array_equal(surv, surv1) and np.array_equal(out_ids, ids1) and np.array_equal(out_dist, dist1)


@pytest.mark.parametrize("mode,Q", [(1, 12), (2, 1100), (2, 300), (2, 40)],
                         ids=["streamed", "grouped-1-block", "grouped-2-blocks", "grouped-8-blocks"])
def test_search_with_masses_of_equal_distances(gpu, mode, Q):
    """Items drawn from 8 code patterns only: thousands of exactly equal distances, so the
    lists are decided by the item ids alone (order (distance, id)) and every cut of a
    running list meets far more ties than it can hold.  Grouped: the lists stay on chip, with
    one, two or eight blocks per query."""
    cfg = small("C1", 40_000, Q)
    rng = np.random.default_rng(5)
    patterns = rng.integers(0, 256, size=(cfg["K"], 8), dtype=np.uint8)
    cfg["codes"] = np.ascontiguousarray(patterns[:, rng.integers(0, 8, size=40_000)])
    g = Gpu(gpu, cfg, mode)
    T, P, D = oracle_all(cfg)
    thr = np.full(Q, np.inf, dtype=np.float32)
    for q in range(6, Q):                                   # let the 5 nearest patterns (by crude distance) through
        u = np.unique(P[q])
        thr[q] = np.float32(0.5 * (u[4] + u[5])) if u.size > 5 else np.inf
    topk = 100
    out_ids, out_dist, surv = g.search(thr, 40_000, topk)
    o_ids, o_dist, o_cnt = orc.search(T, cfg["codes"], cfg["Kf"], thr, topk)
    assert np.array_equal(surv, o_cnt)
    assert np.array_equal(out_ids, o_ids)
    assert np.allclose(out_dist, o_dist, rtol=1e-4, atol=1e-4)


def test_stage_timing_records_the_search_calls(gpu):
    cfg = small("C1", 40_000, 64)
    g = Gpu(gpu, cfg)
    T, P, D = oracle_all(cfg)
    thr = thresholds_quantile(P, 0.01)
    with pytest.raises(g.b.IcqError):
        g.b.icq_index_stage_times(g.index)              # timing is off
    g.b.icq_index_set_stage_timing(g.index, True)
    with pytest.raises(g.b.IcqError):
        g.b.icq_index_stage_times(g.index)              # nothing recorded yet
    ref = g.search(thr, 1024, 100)
    for _ in range(2):
        again = g.search(thr, 1024, 100)
        assert np.array_equal(ref[0], again[0])
    ms, calls, batches = g.b.icq_index_stage_times(g.index)
    assert calls == 3 and batches == 1 and all(0.0 < x < 1e3 for x in ms)
    with pytest.raises(g.b.IcqError):
        g.b.icq_index_stage_times(g.index)              # reading resets the record
    g.b.icq_index_set_stage_timing(g.index, False)
    assert np.array_equal(ref[0], g.search(thr, 1024, 100)[0])


def test_search_in_sub_batches_gives_the_same_lists(gpu):
    cfg = small("C1", 30_000, 300)
    g = Gpu(gpu, cfg)
    T, P, D = oracle_all(cfg)
    thr = thresholds_quantile(P, 0.01)
    cap, topk = 512, 50
    full = g.search(thr, cap, topk)
    need64 = g.b.icq_workspace_bytes(g.index, 64, cap, topk)
    sub = g.search(thr, cap, topk, ws_bytes=need64 + 4096)     # forces batches of 64 queries
    assert np.array_equal(full[0], sub[0]) and np.array_equal(full[1], sub[1])
    assert np.array_equal(full[2], sub[2])
    with pytest.raises(g.b.IcqError):
        g.search(thr, cap, topk, ws_bytes=1024)


def test_empty_inputs(gpu):
    torch, b = gpu
    cfg = small("C1", 10, 4)
    cfg["codes"] = np.ascontiguousarray(cfg["codes"][:, :0])
    g = Gpu(gpu, cfg)
    thr = np.full(4, np.inf, dtype=np.float32)
    out_ids, out_dist, surv = g.search(thr, 16, 5)
    assert (out_ids == 0xFFFFFFFF).all() and np.isposinf(out_dist).all() and (surv == 0).all()
    # Q = 0 is a no-op
    lib = b.load()
    assert lib.icq_search(g.index.handle, None, 0, None, 16, 5, None, None, None, None, 0, None) == 0
    assert lib.icq_build_lut(g.index.handle, None, 0, None, None) == 0


def test_argument_errors_on_a_live_index(gpu):
    torch, b = gpu
    cfg = small("C1", 1000, 4)
    g = Gpu(gpu, cfg)
    lib = b.load()
    one = g.queries.data_ptr()
    h = g.index.handle
    assert lib.icq_search(h, one, 4, one, 16, 0, one, one, None, one, 1 << 20, None) == b.ICQ_ERR_ARG
    assert lib.icq_search(h, one, 4, one, 16, 2000, one, one, None, one, 1 << 20, None) == b.ICQ_ERR_ARG
    assert lib.icq_search(h, one, 4, one, 0, 5, one, one, None, one, 1 << 20, None) == b.ICQ_ERR_ARG
    assert lib.icq_search(h, one, 4, one, 16, 5, one, one, None, None, 0, None) == b.ICQ_ERR_WORKSPACE
    assert lib.icq_search(h, one, 4, one, 16, 5, one, one, None, one + 4, 1 << 20, None) == b.ICQ_ERR_WORKSPACE
    assert lib.icq_search(h, one, -1, one, 16, 5, one, one, None, one, 1 << 20, None) == b.ICQ_ERR_ARG



# ------------------------------------------------------------------ Kf = 3, 4: items grouped by their first two fast sub-codes
# With Kf = 3 or 4 the index also keeps the items ordered by (code_0, code_1); stage 1 then forms
# that pair's table sum once per 16 positions and streams only the other one or two fast rows.
# Inside icq_search the survivors travel as one hit bit per scan position and query, and stage 2
# walks them chunk by chunk (the items of the nearest runs bound what they may add).
# Same additions in the same order as item by item: the two forms must agree bit for bit.
@pytest.mark.parametrize("name,N,Q,over,frac,topk", [
    ("C4", 150_000, 37, {}, 0.01, 100),                      # Kf = 4, 16-byte records
    ("C2", 90_001, 9, dict(d=48, Kf=3), 0.02, 100),          # Kf = 3: one streamed row
    ("C4", 60_000, 3, dict(K=7), 0.01, 10),                  # 8-byte records, three queries (four per pass, ragged)
    ("C4", 60_000, 2, dict(K=4), 0.05, 10),                  # Kf == K, two queries per pass
    ("C4", 45_000, 1, dict(K=5), 0.3, 50),                   # one query per pass, dense hits
    ("C4", 80_000, 20, dict(K=20), 0.01, 100),               # 32-byte records: candidate lists, ids through the position map
    ("C4", 30_000, 12, {}, 0.02, 700),                       # long result: candidate lists
    ("C3", 120_000, 33, dict(K=8, Kf=4), 0.01, 100),         # clustered fast sub-codes: a few huge pairs
])
def test_search_grouped_by_the_first_two_fast_codes(gpu, name, N, Q, over, frac, topk):
    cfg = small(name, N, Q, **over)
    T, P, D = oracle_all(cfg)
    thr = thresholds_quantile(P, frac)
    if Q >= 9:
        thr[1], thr[2], thr[5] = np.inf, np.nan, -np.inf
    exact = np.nan_to_num((P < thr[:, None].astype(np.float64)).sum(axis=1))
    cap = int(exact.max() * 1.2) + 64
    g2 = Gpu(gpu, cfg, 2)
    # (K = 20 terms per distance: more near-ties that fp32 and fp64 order differently; the rule itself is unchanged)
    # (and in a list of 700 some pair always is: there only the rule decides)
    out = _check_search(g2, cfg, T, P, D, thr, topk, cap, min_equal=0.8 if topk <= 100 else 0.0)
    ref = Gpu(gpu, cfg, 1).search(thr, cap, topk)
    for a, c in zip(out, ref):
        assert np.array_equal(a, c, equal_nan=True)
    # the staged calls on the grouped index: ids (not positions) in the lists, same survivors
    lut = g2.lut()
    ids, part, cnt = g2.scan(lut, thr, cap)
    ids, part, cnt = _u32(ids), part.cpu().numpy(), _u32(cnt)
    for q in range(Q):
        if np.isnan(thr[q]):
            assert cnt[q] == 0
            continue
        check_candidates(P[q], thr[q], ids[q], part[q], cnt[q], cap)


@pytest.mark.parametrize("mode,over,Q", [(1, dict(K=12), 16), (2, dict(K=12), 16), (2, dict(K=8, Kf=3), 3),
                                         (1, dict(K=4, Kf=1), 1), (1, dict(K=6, Kf=2), 9), (2, dict(K=4), 5),
                                         (2, dict(K=8, Kf=3), 13), (2, dict(K=16), 21),
                                         (1, dict(K=4, Kf=1), 8), (1, dict(K=8, Kf=3), 12)],
                         ids=["streamed-K12", "grouped-K12", "grouped-Kf3-K8", "streamed-Kf1", "streamed-Kf2", "grouped-K4",
                              "grouped-Kf3-13-queries", "grouped-K16-21-queries", "streamed-Kf1-8-queries",
                              "streamed-Kf3-12-queries"])
def test_search_over_many_chunks_of_hit_bits(gpu, mode, over, Q):
    """From 2^22 items on icq_search hands the survivors of the item-by-item stage 1 to stage 2 as
    hit bits.  Enough items for more than a hundred stage-2 chunks (32768 scan positions each), so
    that the chunk walk is bounded by what the nearest runs hold, with a ragged last chunk; 4-, 8- and 16-byte records,
    one, two and four queries per pass of stage 1, and from six queries on over the pair ordering the
    16-bit pre-filter with eight queries per pass (ragged last pass), whose superset stage 2 cuts back
    by the exact comparison: thresholds that let everything, nothing, or only the items at the very
    smallest crude distance through."""
    cfg = small("C4", 4_300_017, Q, **over)
    T, P, D = oracle_all(cfg)
    thr = thresholds_quantile(P, 0.01)
    thr[Q - 1] = np.inf                                      # every position a survivor: dense rounds
    if Q >= 6:
        thr[0] = -np.inf
        thr[1] = np.nan
        thr[2] = np.nextafter(np.float32(P[2].min()), np.float32(np.inf))     # just above the smallest crude distance
        thr[3] = np.float32(P[3].min())                      # at it: P < t fails for every item (up to rounding)
        thr[4] = np.float32(np.quantile(P[4], 0.3))          # a third of the items survive
    g = Gpu(gpu, cfg, mode)
    out_ids, out_dist, surv = _check_search(g, cfg, T, P, D, thr, 100, cfg["N"], min_equal=0.8 if Q > 4 else 0.0)
    assert surv[Q - 1] == cfg["N"]
    if mode == 2:       # the grouped and the item-by-item order must agree bit for bit
        ref = Gpu(gpu, cfg, 1).search(thr, cfg["N"], 100)
        assert np.array_equal(ref[0], out_ids) and np.array_equal(ref[1], out_dist) and np.array_equal(ref[2], surv)

# ------------------------------------------------------------------ full size, as benchmarked
@pytest.mark.parametrize("mode", [0, 1], ids=["auto", "streamed"])
def test_full_size_workload_sampled_against_oracle(gpu, mode):
    """The benchmark's workload (C1: N = 1e6, Q = 1e4, top-100) in the benchmark's launch
    configuration (all queries in one icq_search call, same candidate capacity and the
    same sampled-quantile thresholds).  A sample of queries is checked against the
    oracle element by element; every query is checked for the properties that hold at
    any size."""
    import bench
    torch, b = gpu
    cfg = synth.make("C1")
    N, Q, Kf, topk = cfg["N"], cfg["Q"], cfg["Kf"], cfg["topk"]
    g = Gpu(gpu, cfg, mode)
    thr_dev = bench.sampled_thresholds(torch, b, g.cb, g.codes, g.queries, Kf, bench.SURVIVE_FRAC, 16384,
                                       cfg["seed"])
    thr = thr_dev.cpu().numpy()
    cap = 16384
    out_ids, out_dist, surv = g.search(thr, cap, topk)
    # properties for every query
    assert (surv <= cap).all(), "candidate capacity exceeded"
    assert (surv >= topk).all()
    assert (out_ids < N).all()
    assert (np.diff(out_dist, axis=1) >= 0).all(), "distances not ascending"
    srt = np.sort(out_ids, axis=1)
    assert (np.diff(srt.astype(np.int64), axis=1) > 0).all(), "duplicate ids in a result"
    assert 0.005 * N < surv.mean() < 0.02 * N
    # element by element on a sample
    sample = np.linspace(0, Q - 1, 12).astype(int)
    T = orc.lut(cfg["codebooks"], cfg["queries"][sample])
    P = orc.partial(T, cfg["codes"], Kf)
    _, _, D = orc.adc_exhaustive(T, cfg["codes"], 1, want_all=True)
    o_ids, o_dist, o_cnt = orc.search(T, cfg["codes"], Kf, thr[sample], topk)
    same = 0
    for r, q in enumerate(sample):
        band = ((P[r] >= thr[q] - tol(thr[q])) & (P[r] <= thr[q] + tol(thr[q]))).sum()
        assert abs(int(surv[q]) - int(o_cnt[r])) <= band
        check_topk(P[r], D[r], thr[q], topk, out_ids[q], out_dist[q])
        same += np.array_equal(out_ids[q], o_ids[r])
    assert same >= 10
    # the staged calls give the same lists as the fused call (same kernels, other plumbing)
    lut = g.lut()
    ids, part, cnt = g.scan(lut, thr, cap)
    assert np.array_equal(_u32(cnt), surv)
    r_ids, r_dist = g.refine(lut, ids, part, cnt, topk)
    assert np.array_equal(r_ids, out_ids) and np.array_equal(r_dist, out_dist)
    for r, q in enumerate(sample[:4]):
        check_candidates(P[r], thr[q], _u32(ids[q]), part[q].cpu().numpy(), int(_u32(cnt)[q]), cap)


@pytest.mark.parametrize("name,Q,n_check", [
    ("C2", None, 32),      # d = 960, K = 16, Kf = 4, N = 1e6, all 1000 queries in one call
    ("C3", 256, 32),       # N = 1e7 clustered codes, one batch of 256 queries (grouped, several blocks per query)
    ("C4", 128, 16),       # N = 1e8 (1.6 GB of codes), K = 16, Kf = 4, one batch of 128 queries
])
def test_other_configs_at_full_size_sampled_against_oracle(gpu, name, Q, n_check):
    """The remaining benchmark shapes at their full N, one icq_search call per query batch with
    thresholds from the library's own sampled quantile (1 %): properties for every query, the
    oracle element by element on a few queries."""
    import bench
    torch, b = gpu
    cfg = synth.make(name, Q=Q)
    N, Q, Kf, topk = cfg["N"], cfg["queries"].shape[0], cfg["Kf"], cfg["topk"]
    g = Gpu(gpu, cfg)
    thr = bench.sampled_thresholds(torch, b, g.cb, g.codes, g.queries, Kf, 0.01, 16384, cfg["seed"]).cpu().numpy()
    cap = int(N * 0.02)
    out_ids, out_dist, surv = g.search(thr, cap, topk)
    assert (surv <= cap).all() and (surv >= topk).all()
    assert (out_ids < N).all()
    assert (np.diff(out_dist, axis=1) >= 0).all(), "distances not ascending"
    srt = np.sort(out_ids, axis=1)
    assert (np.diff(srt.astype(np.int64), axis=1) > 0).all(), "duplicate ids in a result"
    assert 0.005 * N < surv.mean() < 0.02 * N
    sample = np.linspace(0, Q - 1, n_check).astype(int)
    T = orc.lut(cfg["codebooks"], cfg["queries"][sample])
    for r0 in range(0, n_check, 8):         # eight queries at a time: P and D are N doubles per query
        Pg = orc.partial(T[r0:r0 + 8], cfg["codes"], Kf)
        Dg = orc.partial(T[r0:r0 + 8], cfg["codes"], cfg["K"])    # all K terms, k ascending: the full distance
        for r in range(r0, min(r0 + 8, n_check)):
            q, P, D = sample[r], Pg[r - r0], Dg[r - r0]
            band = ((P >= thr[q] - tol(thr[q])) & (P <= thr[q] + tol(thr[q]))).sum()
            exact = int((P < np.float64(thr[q])).sum())
            assert abs(int(surv[q]) - exact) <= band
            check_topk(P, D, thr[q], topk, out_ids[q], out_dist[q])
        del Pg, Dg


def test_stream_scan_at_full_length_properties(gpu):
    """Streaming stage-1 kernel on a long code array (N = 2e7, Kf = 4; one, two and four
    queries per pass, the last with a ragged query group): survivor sets against the oracle's
    crude distances, element by element (the oracle finishes 2e7 items in seconds)."""
    torch, b = gpu
    cfg = synth.make("C4", N=20_000_003, Q=6, K=4)
    g = Gpu(gpu, cfg)
    T = orc.lut(cfg["codebooks"], cfg["queries"])
    P = orc.partial(T, cfg["codes"], 4)
    thr = thresholds_quantile(P, 0.01)
    thr[4] = np.float32(np.quantile(P[4], 0.04))       # a denser list next to sparse ones
    cap = 900_000
    lut = g.lut()
    for nq in (1, 2, 6):
        ids, part, cnt = g.scan(lut[:nq].contiguous(), thr[:nq], cap)
        ids, part, cnt = _u32(ids), part.cpu().numpy(), _u32(cnt)
        for q in range(nq):
            check_candidates(P[q], thr[q], ids[q], part[q], cnt[q], cap)


@pytest.mark.gpu
def test_stream_scan_of_an_array_beyond_the_last_level_cache(gpu):
    """Fast codes of more than 256 MB (Kf = 4, N = 6.72e7): with one or two queries per pass the
    streaming kernel then reads them with the non-temporal hint.  Survivor sets against the
    oracle's crude distances, element by element."""
    torch, b = gpu
    cfg = synth.make("C4", N=67_200_003, Q=2, K=4)
    g = Gpu(gpu, cfg)
    T = orc.lut(cfg["codebooks"], cfg["queries"])
    P = orc.partial(T, cfg["codes"], 4)
    thr = thresholds_quantile(P, 0.005)
    cap = 500_000
    lut = g.lut()
    for nq in (1, 2):
        ids, part, cnt = g.scan(lut[:nq].contiguous(), thr[:nq], cap)
        ids, part, cnt = _u32(ids), part.cpu().numpy(), _u32(cnt)
        for q in range(nq):
            check_candidates(P[q], thr[q], ids[q], part[q], cnt[q], cap)


# ------------------------------------------------------------------ threshold policy, operation counts
@pytest.mark.parametrize("name,N,Q,over,topk,M", [
    ("C1", 30_000, 70, {}, 100, 4096),
    ("C1", 30_000, 9, {}, 10, 1000),                    # sample length not a power of two
    ("C2", 9_000, 33, dict(d=64), 100, 2048),           # K = 16, Kf = 4
    ("C0", 10_000, 100, {}, 10, 4096),                  # K = 4, Kf = 1
    ("C1", 5_000, 513, {}, 10, 4096),                   # more queries than 1024-thread blocks have room for
    ("C1", 5_000, 520, {}, 7, 1025),
    ("C1", 2_000, 1100, {}, 20, 1500),                  # small blocks
    ("C0", 700, 600, {}, 700, 1024),                    # every sample item
    ("C1", 700, 5, {}, 100, 4096),                      # sample = the whole index
    ("C1", 60, 5, {}, 100, 4096),                       # fewer items than topk: nothing is pruned
])
def test_sample_thresholds_match_oracle(gpu, name, N, Q, over, topk, M):
    torch, b = gpu
    cfg = small(name, N, Q, **over)
    g = Gpu(gpu, cfg)
    T, P, D = oracle_all(cfg)
    rng = np.random.default_rng(3)
    sigma = rng.uniform(0.0, 2.0, size=Q).astype(np.float32)
    lut = g.lut()
    thr = torch.full((Q,), float("nan"), dtype=torch.float32, device="cuda")
    b.icq_sample_thresholds(g.index, lut, _dev(torch, sigma), topk, M, thr)
    thr0 = torch.full((Q,), float("nan"), dtype=torch.float32, device="cuda")
    b.icq_sample_thresholds(g.index, lut, None, topk, M, thr0)         # no margin
    torch.cuda.synchronize()
    thr, thr0 = thr.cpu().numpy(), thr0.cpu().numpy()
    want = orc.sample_thresholds(T, cfg["codes"], cfg["Kf"], sigma.astype(np.float64), topk, M)
    n = min(M, N)
    if n < topk:
        assert np.isposinf(thr).all() and np.isposinf(thr0).all() and np.isposinf(want).all()
        return
    exact = 0
    for q in range(Q):
        # fp32 and fp64 may order two sample items differently when their distances nearly tie
        # at the topk-th place: accept the crude distance of any item that ties with it
        Dk = np.sort(D[q, :n])[topk - 1]
        ties = np.nonzero(np.abs(D[q, :n] - Dk) <= tol(Dk))[0]
        err = np.abs(P[q, ties] + sigma[q] - thr[q]).min()
        assert err <= tol(thr[q]), (q, err)
        assert np.abs(P[q, ties] - thr0[q]).min() <= tol(thr0[q])
        exact += abs(want[q] - thr[q]) <= tol(want[q])
    assert exact >= 0.9 * Q
    with pytest.raises(b.IcqError):
        b.icq_sample_thresholds(g.index, lut, None, topk, 4097, torch.empty(Q, dtype=torch.float32, device="cuda"))


def test_two_pass_search_with_sampled_thresholds(gpu):
    """Thresholds from the first items, then the two-step search: the lists equal the oracle's
    two-step search under the same thresholds, and they contain what the paper's serial loop
    finds with the same margin wherever that loop's own running threshold never fell below
    the static one (checked through the crude distances of its results)."""
    torch, b = gpu
    cfg = small("C1", 60_000, 64)
    g = Gpu(gpu, cfg)
    T, P, D = oracle_all(cfg)
    Q, topk, M, Kf = 64, 50, 2048, cfg["Kf"]
    S = D - P
    sigma = (0.5 * S.std(axis=1)).astype(np.float32)
    thr = torch.empty((Q,), dtype=torch.float32, device="cuda")
    b.icq_sample_thresholds(g.index, g.lut(), _dev(torch, sigma), topk, M, thr)
    torch.cuda.synchronize()
    thr = thr.cpu().numpy()
    out_ids, out_dist, surv = _check_search(g, cfg, T, P, D, thr, topk, 60_000)
    r_ids, r_dist, refined = orc.running_search(T, cfg["codes"], Kf, sigma.astype(np.float64), topk)
    for q in range(Q):
        inside = r_ids[q][P[q, r_ids[q]] < thr[q] - tol(thr[q])]      # the loop's results that clearly pass t_q
        worst = out_dist[q][-1]
        need = inside[D[q, inside] < worst - tol(worst)]
        assert np.isin(need, out_ids[q]).all()


RUNNING_CASES = [
    # name, N, Q, overrides, topk, tile bounds, scan mode
    ("C1", 60_000, 48, {}, 100, [0, 300, 2_000, 9_000, 30_000, 60_000], 0),      # Kf = 2: tuples, lists on chip
    ("C1", 60_000, 48, {}, 10, [0, 300, 2_000, 9_000, 30_000, 60_000], 1),       # item by item
    ("C4", 70_001, 32, dict(K=16), 20, [0, 1_000, 8_000, 40_000, 70_001], 0),     # Kf = 4, ragged last tile
    ("C4", 70_001, 32, dict(K=16), 20, [0, 1_000, 8_000, 40_000, 70_001], 2),     # pair ordering forced
    ("C0", 5_000, 20, {}, 7, [0, 3, 9, 100, 101, 2_500, 5_000], 0),               # tiles shorter than the list, one item
    ("C1", 9_000, 5, {}, 1, [0, 9_000], 0),                                       # one tile: exhaustive
]


@pytest.mark.parametrize("name,N,Q,over,topk,bounds,mode", RUNNING_CASES)
def test_running_search_in_tiles_matches_oracle(gpu, name, N, Q, over, topk, bounds, mode):
    """The loop of Sec. 3.4 with the threshold refreshed per tile, against the oracle's statement of
    it.  Both sides decide P < t and D < D(f) in their own precision and a decision taken
    differently feeds back into the later thresholds, so the lists are compared exactly for the
    queries none of whose decisions lies within 1e-5 * (|x| + 1) of its threshold (five times the
    largest error measured between the two sides' distances), and every list is checked to be
    made of true distances in ascending order; the counts of exact comparisons must lie between
    the fewest and the most the band allows."""
    torch, b = gpu
    cfg = small(name, N, Q, **over)
    K, Kf = cfg["K"], cfg["Kf"]
    T, P, D = oracle_all(cfg)
    cbv = cfg["codebooks"].astype(np.float64)
    sig = float(sum(cbv[k].var(axis=0).sum() for k in range(Kf, K)))       # spread of the slow terms
    rng = np.random.default_rng(17)
    sigma = (sig * rng.uniform(0.0, 1.5, size=Q)).astype(np.float32)
    want_ids, want_dist, want_refined = orc.running_search_tiled(T, cfg["codes"], Kf, sigma.astype(np.float64), topk,
                                                                  np.array(bounds))
    cb = _dev(torch, cfg["codebooks"])
    tiles = []
    for a, e in zip(bounds[:-1], bounds[1:]):
        t = b.icq_index_create(cb, _dev(torch, cfg["codes"][:, a:e]), Kf)
        b.icq_index_set_scan_mode(t, mode)
        tiles.append(t)
    cap = max(e - a for a, e in zip(bounds[:-1], bounds[1:]))
    out_ids = torch.empty((Q, topk), dtype=torch.int32, device="cuda")
    out_dist = torch.empty((Q, topk), dtype=torch.float32, device="cuda")
    refined = torch.empty((Q,), dtype=torch.int32, device="cuda")
    ws = torch.empty(b.icq_running_workspace_bytes(tiles, Q, cap, topk), dtype=torch.uint8, device="cuda")
    for _ in range(2):          # a second call on the same workspace and outputs: nothing carried over
        b.icq_search_running(tiles, bounds[:-1], _dev(torch, cfg["queries"]), _dev(torch, sigma), cap, topk, out_ids,
                             out_dist, refined, ws)
    torch.cuda.synchronize()
    ids, dist, ref = _u32(out_ids), out_dist.cpu().numpy().astype(np.float64), _u32(refined)
    nclean = 0
    for q in range(Q):
        valid = ids[q] != 0xFFFFFFFF
        nv = int(valid.sum())
        assert valid[:nv].all() and nv == min(topk, N)
        got = ids[q, :nv].astype(np.int64)
        assert len(np.unique(got)) == nv and got.max() < N
        assert (np.abs(dist[q, :nv] - D[q, got]) <= tol(D[q, got])).all()
        assert (np.diff(dist[q, :nv]) >= 0).all()
        lst, lo, hi, clean = tiled_loop_analysis(P[q], D[q], float(sigma[q]), topk, bounds, lambda x: 1e-5 * (abs(x) + 1.0))
        if not clean:
            continue
        nclean += 1
        assert np.array_equal(lst.astype(np.uint32), want_ids[q])          # the analysis agrees with the oracle
        assert np.array_equal(ids[q], want_ids[q]), q
        assert lo <= ref[q] <= hi and lo <= want_refined[q] <= hi, (q, lo, ref[q], hi)
    assert nclean >= Q // 2, nclean
    if len(bounds) == 2:
        assert (ref == N).all()
    # argument errors: tiles from different codebook shapes, a workspace too small
    other = b.icq_index_create(_dev(torch, cfg["codebooks"][: K - 1]), _dev(torch, cfg["codes"][: K - 1, :64]), min(Kf, K - 1)) \
        if K > 1 else None
    if other is not None:
        with pytest.raises(b.IcqError):
            b.icq_running_workspace_bytes(tiles + [other], Q, cap, topk)
        b.icq_index_destroy(other)
    with pytest.raises(b.IcqError):
        b.icq_search_running(tiles, bounds[:-1], _dev(torch, cfg["queries"]), None, cap, topk, out_ids, out_dist, refined,
                             ws[: ws.numel() // 2 // 256 * 256])
    for t in tiles:
        b.icq_index_destroy(t)


def test_running_search_of_more_queries_than_one_batch(gpu):
    """33 000 queries: each tile's search takes them in two sub-batches over the caller's tables.  Lists and counts are those of
    the queries searched by themselves."""
    torch, b = gpu
    Q, K, Kf, d, topk = 33_000, 4, 3, 8, 20
    g = torch.Generator(device="cuda"); g.manual_seed(5)
    cb = torch.randn((K, 256, d), device="cuda", generator=g) * (0.6 ** torch.arange(K, device="cuda"))[:, None, None]
    bounds = [0, 300, 1300, 3000]
    codes = torch.randint(0, 256, (K, bounds[-1]), dtype=torch.uint8, device="cuda", generator=g)
    queries = torch.randn((Q, d), device="cuda", generator=g)
    tiles = [b.icq_index_create(cb, codes[:, x:y].contiguous(), Kf) for x, y in zip(bounds, bounds[1:])]

    def run(q):
        n = q.shape[0]
        ids, dist = torch.full((n, topk), -7, dtype=torch.int32, device="cuda"), torch.zeros((n, topk), device="cuda")
        count = torch.full((n,), -7, dtype=torch.int32, device="cuda")
        ws = torch.empty(b.icq_running_workspace_bytes(tiles, n, bounds[-1], topk), dtype=torch.uint8, device="cuda")
        b.icq_search_running(tiles, bounds[:-1], q, torch.full((n,), 2.0, device="cuda"), bounds[-1], topk, ids, dist, count, ws)
        return ids, dist, count
    whole = run(queries)
    assert (whole[2] >= 300).all() and (whole[2] < bounds[-1]).any()
    for x, y in ((0, 50), (32_700, 32_850), (Q - 40, Q)):
        assert all(torch.equal(w[x:y], p) for w, p in zip(whole, run(queries[x:y].contiguous())))


def test_running_search_at_full_size_sampled_against_oracle(gpu):
    """The largest workload (N = 1e8, K = 16, Kf = 4) in the launch configuration bench.py times: 8 tiles
    growing fourfold from 8192 items, one batch of 128 queries; four of them against the oracle's tiled loop, the rest by
    properties."""
    import bench
    torch, b = gpu
    cfg = synth.make("C4", Q=128)
    N, Q, K, Kf, topk = cfg["N"], 128, cfg["K"], cfg["Kf"], cfg["topk"]
    bounds = bench.tile_bounds(N)
    cb = _dev(torch, cfg["codebooks"])
    codes = _dev(torch, cfg["codes"])
    tiles = [b.icq_index_create(cb, codes[:, a:e].contiguous(), Kf) for a, e in zip(bounds[:-1], bounds[1:])]
    del codes
    cbv = cfg["codebooks"].astype(np.float64)
    sig = float(sum(cbv[k].var(axis=0).sum() for k in range(Kf, K)))
    sigma = torch.full((Q,), sig, dtype=torch.float32, device="cuda")
    cap = max(bounds[1], int(N * 0.02))
    out_ids = torch.empty((Q, topk), dtype=torch.int32, device="cuda")
    out_dist = torch.empty((Q, topk), dtype=torch.float32, device="cuda")
    refined = torch.empty((Q,), dtype=torch.int32, device="cuda")
    ws = torch.empty(b.icq_running_workspace_bytes(tiles, Q, cap, topk), dtype=torch.uint8, device="cuda")
    b.icq_search_running(tiles, bounds[:-1], _dev(torch, cfg["queries"]), sigma, cap, topk, out_ids, out_dist, refined, ws)
    torch.cuda.synchronize()
    ids, dist, ref = _u32(out_ids), out_dist.cpu().numpy().astype(np.float64), _u32(refined)
    for t in tiles:
        b.icq_index_destroy(t)
    del ws
    torch.cuda.empty_cache()
    assert (ids < N).all() and (np.diff(dist, axis=1) >= 0).all()
    assert (np.diff(np.sort(ids, axis=1).astype(np.int64), axis=1) > 0).all(), "duplicate ids in a result"
    assert (ref >= bounds[1]).all() and ref.mean() < 0.01 * N          # the first tile whole, then a tightening threshold
    sample = np.array([0, 41, 86, 127])
    T = orc.lut(cfg["codebooks"], cfg["queries"][sample])
    want_ids, _, want_refined = orc.running_search_tiled(T, cfg["codes"], Kf, np.full(sample.size, float(np.float32(sig))),
                                                         topk, np.array(bounds))
    nclean = 0
    for r, q in enumerate(sample):
        P = orc.partial(T[r:r + 1], cfg["codes"], Kf)[0]
        D = orc.partial(T[r:r + 1], cfg["codes"], K)[0]
        got = ids[q].astype(np.int64)
        assert (np.abs(dist[q] - D[got]) <= tol(D[got])).all()
        lst, lo, hi, clean = tiled_loop_analysis(P, D, float(np.float32(sig)), topk, bounds, lambda x: 1e-5 * (abs(x) + 1.0))
        if clean:
            nclean += 1
            assert np.array_equal(lst.astype(np.uint32), want_ids[r])
            assert np.array_equal(ids[q], want_ids[r])
            assert lo <= ref[q] <= hi and lo <= want_refined[r] <= hi
        else:
            # At this size some decision of every query hangs on rounding (the 100 nearest of 1e8 items lie
            # closer together than the band); the two runs then part ways by a few items, no more
            same = np.intersect1d(ids[q], want_ids[r]).size
            print("query %d: %d of %d ids as the oracle's, exact comparisons %d (oracle %d, band %d..%d)"
                  % (q, same, topk, ref[q], want_refined[r], lo, hi))
            assert same >= 0.95 * topk
            assert abs(int(ref[q]) - int(want_refined[r])) <= 0.05 * want_refined[r]
        del P, D


@pytest.mark.parametrize("K,Kf,mode", [(4, 3, 0), (12, 4, 0), (4, 3, 1)])
def test_search_from_hit_bits_in_pieces_of_chunks(gpu, K, Kf, mode):
    """Stage 2 takes windows of four to twelve chunks of hit bits by the number of (chunk, query) pairs: 2100 queries at once, in
    twos and in forties have the same lists, distances and counts, bit for bit (a query's work does not depend on the others)."""
    torch, b = gpu
    N, Q, d, topk = (1 << 22) + 4097, 2100, 16, 12
    gen = torch.Generator(device="cuda")
    gen.manual_seed(K)
    cb = torch.randn((K, 256, d), device="cuda", generator=gen) * torch.tensor([0.8 ** k for k in range(K)], device="cuda")[:, None, None]
    codes = torch.randint(0, 256, (K, N), dtype=torch.uint8, device="cuda", generator=gen)
    index = b.icq_index_create(cb.contiguous(), codes, Kf)
    b.icq_index_set_scan_mode(index, mode)
    queries = 1.5 * torch.randn((Q, d), device="cuda", generator=gen)
    lut = torch.empty((Q, K, 256), device="cuda")
    b.icq_build_lut(index, queries, lut)
    P = sum(lut[:, k].index_select(1, codes[k, :20_000].long()) for k in range(Kf))
    thr = P.kthvalue(30, dim=1).values.contiguous()            # 0.15 % of the items
    thr[3], thr[4] = -1.0, float("nan")                        # nothing survives
    cap = 20_000

    def run(step):
        ids = torch.empty((Q, topk), dtype=torch.int32, device="cuda")
        dist = torch.empty((Q, topk), device="cuda")
        count = torch.empty((Q,), dtype=torch.int32, device="cuda")
        ws = torch.empty(b.icq_workspace_bytes(index, min(Q, step), cap, topk), dtype=torch.uint8, device="cuda")
        for q in range(0, Q if step >= 40 else 24, step):
            at = slice(q, min(Q, q + step))
            b.icq_search(index, queries[at], thr[at], cap, topk, ids[at], dist[at], count[at], ws)
        torch.cuda.synchronize()
        return ids, dist, count
    want = run(Q)
    assert (want[2][3:5] == 0).all() and want[2].float().mean() > 1000
    for step, upto in ((40, Q), (2, 24)):
        for x, y in zip(run(step), want):
            assert torch.equal(x[:upto], y[:upto])


@pytest.mark.parametrize("K,Kf,mode,N", [(8, 3, 0, (1 << 22) + 70_001), (8, 2, 1, (1 << 22) + 65_537), (16, 4, 0, (1 << 22) + 1), (4, 3, 0, 20_000_003)])
def test_search_from_hit_bits_in_pieces_over_the_shares(gpu, K, Kf, mode, N):
    """Windows of four to twelve chunks of hit bits: the same lists and counts, bit for bit,
    whether nothing, a thousandth, a third or all of the items survive, and counts that are those of the crude distances."""
    torch, b = gpu
    Q, d, topk = 24, 16, 100
    gen = torch.Generator(device="cuda")
    gen.manual_seed(N)
    cb = torch.randn((K, 256, d), device="cuda", generator=gen) * torch.tensor([0.8 ** k for k in range(K)], device="cuda")[:, None, None]
    codes = torch.randint(0, 256, (K, N), dtype=torch.uint8, device="cuda", generator=gen)
    index = b.icq_index_create(cb.contiguous(), codes, Kf)
    b.icq_index_set_scan_mode(index, mode)
    queries = 1.5 * torch.randn((Q, d), device="cuda", generator=gen)
    lut = torch.empty((Q, K, 256), device="cuda")
    b.icq_build_lut(index, queries, lut)
    thr, survivors = torch.empty((Q,), device="cuda"), torch.empty((Q,), dtype=torch.int32, device="cuda")
    for q in range(Q):
        P = sum(lut[q, k].index_select(0, codes[k].long()) for k in range(Kf))
        thr[q] = (float("-inf"), P[:20_000].kthvalue(20).values, P[:20_000].kthvalue(300).values, P[:20_000].kthvalue(6000).values, float("inf"))[q % 5]
        survivors[q] = (P < thr[q]).sum()

    def run(step):
        ids = torch.empty((Q, topk), dtype=torch.int32, device="cuda")
        dist = torch.empty((Q, topk), device="cuda")
        count = torch.empty((Q,), dtype=torch.int32, device="cuda")
        ws = torch.empty(b.icq_workspace_bytes(index, step, N, topk), dtype=torch.uint8, device="cuda")
        for q in range(0, Q, step):
            at = slice(q, min(Q, q + step))
            b.icq_search(index, queries[at], thr[at], N, topk, ids[at], dist[at], count[at], ws)
        torch.cuda.synchronize()
        return ids, dist, count
    want = run(Q)
    assert torch.equal(want[2], survivors)
    for step in (1, 5, 8):
        for x, y in zip(run(step), want):
            assert torch.equal(x, y), step


@pytest.mark.parametrize("K,Kf,topk,codes", [
    (16, 4, 100, "uniform"), (16, 3, 512, "clustered"), (12, 4, 1, "far"), (9, 3, 300, "far"), (8, 4, 100, "clustered"),
    (4, 3, 47, "uniform"), (16, 2, 100, "uniform"), (8, 2, 512, "far"), (6, 1, 10, "clustered"), (16, 4, 100, "equal")])
def test_search_bounded_before_stage_2_equals_the_staged_calls(gpu, K, Kf, topk, codes):
    """Large indexes bound the result from the nearest runs before stage 2 drops what cannot reach it: the lists and counts of
    the staged calls, bit for bit, where the nearest runs hold the neighbours, nothing at all ("far": no item has a codeword
    near a query's first ones), thousands of items each ("clustered") or masses of equal distances ("equal"), and where fewer
    than topk, a few thousandths, a third, all or none of the items survive.  Few queries take the fp32 stage 1, many the
    8-bit pre-filter (nine: one of its second eight; 27: a last pass of eleven)."""
    torch, b = gpu
    N, d, m = 4_300_001, 24, 3 if codes == "equal" else 256
    gen = torch.Generator(device="cuda")
    gen.manual_seed(100 * K + Kf)
    cb = torch.randn((K, m, d), device="cuda", generator=gen) * torch.tensor([0.8 ** k for k in range(K)], device="cuda")[:, None, None]
    c = torch.randint(0, m, (K, N), dtype=torch.uint8, device="cuda", generator=gen)
    if codes == "clustered":
        centres = torch.randint(0, m, (Kf, 50), dtype=torch.uint8, device="cuda", generator=gen)
        c[:Kf] = centres[:, torch.randint(0, 50, (N,), device="cuda", generator=gen)]
    if codes == "far":
        cb[:2, :128] *= 0.1                                       # the nearest codewords of a query near the origin
        c[:2] |= 128
    for Q in (2, 9, 27) if Kf > 2 else (2, 4):
        queries = (0.3 if codes == "far" else 1.5) * torch.randn((Q, d), device="cuda", generator=gen)
        queries[::2] += sum(cb[k][c[k, :Q].long()] for k in range(K))[::2]        # every other one near an item
        index = b.icq_index_create(cb.contiguous(), c, Kf)
        lut = torch.empty((Q, K, 256), device="cuda")
        b.icq_build_lut(index, queries, lut)
        P = sum(lut[:, k].index_select(1, c[k, :50_000].long()) for k in range(Kf))
        thr = torch.stack([P[q].kthvalue((1, 50, 500, 15_000)[q % 4]).values for q in range(Q)])
        if Q > 4:
            thr[4], thr[5], thr[6] = float("inf"), float("-inf"), float("nan")

        def out():
            return torch.empty((Q, topk), dtype=torch.int32, device="cuda"), torch.empty((Q, topk), device="cuda"), torch.empty((Q,), dtype=torch.int32, device="cuda")
        ids, dist, count = out()
        ws = torch.empty(b.icq_workspace_bytes(index, Q, N, topk), dtype=torch.uint8, device="cuda")
        b.icq_search(index, queries, thr, N, topk, ids, dist, count, ws)
        want_ids, want_dist, want_count = out()
        cand = torch.empty((Q, N), dtype=torch.int32, device="cuda")
        b.icq_scan_fast(index, lut, thr, cand, None, want_count, ws)
        b.icq_refine(index, lut, cand, None, want_count, topk, want_ids, want_dist, ws)
        torch.cuda.synchronize()
        assert torch.equal(count, want_count)
        assert torch.equal(dist, want_dist) and torch.equal(ids, want_ids)
        del index, ws, cand


@pytest.mark.parametrize("K,Kf,topk,codes,mode,share,cap", [
    (16, 4, 100, "late", 0, 0.01, 8192), (16, 4, 512, "far", 0, 0.05, 40960), (16, 4, 100, "far", 1, 0.01, 8192), (12, 3, 100, "far", 0, 0.1, 12288),
    (16, 3, 10, "late", 0, 0.005, 2048), (8, 4, 100, "late", 1, 0.01, 8192), (8, 2, 100, "far", 0, 0.01, 8192), (4, 2, 50, "far", 0, 0.02, 8192),
    (6, 1, 100, "flat", 0, 0.3, 40960), (16, 2, 100, "flat", 0, 0.01, 8192)])
def test_search_from_hit_bits_is_complete_where_cap_is_below_the_survivors(gpu, K, Kf, topk, codes, mode, share, cap):
    """The bound before stage 2 keeps what is written within `cap` keys a query also where the nearest runs say nothing of the neighbours:
    first codebooks that tell little ("late": the first two a third of the next two; "flat": all of one size) and runs that are
    empty or do not survive ("far").  `cap` holds fewer keys than there are survivors, and than reach the bound of the nearest runs (late, far), but more than
    128 topk, or a 64th of the survivors where that is more: the lists are those of the staged calls with room for all, bit for bit."""
    torch, b = gpu
    N, d, m, Q = 4_300_001, 24, 256, 12 if Kf > 2 else 3
    scale = [1.0] * K if codes == "flat" else [0.8 ** k for k in range(K)] if codes == "far" else [0.3, 0.3] + [1.0] * 2 + [0.5] * (K - 4)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1000 * K + 10 * Kf + mode)
    cb = torch.randn((K, m, d), device="cuda", generator=gen) * torch.tensor(scale, device="cuda")[:, None, None]
    c = torch.randint(0, m, (K, N), dtype=torch.uint8, device="cuda", generator=gen)
    if codes == "far":                                            # no item has a codeword near a query's first ones
        cb[:min(2, Kf), :128] *= 0.1
        c[:min(2, Kf)] |= 128
    index = b.icq_index_create(cb.contiguous(), c, Kf)
    b.icq_index_set_scan_mode(index, mode)
    queries = 0.3 * torch.randn((Q, d), device="cuda", generator=gen)
    if codes != "far":
        queries += sum(cb[k][c[k, :Q].long()] for k in range(K))
    lut = torch.empty((Q, K, 256), device="cuda")
    b.icq_build_lut(index, queries, lut)
    P = sum(lut[:, k].index_select(1, c[k, :100_000].long()) for k in range(Kf))
    thr = P.kthvalue(int(share * 100_000), dim=1).values.contiguous()

    def out():
        return torch.empty((Q, topk), dtype=torch.int32, device="cuda"), torch.empty((Q, topk), device="cuda"), torch.empty((Q,), dtype=torch.int32, device="cuda")
    ids, dist, count = out()
    ws = torch.empty(b.icq_workspace_bytes(index, Q, cap, topk), dtype=torch.uint8, device="cuda")
    b.icq_search(index, queries, thr, cap, topk, ids, dist, count, ws)
    want_ids, want_dist, want_count = out()
    cand = torch.empty((Q, N), dtype=torch.int32, device="cuda")
    ws = torch.empty(b.icq_workspace_bytes(index, Q, N, topk), dtype=torch.uint8, device="cuda")
    b.icq_scan_fast(index, lut, thr, cand, None, want_count, ws)
    b.icq_refine(index, lut, cand, None, want_count, topk, want_ids, want_dist, ws)
    torch.cuda.synchronize()
    assert int(count.min()) > cap
    assert torch.equal(count, want_count)
    assert torch.equal(dist, want_dist) and torch.equal(ids, want_ids)


@pytest.mark.parametrize("K,Kf,N,Q,ratio,share", [
    (16, 4, 4_300_001, 5, 1.0, 0.01), (16, 4, 4_300_001, 40, 0.87, 0.02), (12, 3, 4_300_001, 40, 0.95, 0.1), (9, 4, 4_300_001, 12, 4.0, 0.003),
    (16, 3, 1_100_003, 160, 0.8, 0.3), (13, 4, 1_100_003, 140, 1.0, 0.01), (16, 4, 20_000_003, 60, 0.8, 0.004), (16, 4, 20_000_003, 60, 0.9, 0.004),
    (16, 4, 4_300_001, 40, 0.8, 0.01), (10, 3, 4_300_001, 4, 0.8, 0.01)])
def test_search_of_whole_and_half_records_equals_id_order(gpu, K, Kf, N, Q, ratio, share):
    """Over the pair ordering with 9 to 16 codebooks stage 2 reads first halves where the codebooks shrink, whole records where they do
    not: the lists and counts of the walk in id order, bit for bit.  Every third query far from all items (nothing near bounds its
    result), every seventh threshold infinite or below everything."""
    torch, b = gpu
    d, topk, cap = 24, 100, N
    gen = torch.Generator(device="cuda")
    gen.manual_seed(K * Q)
    cb = torch.randn((K, 256, d), device="cuda", generator=gen) * torch.tensor([ratio ** (k if ratio < 2 else k >= 8) for k in range(K)], device="cuda")[:, None, None]
    codes = torch.randint(0, 256, (K, N), dtype=torch.uint8, device="cuda", generator=gen)
    index = b.icq_index_create(cb.contiguous(), codes, Kf)
    queries = sum(cb[k][codes[k, :Q].long()] for k in range(K)) + 0.2 * torch.randn((Q, d), device="cuda", generator=gen)
    queries[::3] *= 3.0
    lut = torch.empty((Q, K, 256), device="cuda")
    b.icq_build_lut(index, queries, lut)
    P = sum(lut[:, k].index_select(1, codes[k, :20_000].long()) for k in range(Kf))
    thr = P.kthvalue(int(share * 20_000), dim=1).values.contiguous()
    thr[1::14], thr[6::14] = float("-inf"), float("inf") if N < 2_000_000 else thr[6::14] * 1.05
    got = []
    for mode in (0, 1):
        b.icq_index_set_scan_mode(index, mode)
        ids = torch.empty((Q, topk), dtype=torch.int32, device="cuda")
        dist = torch.empty((Q, topk), device="cuda")
        count = torch.empty((Q,), dtype=torch.int32, device="cuda")
        ws = torch.empty(b.icq_workspace_bytes(index, Q, cap, topk), dtype=torch.uint8, device="cuda")
        b.icq_search(index, queries, thr, cap, topk, ids, dist, count, ws)
        torch.cuda.synchronize()
        got.append((ids, dist, count))
    b.icq_index_set_scan_mode(index, 0)
    assert b.icq_index_scan_positions(index, Q) > N
    for x, y in zip(*got):
        assert torch.equal(x, y)


@pytest.mark.parametrize("N", [1 << 22, (1 << 22) + 1, 129 * 32768])
@pytest.mark.parametrize("K,Kf,mode", [(8, 2, 0), (16, 4, 1), (4, 3, 1)])
def test_search_from_hit_bits_in_id_order_from_four_million_items_on(gpu, N, K, Kf, mode):
    """From 2^22 items on (128 chunks) every search from hit bits is bounded before stage 2, in id order too; below, only calls of 32
    queries or more keep hit bits, behind the pre-filter, and are not.  Lists and counts are those of the staged calls, bit for bit."""
    torch, b = gpu
    d, topk = 12, 30
    gen = torch.Generator(device="cuda")
    gen.manual_seed(N + K)
    cb = torch.randn((K, 256, d), device="cuda", generator=gen) * torch.tensor([0.8 ** k for k in range(K)], device="cuda")[:, None, None]
    codes = torch.randint(0, 256, (K, N), dtype=torch.uint8, device="cuda", generator=gen)
    for n, Qs in ((N, (1, 4) if Kf == 2 else (1, 5, 6)), (N // 4, (32,) if Kf > 2 else ())):
        part = codes[:, :n].contiguous()
        index = b.icq_index_create(cb.contiguous(), part, Kf)
        b.icq_index_set_scan_mode(index, mode)
        for Q in Qs:
            queries = sum(cb[k][part[k, :Q].long()] for k in range(K)) + 0.1 * torch.randn((Q, d), device="cuda", generator=gen)
            lut = torch.empty((Q, K, 256), device="cuda")
            b.icq_build_lut(index, queries, lut)
            P = sum(lut[:, k].index_select(1, part[k, :20_000].long()) for k in range(Kf))
            thr = P.kthvalue(200, dim=1).values.contiguous()
            got = []
            for staged in (False, True):
                ids = torch.empty((Q, topk), dtype=torch.int32, device="cuda")
                dist = torch.empty((Q, topk), device="cuda")
                count = torch.empty((Q,), dtype=torch.int32, device="cuda")
                ws = torch.empty(b.icq_workspace_bytes(index, Q, n, topk), dtype=torch.uint8, device="cuda")
                if staged:
                    cand = torch.empty((Q, n), dtype=torch.int32, device="cuda")
                    b.icq_scan_fast(index, lut, thr, cand, None, count, ws)
                    b.icq_refine(index, lut, cand, None, count, topk, ids, dist, ws)
                else:
                    b.icq_search(index, queries, thr, n, topk, ids, dist, count, ws)
                torch.cuda.synchronize()
                got.append((ids, dist, count))
            for x, y in zip(*got):
                assert torch.equal(x, y), (n, Q)


@pytest.mark.parametrize("m,N,Q,pairs", [(256, 600_000, 2000, False), (256, 740_000, 2000, False), (256, 1_000_000, 200, True), (64, 600_000, 1000, True), (256, 1_000_000, 31, False)])
def test_the_pair_ordering_is_taken_where_its_padding_is_small(gpu, m, N, Q, pairs):
    """Searches of many queries over half a million to four million items walk the pair ordering unless its runs' padding to 16 makes
    it more than half as long again as the items (7.5e5 items in 65536 runs)."""
    torch, b = gpu
    gen = torch.Generator(device="cuda")
    gen.manual_seed(m + N)
    cb = torch.randn((8, m, 8), device="cuda", generator=gen)
    index = b.icq_index_create(cb, torch.randint(0, m, (8, N), dtype=torch.uint8, device="cuda", generator=gen), 4)
    assert (b.icq_index_scan_positions(index, Q) > N) == pairs
    b.icq_index_set_scan_mode(index, b.ICQ_SCAN_GROUPED)
    assert b.icq_index_scan_positions(index, Q) > N


@pytest.mark.parametrize("K,Kf,N,Q,topk", [(16, 4, 1_000_003, 190, 100), (12, 3, 2_000_001, 40, 300), (8, 4, 600_011, 900, 10)])
def test_search_of_many_queries_over_the_pair_ordering_equals_id_order(gpu, K, Kf, N, Q, topk):
    """Many queries over an index of half a million to four million items walk the pair ordering, the stage-2 bound first: the
    lists and counts of the walk in id order, bit for bit, for thresholds that let all, nothing, a hundredth or a tenth
    through; and in a workspace that holds the bits of id order only (or whole calls of fewer queries) the same again."""
    torch, b = gpu
    d = 20
    gen = torch.Generator(device="cuda")
    gen.manual_seed(N)
    cb = torch.randn((K, 200, d), device="cuda", generator=gen) * torch.tensor([0.8 ** k for k in range(K)], device="cuda")[:, None, None]
    codes = torch.randint(0, 200, (K, N), dtype=torch.uint8, device="cuda", generator=gen)
    index = b.icq_index_create(cb.contiguous(), codes, Kf)
    queries = 1.5 * torch.randn((Q, d), device="cuda", generator=gen)
    queries[::2] += sum(cb[k][codes[k, :Q].long()] for k in range(K))[::2]
    lut = torch.empty((Q, K, 256), device="cuda")
    b.icq_build_lut(index, queries, lut)
    P = sum(lut[:, k].index_select(1, codes[k, :20_000].long()) for k in range(Kf))
    thr = P.kthvalue(200, dim=1).values.contiguous()
    thr[0::7] = P.kthvalue(2000, dim=1).values[0::7]
    thr[1], thr[2], thr[3] = float("inf"), float("-inf"), float("nan")
    cap = N

    def run(bytes_, mode):
        b.icq_index_set_scan_mode(index, mode)
        ids = torch.empty((Q, topk), dtype=torch.int32, device="cuda")
        dist = torch.empty((Q, topk), device="cuda")
        count = torch.empty((Q,), dtype=torch.int32, device="cuda")
        b.icq_search(index, queries, thr, cap, topk, ids, dist, count, torch.empty(bytes_, dtype=torch.uint8, device="cuda"))
        torch.cuda.synchronize()
        return ids, dist, count
    full = b.icq_workspace_bytes(index, Q, cap, topk)
    want = run(full, 1)
    assert int(want[2][1]) == N and int(want[2][2]) == 0
    b.icq_index_set_scan_mode(index, 0)
    assert b.icq_index_scan_positions(index, Q) > N
    bits = Q * (b.icq_index_scan_positions(index, Q) - N) // 8
    for bytes_ in (full, full - bits // 2) + ((full // 2,) if Q > 128 else ()):        # (64 queries are not cut further)
        for x, y in zip(run(bytes_, 0), want):
            assert torch.equal(x, y), bytes_


@pytest.mark.parametrize("K,d", [(1, 1), (4, 17), (8, 100), (8, 128), (8, 132), (8, 64), (16, 33), (3, 260)])
def test_tables_of_few_queries_equal_those_of_many(gpu, K, d):
    """Few queries' tables come from wavefronts of their own, many queries' from blocks that stage in LDS: the same sums in the
    same order, hence the same bits -- also of rows that are not 16-byte aligned, and with infinities and NaN."""
    torch, b = gpu
    gen = torch.Generator(device="cuda")
    gen.manual_seed(d)
    cb = torch.randn((K, 200, d), device="cuda", generator=gen)
    index = b.icq_index_create(cb, torch.empty((K, 0), dtype=torch.uint8, device="cuda"), 1)
    many = 32 * (6 * 256 // (8 * K)) + 65
    flat = torch.randn((many * d + 1,), device="cuda", generator=gen)
    queries = flat[1:].view(many, d)
    queries[5, d - 1], queries[7, 0], queries[40, d // 2] = float("inf"), float("nan"), -float("inf")
    want = torch.empty((many, K, 256), device="cuda")
    b.icq_build_lut(index, queries, want)
    for first, Q in ((0, 1), (0, 31), (3, 32), (5, 33), (1, 65)):
        for aligned in (False, True):
            q = queries[first:first + Q]
            q = q.clone() if aligned else q.contiguous()
            got = torch.full((Q, K, 256), 7.0, device="cuda")
            b.icq_build_lut(index, q, got)
            assert torch.equal(got.view(torch.int32), want[first:first + Q].view(torch.int32)) or \
                ((got == want[first:first + Q]) | (got.isnan() & want[first:first + Q].isnan())).all()


@pytest.mark.parametrize("K,Kf,N,Q", [(4, 3, 4095, 7), (4, 1, 4096, 1), (8, 2, 4097, 3), (12, 4, 8191, 40), (16, 4, 8193, 350), (16, 3, 1_000_003, 2)])
def test_small_index_in_one_kernel_equals_the_streamed_form(gpu, K, Kf, N, Q):
    """Both stages of a small index in one kernel, 4096 items a step, against the forms for larger ones: the same additions, the
    same lists, distances and counts bit for bit."""
    torch, b = gpu
    gen = torch.Generator(device="cuda")
    gen.manual_seed(N)
    d, topk = 24, 33
    cb = torch.randn((K, 256, d), device="cuda", generator=gen) * torch.tensor([0.7 ** k for k in range(K)], device="cuda")[:, None, None]
    codes = torch.randint(0, 256, (K, N), dtype=torch.uint8, device="cuda", generator=gen)
    index = b.icq_index_create(cb.contiguous(), codes, Kf)
    queries = torch.randn((Q, d), device="cuda", generator=gen)
    lut = torch.empty((Q, K, 256), device="cuda")
    b.icq_build_lut(index, queries, lut)
    P = sum(lut[:, k].index_select(1, codes[k, :4000].long()) for k in range(Kf))
    thr = P.kthvalue(200, dim=1).values.contiguous()
    thr[0] = float("inf") if N < 10_000 else thr[0]
    out = []
    for mode in (b.ICQ_SCAN_AUTO, b.ICQ_SCAN_STREAMED):
        b.icq_index_set_scan_mode(index, mode)
        ids, dist = torch.empty((Q, topk), dtype=torch.int32, device="cuda"), torch.empty((Q, topk), device="cuda")
        count = torch.empty((Q,), dtype=torch.int32, device="cuda")
        ws = torch.empty(b.icq_workspace_bytes(index, Q, N, topk), dtype=torch.uint8, device="cuda")
        b.icq_search(index, queries, thr, N, topk, ids, dist, count, ws)
        out.append((ids, dist, count))
    torch.cuda.synchronize()
    for x, y in zip(*out):
        assert torch.equal(x, y)


@pytest.mark.parametrize("K,m,N,Q,clustered", [(8, 256, 3_000_001, 1, False), (4, 256, 1_500_001, 2, True), (12, 200, 1_100_000, 3, False),
                                               (8, 256, 4_300_000, 4, True), (8, 256, 4_300_000, 1, False)])
def test_search_of_few_queries_grouped_by_tuple(gpu, K, m, N, Q, clustered):
    """One to four queries over an index grouped by two fast codes, next to the lines between the small-index kernel, lists and hit
    bits: lists, distances and counts of the streamed form, bit for bit; no survivors, too, and all of them, where the
    call must not take long either (the grouped kernel with its blocks per query took 10 to 25 times the streamed form's time)."""
    torch, b = gpu
    gen = torch.Generator(device="cuda")
    gen.manual_seed(N + Q)
    d, topk = 16, 100
    cb = torch.randn((K, m, d), device="cuda", generator=gen) * torch.tensor([0.6 ** k for k in range(K)], device="cuda")[:, None, None]
    codes = torch.randint(0, m, (K, N), dtype=torch.uint8, device="cuda", generator=gen)
    if clustered:
        codes[:2, : N // 2] = codes[:2, :500].repeat(1, N // 1000 + 1)[:, : N // 2]
    index = b.icq_index_create(cb.contiguous(), codes, 2)
    queries = torch.randn((Q, d), device="cuda", generator=gen)
    lut = torch.empty((Q, K, 256), device="cuda")
    b.icq_build_lut(index, queries, lut)
    P = sum(lut[:, k].index_select(1, codes[k].long()) for k in range(2))
    for thr in (P.kthvalue(N // 200, dim=1).values.contiguous(), torch.full((Q,), -1.0, device="cuda"), torch.full((Q,), float("inf"), device="cuda")):
        cap = N if torch.isinf(thr[0]) else N // 10
        out, times = [], []
        for mode in (b.ICQ_SCAN_AUTO, b.ICQ_SCAN_STREAMED):
            b.icq_index_set_scan_mode(index, mode)
            ids, dist = torch.empty((Q, topk), dtype=torch.int32, device="cuda"), torch.empty((Q, topk), device="cuda")
            count = torch.empty((Q,), dtype=torch.int32, device="cuda")
            ws = torch.empty(b.icq_workspace_bytes(index, Q, cap, topk), dtype=torch.uint8, device="cuda")
            best = float("inf")
            for _ in range(3):
                e0, e1 = torch.cuda.Event(True), torch.cuda.Event(True)
                e0.record()
                b.icq_search(index, queries, thr, cap, topk, ids, dist, count, ws)
                e1.record()
                torch.cuda.synchronize()
                best = min(best, e0.elapsed_time(e1))
            out.append((ids, dist, count))
            times.append(best)
        for x, y in zip(*out):
            assert torch.equal(x, y)
        assert times[0] < 3 * times[1] + 0.05, times


def test_op_counts_match_oracle(gpu):
    torch, b = gpu
    cfg = small("C1", 5_000, 300)
    g = Gpu(gpu, cfg)
    rng = np.random.default_rng(9)
    refined = rng.integers(0, 5_001, size=300).astype(np.int32)
    refined[7] = 0
    refined[8] = 5_000
    ops = torch.empty((300,), dtype=torch.int64, device="cuda")
    summary = torch.empty((4,), dtype=torch.float64, device="cuda")
    b.icq_op_counts(g.index, _dev(torch, refined), ops, summary)
    torch.cuda.synchronize()
    o_ops, o_sum = orc.op_counts(5_000, cfg["K"], cfg["Kf"], refined.astype(np.int64), cfg["K"] * 8.0)
    assert np.array_equal(ops.cpu().numpy(), o_ops.astype(np.int64))
    assert np.array_equal(summary.cpu().numpy(), o_sum)


# ------------------------------------------------------------------ encoding
def _check_encoding(cb, x, codes_gpu, codes_orc):
    """Greedy choices level by level, given the GPU's own earlier choices: the chosen codeword must
    be a nearest one of the residual up to the tolerance (fp32 scores may order near-ties differently)."""
    K, m, d = cb.shape
    cb64, r = cb.astype(np.float64), x.astype(np.float64).copy()
    n = np.arange(x.shape[0])
    for k in range(K):
        d2 = (r * r).sum(axis=1)[:, None] - 2.0 * r @ cb64[k].T + (cb64[k] ** 2).sum(axis=1)[None, :]
        chosen = d2[n, codes_gpu[k]]
        best = d2.min(axis=1)
        assert (chosen <= best + tol(best)).all(), "level %d: a clearly nearer codeword exists" % k
        r -= cb64[k][codes_gpu[k]]
    same = (codes_gpu == codes_orc).all(axis=0).mean()
    assert same >= 0.98, same


@pytest.mark.parametrize("K,m,d,N", [(8, 256, 128, 5_000), (4, 256, 32, 1_000), (16, 256, 96, 777),
                                      (3, 100, 17, 130), (1, 256, 8, 64), (2, 7, 5, 1)])
def test_encode_matches_oracle(gpu, K, m, d, N):
    torch, b = gpu
    rng = np.random.default_rng(K * 1000 + d)
    cb = (rng.standard_normal((K, m, d)) * (0.6 ** np.arange(K))[:, None, None]).astype(np.float32)
    src = rng.integers(0, m, size=(K, N))
    x = sum(cb[k][src[k]] for k in range(K)) + 0.05 * rng.standard_normal((N, d)).astype(np.float32)
    x = np.ascontiguousarray(x, dtype=np.float32)
    index = b.icq_index_create(_dev(torch, cb), torch.empty((K, 0), dtype=torch.uint8, device="cuda"), min(2, K))
    codes = torch.full((K, N), 255, dtype=torch.uint8, device="cuda")
    ws = torch.empty(b.icq_encode_workspace_bytes(index, N), dtype=torch.uint8, device="cuda")
    b.icq_encode(index, _dev(torch, x), codes, ws)
    torch.cuda.synchronize()
    codes = codes.cpu().numpy()
    assert (codes < m).all()
    _check_encoding(cb, x, codes, orc.encode(cb, x))
    with pytest.raises(b.IcqError):
        b.icq_encode(index, _dev(torch, x), torch.empty((K, N), dtype=torch.uint8, device="cuda"), ws[:128])


@pytest.mark.parametrize("m,d,N,sweeps", [
    (256, 32, 40_000, 1), (33, 33, 33, 1), (64, 64, 40_000, 0), (65, 96, 33_000, 1), (31, 97, 70, 1), (129, 128, 33_000, 1),
    (256, 129, 65, 1), (97, 192, 33_000, 1), (225, 193, 17, 1), (256, 256, 16_500, 1), (160, 256, 63, 1), (1, 130, 200, 1),
    (256, 257, 100, 1), (200, 300, 16_400, 0), (256, 384, 33_000, 1), (96, 385, 129, 1), (256, 512, 33_000, 0), (255, 512, 64, 1),
    (256, 512, 33_000, 1), (256, 513, 130, 1),
])
def test_encode_over_the_forms_of_its_kernels(gpu, m, d, N, sweeps):
    """The numbers of 32-wide slices the register form is built for and those next to them, both of its block sizes, the
    residuals in memory beyond; codebooks that end inside a chunk of 32 codewords.  x is drawn, not reconstructed: every level
    has to decide.  Judged on a sample as in test_encode_at_the_edges_of_its_forms: fp32 scores are sums of d terms of up to
    ||r||^2 + ||c||^2, each off by 2^-23 of it at most."""
    torch, b = gpu
    K = 3
    rng = np.random.default_rng(d * 1000 + m)
    cb = (rng.standard_normal((K, m, d)) * (0.7 ** np.arange(K))[:, None, None]).astype(np.float32)
    x = rng.standard_normal((N, d)).astype(np.float32)
    index = b.icq_index_create(_dev(torch, cb), torch.empty((K, 0), dtype=torch.uint8, device="cuda"), 1)
    ws = torch.empty(b.icq_encode_workspace_bytes(index, N), dtype=torch.uint8, device="cuda")
    codes = torch.full((K, N), 255, dtype=torch.uint8, device="cuda")
    xd = _dev(torch, x)
    b.icq_encode(index, xd, codes, ws)
    refined, changed = codes.clone(), torch.full((max(1, sweeps),), 7, dtype=torch.int32, device="cuda")
    b.icq_encode_refine(index, xd, refined, sweeps, changed if sweeps else None, ws)
    torch.cuda.synchronize()
    first, second = codes.cpu().numpy(), refined.cpu().numpy()
    assert (first < m).all() and (second < m).all()
    if sweeps:
        assert int(changed[0]) == int((first != second).sum())
    at = np.unique(np.concatenate([np.arange(min(N, 150)), np.arange(max(0, N - 150), N), rng.integers(0, N, 300)]))
    cb64, xs, n, eps = cb.astype(np.float64), x[at].astype(np.float64), np.arange(at.size), d * 2.0 ** -23

    def judge(r, k, chosen):
        d2 = (r * r).sum(axis=1)[:, None] - 2.0 * r @ cb64[k].T + (cb64[k] ** 2).sum(axis=1)[None]
        slack = eps * ((r * r).sum(axis=1) + (cb64[k] ** 2).sum(axis=1).max())
        assert (d2[n, chosen] <= d2.min(axis=1) + slack).all(), "level %d: a clearly nearer codeword exists" % k
    f, s = first[:, at], second[:, at]
    r = xs.copy()
    for k in range(K):
        judge(r, k, f[k])
        r = r - cb64[k][f[k]]
    for k in range(K if sweeps else 0):
        state = np.concatenate([s[:k], f[k:]])
        judge(xs - sum(cb64[l][state[l]] for l in range(K) if l != k), k, s[k])


@pytest.mark.parametrize("d,N", [(32, 400), (64, 40_000), (96, 33_000), (128, 700), (192, 300), (256, 33_000), (300, 200), (512, 130)])
@pytest.mark.parametrize("equal,wild", [(8, 0), (9, 128), (16, 7), (32, 16), (33, 300), (128, 2)])
def test_encode_where_lists_of_candidates_say_little(gpu, d, N, equal, wild):
    """Up to eight or 32 candidates are looked at one by one, more are scored with all other codewords on the matrix cores, and so
    are items that have no bound, a few of them by themselves: codebooks of `equal` equal codewords each, every `wild`-th vector
    with a component that is infinite.  Among equal codewords the first is taken, refinement keeps a current one; the
    vectors next to a wild one are not disturbed.  Judged as in test_encode_over_the_forms_of_its_kernels."""
    torch, b = gpu
    K, m = 3, 256
    few = m // equal
    rng = np.random.default_rng(d * 1000 + equal)
    cb = (rng.standard_normal((K, few, d)) * (0.7 ** np.arange(K))[:, None, None]).astype(np.float32)
    cb = np.concatenate([cb] * (m // few + 1), axis=1)[:, :m]
    x = rng.standard_normal((N, d)).astype(np.float32)
    strange = np.arange(0, N, wild) if wild else np.zeros(0, dtype=int)
    plain = np.setdiff1d(np.arange(N), strange)
    x[strange, 0] = np.inf
    index = b.icq_index_create(_dev(torch, cb), torch.empty((K, 0), dtype=torch.uint8, device="cuda"), 1)
    ws = torch.empty(b.icq_encode_workspace_bytes(index, N), dtype=torch.uint8, device="cuda")
    codes, changed = torch.empty((K, N), dtype=torch.uint8, device="cuda"), torch.empty((1,), dtype=torch.int32, device="cuda")
    xd = _dev(torch, x)
    b.icq_encode(index, xd, codes, ws)
    start = rng.integers(0, m, (K, N), dtype=np.uint8)
    refined = _dev(torch, start)
    b.icq_encode_refine(index, xd, refined, 1, changed, ws)
    torch.cuda.synchronize()
    first, second = codes.cpu().numpy(), refined.cpu().numpy()
    assert (first < few).all()
    assert ((second < few) | (second == start)).all() and int(changed[0]) == int((second != start).sum())
    # an infinite component: the score is -inf where the codeword has that sign, the first of those is taken
    up = cb[0][:, 0] > 0
    if up.any():
        assert (first[0, strange] == np.argmax(up)).all()
        assert (second[0, strange] == np.where(up[start[0, strange]], start[0, strange], np.argmax(up))).all()
    at = plain[np.unique(np.concatenate([np.arange(min(plain.size, 150)), np.arange(max(0, plain.size - 150), plain.size), rng.integers(0, plain.size, 300)]))]
    cb64, xs, n, eps = cb.astype(np.float64), x[at].astype(np.float64), np.arange(at.size), d * 2.0 ** -23

    def judge(r, k, chosen):
        d2 = (r * r).sum(axis=1)[:, None] - 2.0 * r @ cb64[k].T + (cb64[k] ** 2).sum(axis=1)[None]
        slack = eps * ((r * r).sum(axis=1) + (cb64[k] ** 2).sum(axis=1).max())
        assert (d2[n, chosen] <= d2.min(axis=1) + slack).all(), "level %d: a clearly nearer codeword exists" % k
    r = xs.copy()
    for k in range(K):
        judge(r, k, first[k, at])
        r = r - cb64[k][first[k, at]]
    for k in range(K):
        state = np.concatenate([second[:k, at], start[k:, at]])
        judge(xs - sum(cb64[l][state[l]] for l in range(K) if l != k), k, second[k, at])


def test_encode_refine_does_not_take_long_over_a_few_wild_vectors(gpu):
    """One vector in 128 without a bound costs its wavefront a look at each codeword, not its neighbours a contraction in
    fp32 (with which a sweep took 5.6 times as long as without such vectors; 1.6 now)."""
    torch, b = gpu
    N, d, K = 100_000, 128, 8
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    cb = torch.randn((K, 256, d), device="cuda", generator=gen) * torch.tensor([0.6 ** k for k in range(K)], device="cuda")[:, None, None]
    index = b.icq_index_create(cb.contiguous(), torch.empty((K, 0), dtype=torch.uint8, device="cuda"), 1)
    x = torch.randn((N, d), device="cuda", generator=gen)
    y = x.clone()
    y[::128, 3] = float("inf")
    ws = torch.empty(b.icq_encode_workspace_bytes(index, N), dtype=torch.uint8, device="cuda")
    start = torch.randint(0, 256, (K, N), dtype=torch.uint8, device="cuda", generator=gen)
    times = []
    for v in (x, y):
        best = float("inf")
        for _ in range(6):
            codes = start.clone()
            e0, e1 = torch.cuda.Event(True), torch.cuda.Event(True)
            e0.record()
            b.icq_encode_refine(index, v, codes, 4, None, ws)
            e1.record()
            torch.cuda.synchronize()
            best = min(best, e0.elapsed_time(e1))
        times.append(best)
    assert times[1] < 3.5 * times[0], times


@pytest.mark.parametrize("d", [160, 256, 384, 512])
def test_encode_with_few_codebooks_and_then_many(gpu, d):
    """The register form's LDS grows with the number of codebooks: 64 of them after 2, on one kernel.  Greedy assignment takes
    the codebooks one after another, so the first codes of the long list are those of the short one."""
    torch, b = gpu
    rng = np.random.default_rng(d)
    cb = (rng.standard_normal((64, 256, d)) * (0.9 ** np.arange(64))[:, None, None]).astype(np.float32)
    x = _dev(torch, rng.standard_normal((130, d)).astype(np.float32))
    out = []
    for K in (2, 64):
        index = b.icq_index_create(_dev(torch, cb[:K]), torch.empty((K, 0), dtype=torch.uint8, device="cuda"), 1)
        ws = torch.empty(b.icq_encode_workspace_bytes(index, 130), dtype=torch.uint8, device="cuda")
        codes = torch.empty((K, 130), dtype=torch.uint8, device="cuda")
        b.icq_encode(index, x, codes, ws)
        refined = codes.clone()
        b.icq_encode_refine(index, x, refined, 1, None, ws)
        err = [torch.empty((130,), dtype=torch.float64, device="cuda") for _ in range(2)]
        b.icq_quantization_error(index, x, codes, err[0])
        b.icq_quantization_error(index, x, refined, err[1])
        torch.cuda.synchronize()
        # a replaced sub-code is nearer up to the rounding of its fp32 score, a sum of d terms within ||v||^2 + ||c||^2
        slack = K * d * 2.0 ** -23 * ((x.double() ** 2).sum(1) + float((cb[0] ** 2).sum(1).max()))
        assert (err[1] <= err[0] + slack).all()
        out.append(codes.cpu().numpy())
    assert np.array_equal(out[0], out[1][:2])


@pytest.mark.parametrize("K,m,d,N,kind", [
    (3, 256, 128, 129, "plain"), (3, 256, 129, 257, "plain"),   # the residual in registers / in memory; blocks of 128 items
    (2, 200, 255, 130, "plain"), (2, 256, 960, 200, "plain"),   # an odd end of the last row; several slices
    (3, 256, 33, 300, "offset"), (2, 250, 200, 150, "offset"),  # half precision tells few codewords apart: both halves are taken
    (3, 256, 40, 300, "equal"), (2, 256, 150, 150, "equal"),    # thirteen equal codewords each: the indices decide
    (2, 256, 64, 130, "zero"), (2, 5, 3, 7, "equal"),
])
def test_encode_at_the_edges_of_its_forms(gpu, K, m, d, N, kind):
    """Every level's codeword is a nearest one of the residual the GPU's own earlier choices leave (tolerance of fp32
    scores: d roundings of terms up to ||r||^2 + ||c||^2), the smallest index among equal codewords; a sweep of
    refinement from there keeps what is not strictly nearer."""
    torch, b = gpu
    rng = np.random.default_rng(K * 100_000 + d * 10 + m)
    cb = rng.standard_normal((K, m, d)).astype(np.float32)
    if kind == "offset":            # far from the origin, close to each other
        cb = (3.0 + 0.01 * cb).astype(np.float32)
    if kind == "equal":             # index j holds the codeword of j mod (m // 13 + 1)
        cb = cb[:, np.arange(m) % (m // 13 + 1)].copy()
    if kind == "zero":
        cb[1] = 0.0
    x = (sum(cb[k][rng.integers(0, m, N)] for k in range(K)) + 0.01 * rng.standard_normal((N, d))).astype(np.float32)
    index = b.icq_index_create(_dev(torch, cb), torch.empty((K, 0), dtype=torch.uint8, device="cuda"), min(2, K))
    ws = torch.empty(b.icq_encode_workspace_bytes(index, N), dtype=torch.uint8, device="cuda")
    codes = torch.full((K, N), 255, dtype=torch.uint8, device="cuda")
    xd = _dev(torch, x)
    b.icq_encode(index, xd, codes, ws)
    refined = codes.clone()
    b.icq_encode_refine(index, xd, refined, 1, None, ws)
    torch.cuda.synchronize()
    first, second = codes.cpu().numpy(), refined.cpu().numpy()
    assert (first < m).all() and (second < m).all()
    cb64, n, eps = cb.astype(np.float64), np.arange(N), d * 2.0 ** -23

    def judge(r, k, chosen, old):
        d2 = ((r[:, None, :] - cb64[k][None]) ** 2).sum(axis=2)
        slack = eps * ((r * r).sum(axis=1) + (cb64[k] ** 2).sum(axis=1).max())
        assert (d2[n, chosen] <= d2.min(axis=1) + slack).all(), "level %d: a clearly nearer codeword exists" % k
        if kind == "equal":
            g = m // 13 + 1
            assert (np.where(chosen == old, 0, chosen) < g).all()      # a current codeword is kept, else the first of its equals
    r = x.astype(np.float64)
    for k in range(K):
        judge(r, k, first[k], -1)
        r = r - cb64[k][first[k]]
    for k in range(K):
        state = np.concatenate([second[:k], first[k:]])
        judge(x - sum(cb64[l][state[l]] for l in range(K) if l != k), k, second[k], first[k])
    if kind == "zero":
        assert (first[1] == 0).all() and (second[1] == 0).all()


@pytest.mark.parametrize("K,m,d", [(2, 256, 48), (2, 201, 176)])
def test_encode_of_vectors_beyond_the_halves_range(gpu, K, m, d):
    """An infinite component decides by its sign alone (scores of -inf: the smallest index among them, a current
    codeword kept), 1e24 by the products, NaN leaves index 0; the vectors beside them in the block stay what they are."""
    torch, b = gpu
    rng = np.random.default_rng(d)
    N, e = 150, 5
    cb = rng.standard_normal((K, m, d)).astype(np.float32)
    x = (sum(cb[k][rng.integers(0, m, N)] for k in range(K)) + 0.01 * rng.standard_normal((N, d))).astype(np.float32)
    x[3, e], x[4, e], x[70, e] = np.inf, -np.inf, np.nan
    x[[9, 140]] *= 1e24
    index = b.icq_index_create(_dev(torch, cb), torch.empty((K, 0), dtype=torch.uint8, device="cuda"), 1)
    ws = torch.empty(b.icq_encode_workspace_bytes(index, N), dtype=torch.uint8, device="cuda")
    codes = torch.full((K, N), 255, dtype=torch.uint8, device="cuda")
    xd = _dev(torch, x)
    b.icq_encode(index, xd, codes, ws)
    refined = codes.clone()
    b.icq_encode_refine(index, xd, refined, 1, None, ws)
    torch.cuda.synchronize()
    first, second = codes.cpu().numpy(), refined.cpu().numpy()
    plain = np.setdiff1d(np.arange(N), [3, 4, 70, 9, 140])
    r = x.astype(np.float64)
    for k in range(K):
        c = cb[k].astype(np.float64)
        assert first[k, 3] == np.argmax(c[:, e] > 0) and first[k, 4] == np.argmax(c[:, e] < 0) and first[k, 70] == 0
        for i in (9, 140):
            dot = c @ r[i]              # d roundings of terms up to ||r|| ||c||
            assert dot[first[k, i]] >= dot.max() - d * 2.0 ** -23 * np.linalg.norm(r[i]) * np.linalg.norm(c, axis=1).max()
        d2 = ((r[plain][:, None, :] - c[None]) ** 2).sum(axis=2)
        slack = d * 2.0 ** -23 * ((r[plain] ** 2).sum(axis=1) + (c ** 2).sum(axis=1).max())
        assert (d2[np.arange(plain.size), first[k, plain]] <= d2.min(axis=1) + slack).all()
        r = r - c[first[k]]
    assert (first[:, [3, 4, 70]] == second[:, [3, 4, 70]]).all()


@pytest.mark.parametrize("N,d", [(1, 129), (2, 300), (129, 200), (130, 128), (257, 960), (383, 64)])
def test_encode_of_a_last_block_with_few_items(gpu, N, d):
    """The places past the last item take part in nothing: the last items get what they get in the middle of full blocks,
    from vectors far from any tie, and the oracle's codes; twice the same, and with sweeps of refinement."""
    torch, b = gpu
    K, m, more = 4, 256, 512
    rng = np.random.default_rng(N * 1000 + d)
    cb = (rng.standard_normal((K, m, d)) * (0.5 ** np.arange(K))[:, None, None]).astype(np.float32)
    src = rng.integers(0, m, (K, more))
    x = (sum(cb[k][src[k]] for k in range(K)) + 0.001 * rng.standard_normal((more, d))).astype(np.float32)
    x[:N] *= 1.0 + 0.001 * rng.random((N, 1), dtype=np.float32)
    index = b.icq_index_create(_dev(torch, cb), torch.empty((K, 0), dtype=torch.uint8, device="cuda"), 1)
    out = []
    for n in (N, more, N):
        ws = torch.empty(b.icq_encode_workspace_bytes(index, n), dtype=torch.uint8, device="cuda")
        codes, changed = torch.full((K, n), 255, dtype=torch.uint8, device="cuda"), torch.full((2,), -1, dtype=torch.int32, device="cuda")
        b.icq_encode(index, _dev(torch, x[:n]), codes, ws)
        start = _dev(torch, rng.integers(0, m, (K, n), dtype=np.uint8) if not out else out[0][2][:, :n] if n == N else
                     np.concatenate([out[0][2], rng.integers(0, m, (K, n - N), dtype=np.uint8)], axis=1))
        refined = start.clone()
        b.icq_encode_refine(index, _dev(torch, x[:n]), refined, 2, changed, ws)
        torch.cuda.synchronize()
        out.append([t.cpu().numpy() for t in (codes, refined, start, changed)])
    want = orc.encode(cb, x[:N])
    for o in out:
        assert np.array_equal(o[0][:, :N], want) and np.array_equal(o[1][:, :N], out[0][1])
    assert np.array_equal(out[0][3], out[2][3]) and out[0][3][0] <= K * N


@pytest.mark.parametrize("m,d", [(2, 2), (5, 40), (201, 128), (256, 130)])
def test_encode_where_the_halves_overflow_for_few_codewords(gpu, m, d):
    """Vectors whose halves are infinite, in a codebook in which few products then are +inf: these decide nothing.  1e30
    in two components meets (1, -0.5) and (0.1, 0.1): 0.5e30 against 0.2e30, but inf - inf against inf in halves.  An
    infinite component is decided by the codeword's sign there, also where the codeword is too small for a half.  NaN of
    either sign: index 0, a current codeword kept."""
    torch, b = gpu
    K, N = 2, 140
    rng = np.random.default_rng(m * 1000 + d)
    cb = np.full((K, m, d), -1.0, np.float32)              # -1e30 - 1e30 and -inf: never the best
    cb[:, :, 2:] = 0.01 * rng.standard_normal((K, m, max(d - 2, 0))).astype(np.float32)
    cb[:, m - 1, :2] = 0.1, 0.1
    cb[:, m - 2, :2] = 1.0, -0.5
    x = np.zeros((N, d), np.float32)
    x[:, 0] = -1.0                                         # plain vectors around them
    x[7, :2] = x[139, :2] = 1e30
    x[20, d - 1] = np.nan
    x[21, d - 1] = np.copysign(np.float32(np.nan), np.float32(-1.0))
    assert np.signbit(x[21, d - 1]) and not np.signbit(x[20, d - 1])
    tiny = cb.copy()                                       # the first positive one is no half: 1e-12 against 1
    tiny[:, :, 0] = -1.0
    tiny[:, m - 2, 0], tiny[:, m - 1, 0] = 1e-12, 1.0
    y = x.copy()
    y[:, 0] = -1.0
    y[7, 0] = y[139, 0] = np.inf

    def both(cb, x, start):
        index = b.icq_index_create(_dev(torch, cb), torch.empty((K, 0), dtype=torch.uint8, device="cuda"), 1)
        ws = torch.empty(b.icq_encode_workspace_bytes(index, N), dtype=torch.uint8, device="cuda")
        codes = torch.full((K, N), 255, dtype=torch.uint8, device="cuda")
        refined = torch.full((K, N), start, dtype=torch.uint8, device="cuda")
        b.icq_encode(index, _dev(torch, x), codes, ws)
        b.icq_encode_refine(index, _dev(torch, x), refined, 1, None, ws)
        torch.cuda.synchronize()
        return codes.cpu().numpy(), refined.cpu().numpy()
    first, second = both(cb, x, m - 1)
    assert (first[:, [7, 139]] == m - 2).all() and (second[:, [7, 139]] == m - 2).all()
    assert (first[:, 20:22] == 0).all() and (second[:, 20:22] == m - 1).all()
    first, second = both(tiny, y, 0)
    assert (first[:, [7, 139]] == m - 2).all()
    assert (second[:, [7, 139]] == (0 if m == 2 else m - 2)).all()


@pytest.mark.parametrize("m,distinct,d,N", [(256, 16, 40, 300), (256, 1, 128, 129), (200, 19, 130, 140), (90, 9, 99, 128),
                                            (256, 28, 960, 257)])
def test_encode_with_masses_of_equal_codewords(gpu, m, distinct, d, N):
    """Codebooks whose codewords are there nine times or more, beside vectors that have infinities, NaN or a norm beyond
    fp32 in every block: the smallest index of the nearest (the oracle's), a current codeword kept among equal ones, and
    the neighbours' codes as without them."""
    torch, b = gpu
    K = 3
    rng = np.random.default_rng(m * 1000 + d)
    base = (rng.standard_normal((K, distinct, d)) * (0.5 ** np.arange(K))[:, None, None]).astype(np.float32)
    cb = base[:, np.arange(m) % distinct]
    src = rng.integers(0, distinct, (K, N))
    x = (sum(base[k][src[k]] for k in range(K)) + 0.01 * rng.standard_normal((N, d))).astype(np.float32)
    bad = np.arange(5, N, 64)
    y = x.copy()
    y[bad[0::3], 0] = np.inf
    y[bad[1::3], d - 1] = np.nan
    y[bad[2::3]] *= 1e20
    index = b.icq_index_create(_dev(torch, cb), torch.empty((K, 0), dtype=torch.uint8, device="cuda"), 1)
    ws = torch.empty(b.icq_encode_workspace_bytes(index, N), dtype=torch.uint8, device="cuda")
    start = rng.integers(0, m, (K, N), dtype=np.uint8)
    out = []
    for v in (x, y):
        codes = torch.full((K, N), 255, dtype=torch.uint8, device="cuda")
        refined, changed = _dev(torch, start), torch.full((2,), -1, dtype=torch.int32, device="cuda")
        b.icq_encode(index, _dev(torch, v), codes, ws)
        b.icq_encode_refine(index, _dev(torch, v), refined, 2, changed, ws)
        torch.cuda.synchronize()
        out.append([t.cpu().numpy() for t in (codes, refined, changed)])
    good = np.setdiff1d(np.arange(N), bad)
    want = orc.encode(cb, x)
    assert (want < distinct).all() and np.array_equal(out[0][0], want)
    assert np.array_equal(out[1][0][:, good], want[:, good]) and (out[1][0] < m).all()
    assert np.array_equal(out[1][1][:, good], out[0][1][:, good]) and (out[1][1] < m).all()
    want, moved = orc.encode_icm(cb, x, start, 2)
    assert np.array_equal(out[0][1], want) and np.array_equal(out[0][2], moved)


@pytest.mark.parametrize("d", [40, 130])
def test_encode_with_codewords_that_are_no_numbers(gpu, d):
    """Codewords with an infinity or NaN are nobody's nearest: the codes are those of a codebook with far codewords there."""
    torch, b = gpu
    K, m, N = 3, 100, 200
    rng = np.random.default_rng(d)
    far = rng.standard_normal((K, m, d)).astype(np.float32)
    x = (sum(far[k][rng.integers(8, m, N)] for k in range(K)) + 0.01 * rng.standard_normal((N, d))).astype(np.float32)
    far[1, 3:6] = 1e6
    cb = far.copy()
    cb[1, 3, 0], cb[1, 4, d - 1], cb[1, 5, 2] = np.inf, np.nan, -np.inf
    index = b.icq_index_create(_dev(torch, cb), torch.empty((K, 0), dtype=torch.uint8, device="cuda"), 1)
    ws = torch.empty(b.icq_encode_workspace_bytes(index, N), dtype=torch.uint8, device="cuda")
    codes = torch.full((K, N), 255, dtype=torch.uint8, device="cuda")
    b.icq_encode(index, _dev(torch, x), codes, ws)
    want = orc.encode(far, x)
    assert np.array_equal(codes.cpu().numpy(), want)
    refined = _dev(torch, want)
    b.icq_encode_refine(index, _dev(torch, x), refined, 2, None, ws)
    assert np.array_equal(refined.cpu().numpy(), orc.encode_icm(far, x, want, 2)[0])


def test_encode_on_disjoint_supports_recovers_the_codes(gpu):
    """Codebooks with pairwise-disjoint supports, vectors that are exact reconstructions: every
    greedy step has a codeword at distance zero, so the codes come back bit for bit; an index
    over the encoded items then reproduces them through the storage round trip."""
    torch, b = gpu
    rng = np.random.default_rng(77)
    K, m, d, N = 8, 256, 64, 20_000
    cb = np.zeros((K, m, d), dtype=np.float32)
    groups = np.array_split(rng.permutation(d), K)
    for k in range(K):
        cb[k][:, groups[k]] = rng.standard_normal((m, len(groups[k]))).astype(np.float32)
    codes = rng.integers(0, m, size=(K, N)).astype(np.uint8)
    x = orc.reconstruct(cb, codes, np.arange(N)).astype(np.float32)
    index = b.icq_index_create(_dev(torch, cb), torch.empty((K, 0), dtype=torch.uint8, device="cuda"), 2)
    out = torch.empty((K, N), dtype=torch.uint8, device="cuda")
    ws = torch.empty(b.icq_encode_workspace_bytes(index, N), dtype=torch.uint8, device="cuda")
    b.icq_encode(index, _dev(torch, x), out, ws)
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy(), codes)
    full = b.icq_index_create(_dev(torch, cb), out, 2)
    back = torch.empty((K, N), dtype=torch.uint8, device="cuda")
    b.icq_index_export_codes(full, 2, back)
    torch.cuda.synchronize()
    assert np.array_equal(back.cpu().numpy(), codes)


@pytest.mark.parametrize("K,m,d,N,sweeps,start", [
    (8, 256, 128, 5_000, 3, "greedy"), (4, 256, 32, 1_000, 2, "random"), (16, 256, 96, 777, 2, "greedy"),
    (3, 100, 17, 130, 4, "random"), (1, 256, 8, 64, 1, "random"), (2, 7, 5, 1, 2, "greedy")])
def test_encode_refine_matches_oracle(gpu, K, m, d, N, sweeps, start):
    """Coordinate descent over the codebooks from the same starting codes on both sides.  fp32 scores
    may order near-ties differently and a different choice changes every later step, so each GPU
    sweep is judged given the GPU's own codes before it: level by level the chosen codeword must be
    a nearest one up to the tolerance and a replaced one must not have been clearly nearer; the
    error never grows beyond the tolerance; the counts of replaced sub-codes are exact; and the
    end result is as good as the oracle's, mostly identical."""
    torch, b = gpu
    rng = np.random.default_rng(K * 1000 + d + 1)
    cb = (rng.standard_normal((K, m, d)) * (0.8 ** np.arange(K))[:, None, None]).astype(np.float32)
    src = rng.integers(0, m, size=(K, N))
    x = np.ascontiguousarray(sum(cb[k][src[k]] for k in range(K)) + 0.3 * rng.standard_normal((N, d)), dtype=np.float32)
    first = orc.encode(cb, x) if start == "greedy" else rng.integers(0, m, size=(K, N)).astype(np.uint8)
    index = b.icq_index_create(_dev(torch, cb), torch.empty((K, 0), dtype=torch.uint8, device="cuda"), min(2, K))
    ws = torch.empty(b.icq_encode_workspace_bytes(index, N), dtype=torch.uint8, device="cuda")
    xd = _dev(torch, x)
    # the error call against the oracle's
    err = torch.empty((N,), dtype=torch.float64, device="cuda")
    b.icq_quantization_error(index, xd, _dev(torch, first), err)
    torch.cuda.synchronize()
    err0 = orc.quantization_error(cb, x, first)
    assert np.allclose(err.cpu().numpy(), err0, rtol=1e-10, atol=1e-12)
    # all sweeps in one call, and one by one
    codes_all = _dev(torch, first)
    changed_all = torch.full((sweeps,), -1, dtype=torch.int32, device="cuda")
    b.icq_encode_refine(index, xd, codes_all, sweeps, changed_all, ws)
    cur = _dev(torch, first)
    one = torch.full((1,), -1, dtype=torch.int32, device="cuda")
    cb64, x64, n = cb.astype(np.float64), x.astype(np.float64), np.arange(N)
    before, prev_err = first.copy(), err0
    for sw in range(sweeps):
        b.icq_encode_refine(index, xd, cur, 1, one, ws)
        torch.cuda.synchronize()
        after = cur.cpu().numpy()
        assert (after < m).all()
        assert int(one.cpu()[0]) == int((after != before).sum()) == int(changed_all.cpu()[sw])
        for k in range(K):
            state = np.concatenate([after[:k], before[k:]])          # the codes this level saw
            r = x64 - sum(cb64[l][state[l]] for l in range(K) if l != k)
            d2 = ((r[:, None, :] - cb64[k][None, :, :]) ** 2).sum(axis=2) if N * m * d < 4e7 else \
                (r * r).sum(axis=1)[:, None] - 2.0 * r @ cb64[k].T + (cb64[k] ** 2).sum(axis=1)[None, :]
            chosen, old, best = d2[n, after[k]], d2[n, before[k]], d2.min(axis=1)
            assert (chosen <= best + tol(best)).all(), "sweep %d level %d: a clearly nearer codeword exists" % (sw, k)
            moved = after[k] != before[k]
            assert (chosen[moved] <= old[moved] + tol(old[moved])).all(), "replaced a clearly nearer codeword"
        e = orc.quantization_error(cb, x, after)
        assert (e <= prev_err + tol(prev_err)).all()
        before, prev_err = after, e
    assert np.array_equal(codes_all.cpu().numpy(), before)            # one call = the same sweeps one by one
    want, want_changed = orc.encode_icm(cb, x, first, sweeps)
    e_want = orc.quantization_error(cb, x, want)
    assert abs(prev_err.mean() - e_want.mean()) <= 0.01 * e_want.mean() + 1e-12
    assert (before == want).all(axis=0).mean() >= 0.9
    assert prev_err.mean() <= err0.mean()
    # no sweeps: untouched; too many: refused
    b.icq_encode_refine(index, xd, cur, 0, None, ws)
    torch.cuda.synchronize()
    assert np.array_equal(cur.cpu().numpy(), before)
    with pytest.raises(b.IcqError):
        b.icq_encode_refine(index, xd, cur, 65, None, ws)
    with pytest.raises(b.IcqError):
        b.icq_encode_refine(index, xd, cur, 1, None, ws[:128])


def test_encode_refine_on_disjoint_supports_finds_the_planted_codes_in_one_sweep(gpu):
    torch, b = gpu
    rng = np.random.default_rng(78)
    K, m, d, N = 8, 256, 64, 20_000
    cb = np.zeros((K, m, d), dtype=np.float32)
    groups = np.array_split(rng.permutation(d), K)
    for k in range(K):
        cb[k][:, groups[k]] = rng.standard_normal((m, len(groups[k]))).astype(np.float32)
    codes = rng.integers(0, m, size=(K, N)).astype(np.uint8)
    x = orc.reconstruct(cb, codes, np.arange(N)).astype(np.float32)
    index = b.icq_index_create(_dev(torch, cb), torch.empty((K, 0), dtype=torch.uint8, device="cuda"), 2)
    cur = _dev(torch, rng.integers(0, m, size=(K, N)).astype(np.uint8))
    changed = torch.zeros((2,), dtype=torch.int32, device="cuda")
    ws = torch.empty(b.icq_encode_workspace_bytes(index, N), dtype=torch.uint8, device="cuda")
    b.icq_encode_refine(index, _dev(torch, x), cur, 2, changed, ws)
    torch.cuda.synchronize()
    assert np.array_equal(cur.cpu().numpy(), codes)
    assert int(changed.cpu()[1]) == 0 and int(changed.cpu()[0]) > 0


# ------------------------------------------------------------------ quantities around the fast set
@pytest.mark.parametrize("mode", [1, 2], ids=["streamed", "grouped"])
def test_search_over_an_index_encoded_from_mixture_vectors(gpu, mode):
    """The clustered shape with codes that come from the encoder: Gaussian-mixture vectors, greedy
    assignment plus two sweeps of coordinate descent.  Both sides encode the vectors themselves;
    the index the search runs over is built from the ORACLE's codes on both sides."""
    torch, b = gpu
    cfg = synth.make_vectors("C3", N=20_000, Q=64)
    cb, x, K, Kf = cfg["codebooks"], cfg["x"], cfg["K"], cfg["Kf"]
    N = x.shape[0]
    want, _ = orc.encode_icm(cb, x, orc.encode(cb, x), 2)
    enc = b.icq_index_create(_dev(torch, cb), torch.empty((K, 0), dtype=torch.uint8, device="cuda"), Kf)
    ws = torch.empty(b.icq_encode_workspace_bytes(enc, N), dtype=torch.uint8, device="cuda")
    got = torch.empty((K, N), dtype=torch.uint8, device="cuda")
    xd = _dev(torch, x)
    b.icq_encode(enc, xd, got, ws)
    b.icq_encode_refine(enc, xd, got, 2, None, ws)
    torch.cuda.synchronize()
    got = got.cpu().numpy()
    assert (got == want).all(axis=0).mean() >= 0.95
    e_got, e_want = orc.quantization_error(cb, x, got).mean(), orc.quantization_error(cb, x, want).mean()
    assert abs(e_got - e_want) <= 1e-3 * e_want
    # the structure the encoder gives the fast sub-codes: a cluster's vectors share the first, mostly the second
    pairs = want[0].astype(np.int64) * 256 + want[1]
    share = np.mean([(pairs[cfg["cluster"] == c] == np.bincount(pairs[cfg["cluster"] == c]).argmax()).mean()
                     for c in range(0, cfg["n_centres"], 10) if (cfg["cluster"] == c).any()])
    assert 0.8 <= share <= 0.999
    cfg["codes"] = want
    g = Gpu(gpu, cfg, mode)
    T, P, D = oracle_all(cfg)
    for rule in (("q", 0.01), ("q", 0.05)):
        thr = _thr(P, rule)
        exact = (P < thr[:, None].astype(np.float64)).sum(axis=1)
        _check_search(g, cfg, T, P, D, thr, cfg["topk"], int(exact.max() * 1.2) + 64)


def test_moments_online_variance_mask_fast_set_and_margin_match_oracle(gpu):
    torch, b = gpu
    rng = np.random.default_rng(12)
    d, n, B = 96, 5_003, 4
    scale = rng.uniform(0.05, 3.0, size=d)
    mean = torch.zeros(d, dtype=torch.float64, device="cuda")
    var = torch.zeros(d, dtype=torch.float64, device="cuda")
    o_mean, o_var = np.zeros(d), np.zeros(d)
    bm = torch.empty(d, dtype=torch.float64, device="cuda")
    bv = torch.empty(d, dtype=torch.float64, device="cuda")
    for step in range(1, B + 1):
        x = (rng.standard_normal((n, d)) * scale + rng.uniform(-1, 1, size=d)).astype(np.float32)
        b.icq_batch_moments(_dev(torch, x), bm, bv)
        b.icq_online_variance_update(mean, var, bm, bv, step)
        torch.cuda.synchronize()
        om, ov = orc.batch_moments(x)
        assert np.allclose(bm.cpu().numpy(), om, rtol=1e-11, atol=1e-13)
        assert np.allclose(bv.cpu().numpy(), ov, rtol=1e-10, atol=1e-13)
        o_mean, o_var = orc.online_variance(o_mean, o_var, om, ov, step)
    lam = var.cpu().numpy()
    assert np.allclose(mean.cpu().numpy(), o_mean, rtol=1e-10, atol=1e-12)
    assert np.allclose(lam, o_var, rtol=1e-9, atol=1e-12)
    # subspace mask from the bimodal prior
    prior = (0.8, 0.6, 0.2, 5.0, 2.0, -10.0)
    xi = torch.empty(d, dtype=torch.uint8, device="cuda")
    b.icq_subspace_mask(var, *prior, xi)
    torch.cuda.synchronize()
    o_xi, pm, pn = orc.subspace_mask(lam, *prior, want_densities=True)
    clear = np.abs(pn - pm) > 1e-9 * (pn + pm)
    assert np.array_equal(xi.cpu().numpy()[clear], o_xi[clear]) and 0 < o_xi.sum() < d
    # fast set of codebooks built inside / outside / across psi, and the margin
    K, m = 6, 256
    inside, outside = np.nonzero(o_xi)[0], np.nonzero(o_xi == 0)[0]
    cb = np.zeros((K, m, d), dtype=np.float32)
    cb[0][:, inside] = rng.standard_normal((m, inside.size))
    cb[1][:, outside] = rng.standard_normal((m, outside.size))
    cb[2][:, inside] = rng.standard_normal((m, inside.size))
    cb[2][200] = 0.0
    cb[2][200, outside[0]] = 0.5
    cb[3] = rng.standard_normal((m, d)).astype(np.float32)
    cb[4][:, inside] = 5.0 * rng.standard_normal((m, inside.size))
    cb[4][:, outside] = 0.01 * rng.standard_normal((m, outside.size))
    cb[5][:, outside] = rng.standard_normal((m, outside.size))
    index = b.icq_index_create(_dev(torch, cb), torch.empty((K, 0), dtype=torch.uint8, device="cuda"), 1)
    fast = torch.empty(K, dtype=torch.uint8, device="cuda")
    b.icq_fast_set(index, _dev(torch, o_xi), fast)
    sigma = torch.empty(1, dtype=torch.float64, device="cuda")
    b.icq_margin(var, _dev(torch, o_xi), sigma)
    torch.cuda.synchronize()
    assert np.array_equal(fast.cpu().numpy(), orc.fast_set(cb, o_xi))
    assert np.array_equal(fast.cpu().numpy()[[0, 1, 2, 4, 5]], [1, 0, 0, 1, 0])
    assert abs(float(sigma.item()) - orc.margin(lam, o_xi)) <= 1e-12 * max(1.0, orc.margin(lam, o_xi))


# ------------------------------------------------------------------ seeded sweep over shapes
def _sweep_cases():
    rng = np.random.default_rng(20240)
    cases = []
    for i in range(36):
        K = int(rng.choice([1, 2, 3, 4, 5, 8, 9, 16, 17]))
        Kf = int(rng.integers(1, min(K, 5) + 1))
        m = int(rng.choice([256, 256, 256, 100, 17]))
        d = int(rng.choice([8, 24, 33, 64]))
        N = int(rng.choice([1, 63, 64, 65, 1_000, 4_097, 16_384, 40_000, 70_001]))
        Q = int(rng.choice([1, 2, 3, 4, 5, 7, 8, 63, 64, 65, 130, 515]))
        topk = int(rng.choice([1, 10, 100, 129, 257]))
        frac = float(rng.choice([0.002, 0.01, 0.05, 0.3, 1.0]))
        mode = int(rng.choice([0, 0, 1, 2]))
        cases.append((i, K, Kf, m, d, N, Q, topk, frac, mode))
    return cases


@pytest.mark.parametrize("case", _sweep_cases(), ids=lambda c: "s%02d-K%d-Kf%d-m%d-N%d-Q%d-k%d-f%g-mode%d" % (
    c[0], c[1], c[2], c[3], c[5], c[6], c[7], c[8], c[9]))
def test_search_sweep_against_oracle(gpu, case):
    """Shapes drawn from a fixed seed: codebook counts around the record widths (4 / 8 / 16 / wider),
    every Kf up to 5, short codebooks, ragged N and Q around the tile sizes, lists from 1 to 257,
    survivor fractions from 0.2 % to all, every stage-1 form."""
    i, K, Kf, m, d, N, Q, topk, frac, mode = case
    rng = np.random.default_rng(1000 + i)
    cb = (rng.standard_normal((K, m, d)) * (0.7 ** np.arange(K))[:, None, None]).astype(np.float32)
    codes = rng.integers(0, m, size=(K, N), dtype=np.uint8)
    src = rng.integers(0, N, size=Q)
    queries = sum(cb[k][codes[k, src]] for k in range(K)) + 0.1 * rng.standard_normal((Q, d))
    cfg = dict(codebooks=cb, codes=codes, queries=np.ascontiguousarray(queries, dtype=np.float32),
               K=K, Kf=Kf, d=d, N=N, Q=Q, topk=topk)
    g = Gpu(gpu, cfg, mode if Kf <= 4 else (0 if mode == 2 else mode))
    T, P, D = oracle_all(cfg)
    if frac >= 1.0:
        thr = np.full(Q, np.inf, dtype=np.float32)
    else:
        thr = np.quantile(P, frac, axis=1).astype(np.float32)
    _check_search(g, cfg, T, P, D, thr, topk, N + 1)


@pytest.mark.parametrize("K,Kf,m,N,Q,topk,frac", [
    (4, 1, 256, 1, 3, 5, 1.0), (16, 4, 256, 63, 8, 10, 0.5), (8, 3, 200, 2047, 5, 100, 0.1), (6, 2, 256, 2049, 4, 10, 0.01),
    (12, 4, 256, 4096, 37, 257, 1.0), (3, 3, 77, 8191, 70, 100, 0.2), (16, 3, 256, 50_001, 33, 100, 0.02),
    (5, 2, 256, 400_003, 4, 512, 0.01), (16, 4, 256, 4095, 5, 100, 1.0), (8, 3, 256, 4097, 7, 20, 0.3), (4, 3, 130, 8193, 3, 50, 1.0),
    (8, 3, 256, 2048, 600, 20, 0.2), (16, 4, 256, 2049, 513, 10, 0.1), (4, 2, 256, 700, 1030, 30, 1.0)])
def test_search_of_a_small_index_in_one_kernel(gpu, K, Kf, m, N, Q, topk, frac):
    """Both stages in one kernel (few items times queries): against the oracle, and bit for bit against the scan with
    candidate lists (the sums are the same fp32 additions).  Sizes around a step of 4096 items and half of it, all record widths;
    600, 513 and 1030 queries: either side of the line where a block is half as large."""
    rng = np.random.default_rng(K * 1000 + N)
    cb = (rng.standard_normal((K, m, 24)) * (0.7 ** np.arange(K))[:, None, None]).astype(np.float32)
    codes = rng.integers(0, m, size=(K, N), dtype=np.uint8)
    src = rng.integers(0, N, size=Q)
    queries = sum(cb[k][codes[k, src]] for k in range(K)) + 0.1 * rng.standard_normal((Q, 24))
    cfg = dict(codebooks=cb, codes=codes, queries=np.ascontiguousarray(queries, dtype=np.float32),
               K=K, Kf=Kf, d=24, N=N, Q=Q, topk=topk)
    T, P, D = oracle_all(cfg)
    thr = np.full(Q, np.inf, dtype=np.float32) if frac >= 1.0 else np.quantile(P, frac, axis=1).astype(np.float32)
    if Q >= 5:
        thr[1], thr[2], thr[3] = np.inf, np.nan, -np.inf
    out = _check_search(Gpu(gpu, cfg), cfg, T, P, D, thr, topk, N + 1, min_equal=0.9 if topk <= 100 else 0.0)
    for a, c in zip(out, Gpu(gpu, cfg, 1).search(thr, N + 1, topk)):
        assert np.array_equal(a, c, equal_nan=True)


@pytest.mark.parametrize("Kf,Q,bounds", [(4, 130, [0, 60_001, 63_000]), (2, 300, [0, 9_000, 20_001])])
def test_running_search_with_a_long_first_tile(gpu, Kf, Q, bounds):
    """Nothing is excluded from the first tile: a block of the one-kernel form takes several steps of it.  Bit for bit what
    the scan with candidate lists gives."""
    torch, b = gpu
    cfg = small("C4", bounds[-1], Q, K=8, Kf=Kf)
    cb, queries = _dev(torch, cfg["codebooks"]), _dev(torch, cfg["queries"])
    sigma = torch.full((Q,), 5.0, dtype=torch.float32, device="cuda")
    results = []
    for mode in (0, 1):
        tiles = [b.icq_index_create(cb, _dev(torch, cfg["codes"][:, a:e]), Kf) for a, e in zip(bounds[:-1], bounds[1:])]
        for t in tiles:
            b.icq_index_set_scan_mode(t, mode)
        out = [torch.empty((Q, 100), dtype=torch.int32, device="cuda"), torch.empty((Q, 100), dtype=torch.float32, device="cuda"),
               torch.empty((Q,), dtype=torch.int32, device="cuda")]
        ws = torch.empty(b.icq_running_workspace_bytes(tiles, Q, bounds[1], 100), dtype=torch.uint8, device="cuda")
        b.icq_search_running(tiles, bounds[:-1], queries, sigma, bounds[1], 100, *out, ws)
        torch.cuda.synchronize()
        results.append([o.cpu().numpy() for o in out])
    assert (results[0][2] >= bounds[1]).all()
    for a, c in zip(*results):
        assert np.array_equal(a, c)


def _hit_bit_cases():
    rng = np.random.default_rng(20241)
    cases = []
    for i in range(14):
        K = int(rng.choice([4, 5, 8, 12, 16]))
        Kf = int(rng.integers(1, 5))
        m = int(rng.choice([256, 256, 100]))
        big = i % 3 == 0                      # from 2^22 items on: also the pair ordering (Kf = 3, 4), any six queries
        N = int(rng.choice([4_200_000, 4_456_449]) if big else rng.choice([524_288, 530_001, 1_048_577, 1_300_000]))
        Q = int(rng.choice([6, 9, 16, 33]) if big else rng.choice([32, 40, 65]))
        topk = int(rng.choice([1, 10, 100, 257]))
        fracs = [float(f) for f in rng.choice([0.0005, 0.002, 0.01, 0.1, 0.5], size=2, replace=False)]
        # Kf <= 2: the tuple walk would take the call otherwise; large and Kf = 3, 4: mostly the pair ordering
        mode = 1 if Kf <= 2 else (int(i % 12 != 6) ^ 1 if big else int(rng.choice([0, 1])))
        cases.append((i, K, Kf, m, N, Q, topk, fracs, mode))
    return cases


@pytest.mark.parametrize("case", _hit_bit_cases(), ids=lambda c: "h%02d-K%d-Kf%d-m%d-N%d-Q%d-k%d-mode%d" % (
    c[0], c[1], c[2], c[3], c[4], c[5], c[6], c[8]))
def test_search_sweep_over_hit_bits(gpu, case):
    """Shapes drawn from a fixed seed at sizes where icq_search keeps hit bits and stage 1 is the 16-bit
    pre-filter: every Kf from 1 to 4 in id order, Kf = 3, 4 over the pair ordering, short codebooks (table
    entries at +inf), ragged N, query counts around the pass width of eight, and per query a threshold
    from a mix of quantiles (a sparse and a dense one per case), +inf and -inf."""
    i, K, Kf, m, N, Q, topk, fracs, mode = case
    rng = np.random.default_rng(3000 + i)
    d = 16
    cb = (rng.standard_normal((K, m, d)) * (0.8 ** np.arange(K))[:, None, None]).astype(np.float32)
    codes = rng.integers(0, m, size=(K, N), dtype=np.uint8)
    src = rng.integers(0, N, size=Q)
    queries = sum(cb[k][codes[k, src]] for k in range(K)) + 0.2 * rng.standard_normal((Q, d))
    cfg = dict(codebooks=cb, codes=codes, queries=np.ascontiguousarray(queries, dtype=np.float32),
               K=K, Kf=Kf, d=d, N=N, Q=Q, topk=topk)
    g = Gpu(gpu, cfg, mode)
    T, P, D = oracle_all(cfg)
    thr = np.empty(Q, dtype=np.float32)
    for q in range(Q):
        thr[q] = np.quantile(P[q], fracs[q % 2])
    thr[Q - 1] = np.inf
    thr[Q - 2] = -np.inf
    exact = (P < thr[:, None].astype(np.float64)).sum(axis=1)
    _check_search(g, cfg, T, P, D, thr, topk, int(exact.max()) + 64, min_equal=0.8)


def test_search_calls_overlapping_on_two_streams(gpu):
    """The configuration the benchmark times: the batches of a query set alternate between two streams, each with
    a workspace of its own, on ONE index, so that one batch's stage 2 runs beside the next batch's stage 1.  The
    lists must be those of the same calls made one after the other, and those the oracle accepts."""
    torch, b = gpu
    cfg = small("C4", 4_300_017, 96, K=12)
    Q, topk, batch = 96, 100, 16
    T, P, D = oracle_all(cfg)
    thr = thresholds_quantile(P, 0.01)
    g = Gpu(gpu, cfg, 0)
    cap = int((P < thr[:, None].astype(np.float64)).sum(axis=1).max() * 1.2) + 64
    thr_dev = _dev(torch, thr)
    one = g.search(thr, cap, topk)
    out_ids = torch.full((Q, topk), -1, dtype=torch.int32, device="cuda")
    out_dist = torch.full((Q, topk), float("nan"), dtype=torch.float32, device="cuda")
    surv = torch.full((Q,), 12345, dtype=torch.int32, device="cuda")
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    wss = [g.workspace(batch, cap, topk), g.workspace(batch, cap, topk)]
    torch.cuda.synchronize()
    for rep in range(3):                                   # the same overlap three times over: no state carried along
        cur = torch.cuda.current_stream()
        for st in streams:
            st.wait_stream(cur)
        for i, q0 in enumerate(range(0, Q, batch)):
            with torch.cuda.stream(streams[i % 2]):
                b.icq_search(g.index, g.queries[q0:q0 + batch], thr_dev[q0:q0 + batch], cap, topk,
                             out_ids[q0:q0 + batch], out_dist[q0:q0 + batch], surv[q0:q0 + batch], wss[i % 2])
        for st in streams:
            cur.wait_stream(st)
        torch.cuda.synchronize()
        assert np.array_equal(_u32(out_ids), one[0]) and np.array_equal(out_dist.cpu().numpy(), one[1])
        assert np.array_equal(_u32(surv), one[2])
        out_ids.fill_(-1)
        out_dist.fill_(float("nan"))
    o_ids = orc.search(T, cfg["codes"], cfg["Kf"], thr, topk)[0]
    for q in range(Q):
        check_topk(P[q], D[q], thr[q], topk, one[0][q], one[1][q])
    assert (one[0] == o_ids).all(axis=1).mean() >= 0.9


# ------------------------------------------------------------------ HIP graphs
@pytest.mark.parametrize("name,N,Q,over", [("C0", 10_000, 100, {}), ("C1", 200_003, 130, {}), ("C4", 4_300_017, 16, dict(K=12))],
                         ids=["tuples-Kf1", "tuples-Kf2", "pairs-hit-bits"])
def test_search_replayed_from_a_captured_graph(gpu, name, N, Q, over):
    """icq_search only launches kernels on the caller's stream (counters are cleared by fill kernels,
    not memset nodes), so a call can be captured into a HIP graph and replayed: three replays, with
    eager work and synchronisations in between and the outputs scrubbed before each, give the eager
    call's lists bit for bit -- also after the queries and thresholds behind the captured pointers
    have been replaced."""
    torch, b = gpu
    cfg = small(name, N, Q, **over)
    g = Gpu(gpu, cfg)
    topk = cfg["topk"]
    rng = np.random.default_rng(5)
    P = orc.partial(orc.lut(cfg["codebooks"], cfg["queries"]), cfg["codes"], cfg["Kf"])
    thr_np = thresholds_quantile(P, 0.01)
    cap = int(N * 0.03) + 64
    queries = g.queries.clone()
    thr = _dev(torch, thr_np)
    out_ids = torch.empty((Q, topk), dtype=torch.int32, device="cuda")
    out_dist = torch.empty((Q, topk), dtype=torch.float32, device="cuda")
    surv = torch.empty((Q,), dtype=torch.int32, device="cuda")
    ws = g.workspace(Q, cap, topk)
    b.icq_search(g.index, queries, thr, cap, topk, out_ids, out_dist, surv, ws)      # eager: also sets kernel attributes
    torch.cuda.synchronize()
    want = (out_ids.clone(), out_dist.clone(), surv.clone())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        b.icq_search(g.index, queries, thr, cap, topk, out_ids, out_dist, surv, ws)
    for rep in range(3):
        out_ids.fill_(-7); out_dist.fill_(float("nan")); surv.fill_(-7)
        ws.fill_(rep + 1)                                   # whatever an earlier call left must not matter
        junk = torch.randn(1 << 20, device="cuda").sum()    # eager work between the replays
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out_ids, want[0]) and torch.equal(out_dist, want[1]) and torch.equal(surv, want[2]), rep
        del junk
    # other queries behind the same pointers: the graph follows the data, not the values it was captured with
    perm = torch.from_numpy(rng.permutation(Q)).cuda()
    queries.copy_(g.queries[perm])
    thr.copy_(thr[perm])
    graph.replay()
    torch.cuda.synchronize()
    assert torch.equal(out_ids, want[0][perm]) and torch.equal(out_dist, want[1][perm]) and torch.equal(surv, want[2][perm])
