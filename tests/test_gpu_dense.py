"""GPU parity of dense_ip_topk (exact inner-product top-k over an fp16 store) against the oracle.

The call has three regimes, each covered here:
  * the store is no larger than the exact sample, or all its scores are few enough to be kept
    (at most 2^26, of at most 2^21 rows, and fewer where filtering them is the faster way): every
    row is scored and selected directly;
  * the filter path: rows past the sample are kept only when they beat the sample's k-th score;
  * the exact fallback: a query whose candidate list overflows is queued on the device and its
    k-th key found by a radix select over rescans of the store, then its top-k collected; the
    call stays asynchronous (it is captured and replayed in a HIP graph here).
Top-k lists are checked with the rules of tests/topk_check.py at tolerance 2e-3 (fp16 products
are exact in fp32, so scores differ from the oracle only by the fp32 summation order).
"""

import numpy as np
import pytest
import torch

import oracle
import paper_2505_04846_amd as hpr
import synth
from topk_check import check_topk

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
REL = 2e-3
SAMPLE_ROWS = 131072  # rows scored exactly before the filtered scan (k <= 4096)


def _f16(t):
    return oracle.decode_fp16(t.detach().cpu().contiguous().view(torch.int16).numpy())


def _rows(n, dim, seed):
    g = torch.Generator().manual_seed(seed)
    return synth.unit_rows(n, dim, g, "cpu", torch.float16)


def _check_structure(s, i, n, k):
    assert s.shape[1] == k and i.shape[1] == k
    assert np.all((i >= 0) & (i < n))
    for q in range(s.shape[0]):
        assert np.unique(i[q]).size == k
        a, b = s[q, :-1], s[q, 1:]
        assert np.all((a > b) | ((a == b) & (i[q, :-1] < i[q, 1:])))


def _tile(filtered, nq, rows, dim, k):
    """The GEMM tile of a launch, as the library chooses it (so that no case drifts off its line)."""
    def grid(tq, tr):
        return -(-nq // tq) * -(-rows // tr)
    if nq > 128 and grid(256, 256) >= 144:
        return "wide"
    if filtered and 64 < nq <= 128 and nq * k > 192 * dim:
        return "wide"
    if nq > 64 and grid(128, 128) >= 384:
        return "mid"
    if nq > 32 and grid(64, 128) >= 300:
        return "long" if filtered else "narrow"
    if filtered and nq <= 32:
        return "skinny" if dim >= 640 and dim & (dim - 1) and nq * k <= 5 * dim else "long"
    if nq <= 32 and dim >= 4096 and rows * dim >= 3 << 29:
        return "short"
    return "skinny" if grid(32, 128) >= 192 else "short"


def _filtered(nq, n, dim, k):
    """Whether a call filters the rows past its sample; otherwise it stores every score."""
    past = n - SAMPLE_ROWS
    if past <= 0:
        return False
    if n > 1 << 21 or nq * n > 1 << 26:
        return True
    most = 9 << 22 if dim < 256 else 5 << 22 if dim < 2048 else 1 << 24
    k_most = 64 + dim // 6
    return nq <= 128 and k < k_most and nq * past * (k_most - k) > most * k_most


def _device_rows(n, dim, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    X = torch.empty((n, dim), dtype=torch.float16, device=DEV)
    step = (1 << 27) // dim
    for r in range(0, n, step):
        x = torch.randn((min(n - r, step), dim), generator=g, device=DEV)
        X[r:r + step] = synth._normalise(x).to(torch.float16)
    return X


def _scores64(Q, X):
    """The exact scores of device rows, in 64 bits, on the host."""
    q, step = Q.double(), (1 << 27) // X.shape[1]
    return torch.cat([q @ X[r:r + step].double().t().contiguous()
                      for r in range(0, X.shape[0], step)], 1).cpu().numpy()


@pytest.mark.parametrize("nq,n,dim,k", [
    (1, 1, 8, 1),          # smallest shapes
    (37, 5000, 200, 10),   # K tail (200 = 6 chunks of 32 + 8), ragged query and row tiles
    (300, 2048, 4096, 100),
    (5, 1000, 8192, 1000),  # largest dim; k = n
    (3, 777, 24, 777),
    (64, 3000, 128, 10),   # whole tiles of 32 queries
    (65, 3000, 136, 10),   # one query past them
])
def test_dense_topk_whole_store_sampled(nq, n, dim, k):
    Q, X = _rows(nq, dim, 1 + n), _rows(n, dim, 2 + n)
    s, i = hpr.dense_ip_topk(Q.to(DEV), X.to(DEV), k)
    s, i = s.cpu().numpy(), i.cpu().numpy()
    O = oracle.dense_scores(_f16(Q), _f16(X))
    for q in range(nq):
        check_topk(s[q], i[q], O[q], k, rel=REL)


def test_dense_topk_filter_path_matches_oracle():
    nq, n, dim, k = 300, 240_000, 96, 50
    assert _filtered(nq, n, dim, k) and _tile(True, nq, n - SAMPLE_ROWS, dim, k) == "wide"
    Q, X = _rows(nq, dim, 11), _rows(n, dim, 12)
    s, i = hpr.dense_ip_topk(Q.to(DEV), X.to(DEV), k)
    s, i = s.cpu().numpy(), i.cpu().numpy()
    _check_structure(s, i, n, k)
    Xh = _f16(X)
    Qh = _f16(Q)
    # every returned score against the oracle's score of the same row
    for q in range(nq):
        o = Xh[i[q]] @ Qh[q]
        err = np.abs(s[q] - o)
        assert np.all(err <= REL * np.maximum(np.abs(o), 1e-3)), f"query {q}"
    # full oracle rows for the tile edges and a seeded sample of queries
    rng = np.random.default_rng(0)
    pick = sorted(set([0, 1, 255, 256, 299]) | set(rng.choice(nq, 11, replace=False).tolist()))
    O = oracle.dense_scores(Qh[pick], Xh)
    for r, q in enumerate(pick):
        res = check_topk(s[q], i[q], O[r], k, rel=REL)
        assert res["exact"] or res["exception_used"]


def test_dense_topk_filter_path_few_queries():
    # the sample takes tiles of 32 queries, the filtered scan of 64
    nq, n, dim, k = 17, 2_100_003, 256, 100
    assert _filtered(nq, n, dim, k)
    assert _tile(False, nq, SAMPLE_ROWS, dim, k) == "skinny"
    assert _tile(True, nq, n - SAMPLE_ROWS, dim, k) == "long"
    Q, X = _device_rows(nq, dim, 13), _device_rows(n, dim, 14)
    s, i = hpr.dense_ip_topk(Q, X, k)
    s, i = s.cpu().numpy(), i.cpu().numpy()
    _check_structure(s, i, n, k)
    O = _scores64(Q, X)
    for q in range(nq):
        check_topk(s[q], i[q], O[q], k, rel=REL)


def test_dense_topk_overflowing_lists_take_the_exact_fallback():
    nq, n, dim, k = 460, 150_000, 200, 20
    assert _filtered(nq, n, dim, k) and _tile(True, nq, n - SAMPLE_ROWS, dim, k) == "wide"
    Q, X = _rows(nq, dim, 21), _rows(n, dim, 22)
    a0 = SAMPLE_ROWS + 100
    a1 = SAMPLE_ROWS + 5000
    X[a0:a0 + 3000] = Q[0]   # 3000 bit-identical rows equal to query 0, past the sample
    X[a1:a1 + 2000] = Q[1]
    Qd, Xd = Q.to(DEV), X.to(DEV)
    s, i = hpr.dense_ip_topk(Qd, Xd, k)
    s2, i2 = hpr.dense_ip_topk(Qd, Xd, k)
    assert torch.equal(s, s2) and torch.equal(i, i2)
    s, i = s.cpu().numpy(), i.cpu().numpy()
    _check_structure(s, i, n, k)
    # the copies tie exactly and outrank every other row: the lowest k indices win
    assert i[0].tolist() == list(range(a0, a0 + k))
    assert i[1].tolist() == list(range(a1, a1 + k))
    assert np.all(s[0] == s[0, 0]) and np.all(s[1] == s[1, 0])
    Qh, Xh = _f16(Q), _f16(X)
    O = oracle.dense_scores(Qh[:4], Xh)
    assert abs(s[0, 0] - O[0, a0]) <= REL * abs(O[0, a0])
    for q in range(2, 4):
        check_topk(s[q], i[q], O[q], k, rel=REL)


def _overflowing_store(nq, n, dim, copies, seed):
    # queries near a common direction u; `copies` bit-identical rows equal to u past the sample
    # outscore every random row for every query, so every candidate list overflows
    g = torch.Generator().manual_seed(seed)
    u = synth.unit_rows(1, dim, g, "cpu", torch.float32)
    noise = torch.randn((nq, dim), generator=g)
    Q = synth._normalise(u + 0.1 * noise / dim ** 0.5).to(torch.float16)
    X = _rows(n, dim, seed + 1)
    a0 = SAMPLE_ROWS + 777
    X[a0:a0 + copies] = u.to(torch.float16)
    return Q, X, a0


@pytest.mark.parametrize("nq,n,copies,tile", [(70, 960_000, 4000, "mid"), (520, 150_000, 2500, "wide")])
def test_dense_topk_every_list_overflows(nq, n, copies, tile):
    # every query is queued: the fallback's rescans take two and nine 64-query tiles, over seven
    # K stages (the last one ragged)
    dim, k = 200, 100
    assert _filtered(nq, n, dim, k) and _tile(True, nq, n - SAMPLE_ROWS, dim, k) == tile
    Q, X, a0 = _overflowing_store(nq, n, dim, copies, 41)
    Qd, Xd = Q.to(DEV), X.to(DEV)
    s, i = hpr.dense_ip_topk(Qd, Xd, k)
    s, i = s.cpu().numpy(), i.cpu().numpy()
    _check_structure(s, i, n, k)
    for q in range(nq):
        assert i[q].tolist() == list(range(a0, a0 + k)), f"query {q}"
        assert np.all(s[q] == s[q, 0])
    pick = [0, 63, 64, nq - 1]
    O = _scores64(Qd[pick], Xd)
    for r, q in enumerate(pick):
        check_topk(s[q], i[q], O[r], k, rel=REL)


def test_dense_topk_replays_in_a_hip_graph_with_overflow():
    # the whole call, the device-decided fallback included, is captured once and replayed with
    # eager work and synchronisation in between; every replay reproduces the eager result
    nq, n, dim, k = 460, 150_000, 136, 20
    assert _filtered(nq, n, dim, k)
    Q, X = _rows(nq, dim, 21), _rows(n, dim, 22)
    a0 = SAMPLE_ROWS + 100
    X[a0:a0 + 3000] = Q[0]
    Qd, Xd = Q.to(DEV), X.to(DEV)
    ref_s, ref_i = hpr.dense_ip_topk(Qd, Xd, k)
    ws = hpr.dense_workspace(Qd, Xd, k)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        hpr.dense_ip_topk(Qd, Xd, k, ws=ws)
    torch.cuda.current_stream().wait_stream(side)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        gs, gi = hpr.dense_ip_topk(Qd, Xd, k, ws=ws)
    for rep in range(3):
        gs.fill_(float("nan"))
        gi.fill_(-1)
        g.replay()
        hpr.dense_ip_topk(Qd[:3].contiguous(), Xd, 5)   # unrelated eager work
        torch.cuda.synchronize()
        assert torch.equal(gs, ref_s) and torch.equal(gi, ref_i), f"replay {rep}"
    assert gi[0].tolist() == list(range(a0, a0 + k))


@pytest.mark.parametrize("nq,n,dim,k,copies,tile", [
    (520, 150_000, 136, 50, 0, "wide"),
    (64, 1_100_000, 72, 20, 0, "long"),
    (520, 150_000, 136, 20, 3000, "wide"),  # two overflowing lists: the exact fallback
    (64, 1_100_000, 72, 20, 5000, "long"),
])
def test_dense_topk_past_the_stored_scores(nq, n, dim, k, copies, tile):
    # more than 2^26 scores: sample, filtered scan, merge, and the fallback for the overflowing lists
    assert _filtered(nq, n, dim, k) and _tile(True, nq, n - SAMPLE_ROWS, dim, k) == tile
    Q, X = _rows(nq, dim, 51 + nq), _rows(n, dim, 52 + nq)
    at = {0: SAMPLE_ROWS + 100, nq - 1: n - copies - 1}
    if copies:
        for q, a in at.items():
            X[a:a + copies] = Q[q]
    Qd, Xd = Q.to(DEV), X.to(DEV)
    s, i = hpr.dense_ip_topk(Qd, Xd, k)
    ws = hpr.dense_workspace(Qd, Xd, k)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        hpr.dense_ip_topk(Qd, Xd, k, ws=ws)
    torch.cuda.current_stream().wait_stream(side)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        gs, gi = hpr.dense_ip_topk(Qd, Xd, k, ws=ws)
    for rep in range(3):
        gs.fill_(float("nan"))
        g.replay()
        hpr.dense_ip_topk(Qd[:3].contiguous(), Xd, 5)   # unrelated eager work
        torch.cuda.synchronize()
        assert torch.equal(gs, s) and torch.equal(gi, i), f"replay {rep}"
    s, i = s.cpu().numpy(), i.cpu().numpy()
    _check_structure(s, i, n, k)
    pick = [0, 1, nq // 2, nq - 1]
    O = oracle.dense_scores(_f16(Q[pick]), _f16(X))
    for r, q in enumerate(pick):
        if copies and q in at:  # bit-identical rows, the highest scores: the lowest indices
            dup = O[r].max() - 1e-9
            lowest = np.nonzero(O[r] >= dup)[0][:k]
            assert i[q].tolist() == lowest.tolist()
        else:
            check_topk(s[q], i[q], O[r], k, rel=REL)


@pytest.mark.parametrize("nq,n,dim,k,tile", [
    (600, SAMPLE_ROWS + 48 * 256 - 3, 136, 20, "wide"),  # 144 of them; one fewer
    (600, SAMPLE_ROWS + 47 * 256, 136, 20, "mid"),
    (100, 700_003, 72, 10, "mid"), (100, 700_003, 72, 138, "mid"), (100, 700_003, 72, 139, "wide"),
    (65, 1_100_001, 200, 10, "mid"), (64, 1_100_001, 200, 10, "long"), (33, 2_100_001, 136, 20, "long"),
    (32, 2_100_001, 200, 10, "long"), (1, 2_100_001, 136, 1000, "long"),
    (32, 2_100_001, 648, 101, "skinny"), (32, 2_100_001, 648, 102, "long"),
    (3, 2_100_001, 768, 10, "skinny"), (3, 2_100_001, 1024, 10, "long"),
    (520, SAMPLE_ROWS + 1629, 136, 50, "skinny"), (520, SAMPLE_ROWS + 929, 136, 50, "short"),
])
def test_dense_topk_filter_tiles(nq, n, dim, k, tile):
    # the filter of every tile, on both sides of the lines between them, over several K stages
    assert _filtered(nq, n, dim, k) and _tile(True, nq, n - SAMPLE_ROWS, dim, k) == tile
    Q, X = _device_rows(nq, dim, 81 + nq), _device_rows(n, dim, 82 + dim)
    X[n - 1], X[SAMPLE_ROWS] = Q[nq - 1], Q[0]  # the edges of the scan hold winners
    s, i = hpr.dense_ip_topk(Q, X, k)
    s, i = s.cpu().numpy(), i.cpu().numpy()
    _check_structure(s, i, n, k)
    assert n - 1 in i[nq - 1] and SAMPLE_ROWS in i[0]
    pick = sorted({0, nq // 2, nq - 1})
    O = _scores64(Q[pick], X)
    for r, q in enumerate(pick):
        check_topk(s[q], i[q], O[r], k, rel=REL)


@pytest.mark.parametrize("nq,n,dim,k,tile", [
    (129, 36_700, 72, 10, "wide"), (256, 36_609, 64, 10, "wide"), (257, 18_177, 40, 10, "wide"),  # 144
    (129, 36_600, 72, 10, "mid"), (257, 18_176, 40, 10, "mid"),  # of them, and fewer
    (128, 49_100, 24, 10, "mid"), (65, 49_025, 136, 10, "mid"), (65, 49_024, 136, 10, "narrow"),
    (33, 38_300, 200, 10, "narrow"), (64, 38_273, 8, 10, "narrow"), (64, 38_272, 8, 10, "skinny"),
    (32, 24_500, 72, 10, "skinny"), (1, 24_449, 1032, 10, "skinny"), (33, 12_200, 128, 10, "skinny"),
    (31, 24_448, 72, 10, "short"), (1, 65, 4096, 10, "short"),
    # many rounds of long rows
    (2, 196_608, 8192, 5, "short"), (2, 196_607, 8192, 5, "skinny"), (32, 393_217, 4096, 5, "short"),
    (32, 400_000, 4088, 5, "skinny"),
])
def test_dense_topk_tile_choice(nq, n, dim, k, tile):
    # both sides of every line between the GEMM's tiles, ragged in queries, rows and K
    assert not _filtered(nq, n, dim, k) and _tile(False, nq, n, dim, k) == tile
    Q, X = _device_rows(nq, dim, 61 + n), _device_rows(n, dim, 62 + n)
    X[n - 1], X[0] = Q[nq - 1], Q[0]  # the edges of the tiles hold winners
    s, i = hpr.dense_ip_topk(Q, X, k)
    s, i = s.cpu().numpy(), i.cpu().numpy()
    _check_structure(s, i, n, k)
    assert i[nq - 1, 0] == n - 1 or nq == 1
    assert 0 in i[0]
    pick = sorted({0, nq // 2, nq - 1})
    O = _scores64(Q[pick], X)
    for r, q in enumerate(pick):
        check_topk(s[q], i[q], O[r], k, rel=REL)


def _exact_scores(kind, n, rng):
    """Integers below 2^20 in magnitude whose order the select must reproduce, ties included."""
    if kind == "normal":
        v = np.round(rng.standard_normal(n) * 2e5)
    elif kind == "ties":         # a few distinct scores, the k-th among hundreds of equals
        v = np.round(rng.standard_normal(n) * 3) * 4096
    elif kind == "negative":     # the winners are the smallest magnitudes
        v = -np.abs(np.round(rng.standard_normal(n) * 2e5)) - 3
    elif kind == "ascending":    # the winners are the row's last entries
        v = np.arange(n) * (2 ** 20 - 1) // n
    elif kind == "equal":
        v = np.full(n, 77)
    else:                        # one score far above a narrow crowd
        v = rng.integers(500_000, 500_400, n)
        v[n // 3] = 2 ** 20 - 1
    return np.clip(v, -2 ** 20, 2 ** 20 - 1).astype(np.int64)


@pytest.mark.parametrize("nq,n,k", [
    (2, 64, 64), (2, 1025, 129), (2, 8192, 1000), (2, 8193, 1000),  # whole-row lists, then streams
    (1, 59_999, 128), (1, 60_000, 129), (3, 60_001, 1), (2, 300_003, 1024),  # then slices
    (64, 70_000, 10), (65, 70_000, 10),                               # ... of at most 64 rows
])
@pytest.mark.parametrize("kind", ["normal", "ties", "negative", "ascending", "equal", "outlier"])
def test_dense_topk_select(nq, n, k, kind):
    # scores of 20 bits, exact in fp32: the list must be exactly the sorted order (score desc,
    # index asc), whatever the spread of the scores, on every path of the select
    rng = np.random.default_rng(n + k)
    v = _exact_scores(kind, n, rng)
    X = np.zeros((n, 8), dtype=np.float16)
    X[:, 0], X[:, 1] = v >> 10, v & 1023
    Q = np.zeros((nq, 8), dtype=np.float16)
    Q[:, 0], Q[:, 1] = 1.0, 2.0 ** -10
    Q[1::2] *= -1  # the other queries rank by the negated scores
    s, i = hpr.dense_ip_topk(torch.from_numpy(Q).to(DEV), torch.from_numpy(X).to(DEV), k)
    s, i = s.cpu().numpy(), i.cpu().numpy()
    for q in range(nq):
        sign = -1 if q % 2 else 1
        order = np.lexsort((np.arange(n), -sign * v))[:k]
        assert np.array_equal(i[q], order), f"query {q}"
        assert np.array_equal(s[q] * 1024, sign * v[order])


@pytest.mark.parametrize("nq,n,dim,k,stored", [
    (600, 131_072, 8, 10, True),  # no longer than the sample, though more than 2^26 scores
    (2, 1 << 21, 8, 10, True), (2, (1 << 21) + 1, 8, 10, False),
    (129, 520_222, 16, 10, True), (129, 520_224, 16, 10, False),  # 2^26 scores
    (129, 520_222, 2048, 1, True), (128, 262_144, 2048, 1, True), (128, 262_870, 2048, 1, False),
    (64, 788_000, 200, 10, True), (64, 790_000, 200, 10, False), (64, 790_000, 200, 97, True),
    (32, 850_000, 256, 10, True), (32, 855_000, 256, 10, False),
])
def test_bench_names_the_launch_that_scores(nq, n, dim, k, stored):
    # every line between the stored scores and the filter; the benchmark's FLOPs and times are those
    # of the launch that ran; either way the lists are exact
    import bench
    Q, X = _device_rows(nq, dim, 91), _device_rows(n, dim, 92)
    hpr.kernel_timing(True)
    for name in ("dense_sample", "dense_scan"):
        hpr.kernel_timing_read(name)
    s, i = hpr.dense_ip_topk(Q, X, k)
    sample, scan = [hpr.kernel_timing_read(name)[1] for name in ("dense_sample", "dense_scan")]
    hpr.kernel_timing(False)
    assert (sample, scan) == (1, 0 if stored else 1)
    assert bench.dense_scored_rows(nq, n, dim, k) == (n if stored else n - SAMPLE_ROWS, stored)
    assert stored != _filtered(nq, n, dim, k)
    O = _scores64(Q[nq - 1:], X)
    check_topk(s[nq - 1].cpu().numpy(), i[nq - 1].cpu().numpy(), O[0], k, rel=REL)


def _topk_us(Qd, Xd, k):
    hpr.dense_ip_topk(Qd, Xd, k)
    hpr.kernel_timing(True)
    hpr.kernel_timing_read("topk")
    us = []
    for _ in range(5):
        hpr.dense_ip_topk(Qd, Xd, k)
        us.append(1e3 * hpr.kernel_timing_read("topk")[0])
    hpr.kernel_timing(False)
    return min(us)


@pytest.mark.parametrize("nq,n,k,cluster", [
    (64, 1_000_000, 100, 200), (64, 300_000, 100, 100), (512, 131_072, 100, 200),
    (64, 1_000_000, 1000, 400),
])
def test_dense_topk_of_clustered_rows(nq, n, k, cluster):
    # a paper's chunks lie together: rows whose best scores are neighbours give the same lists as
    # the shuffled store, and do not send the select through its slow path (15 to 25 times as long)
    g = torch.Generator(device=DEV).manual_seed(n + nq)
    Q = synth.unit_rows(nq, 64, g, DEV, torch.float16)
    X = synth.unit_rows(n, 64, g, DEV, torch.float16)
    first = torch.randperm(n // cluster - 1, generator=g, device=DEV)[:nq] * cluster + 37
    for q, a in enumerate(first.tolist()):
        x = Q[q].float() + 0.06 * torch.randn((cluster, 64), generator=g, device=DEV)
        X[a:a + cluster] = synth._normalise(x).to(torch.float16)
    P = X[torch.randperm(n, generator=g, device=DEV)].contiguous()
    s, i = hpr.dense_ip_topk(Q, X, k)
    sp, _ = hpr.dense_ip_topk(Q, P, k)
    assert torch.equal(s, sp)
    inside = (i >= first[:, None]) & (i < first[:, None] + cluster)
    assert bool((inside[:, :min(k, cluster)].float().mean(1) > 0.9).all())
    clustered, shuffled = _topk_us(Q, X, k), _topk_us(Q, P, k)
    assert clustered <= 3.0 * shuffled, (clustered, shuffled)


@pytest.mark.parametrize("nq,n,filtered", [(2, 1 << 21, False), (2, (1 << 21) + 1, True),
                                           (3, 10_000_019, True)])
def test_dense_topk_long_store(nq, n, filtered):
    # few queries over a long store: exact order on both sides of the longest stored rows, and the
    # filter beyond (the select alone would have one workgroup walk a row of ten million)
    k = 100
    v = _exact_scores("normal", n, np.random.default_rng(n))
    X = np.zeros((n, 8), dtype=np.float16)
    X[:, 0], X[:, 1] = v >> 10, v & 1023
    Q = np.zeros((nq, 8), dtype=np.float16)
    Q[:, 0], Q[:, 1] = 1.0, 2.0 ** -10
    Q[1::2] *= -1
    Qd, Xd = torch.from_numpy(Q).to(DEV), torch.from_numpy(X).to(DEV)
    hpr.kernel_timing(True)
    hpr.kernel_timing_read("dense_scan")
    s, i = hpr.dense_ip_topk(Qd, Xd, k)
    scans = hpr.kernel_timing_read("dense_scan")[1]
    hpr.kernel_timing(False)
    assert scans == (1 if filtered else 0)
    s, i = s.cpu().numpy(), i.cpu().numpy()
    for q in range(nq):
        sign = -1 if q % 2 else 1
        order = np.argsort(-sign * v, kind="stable")[:k]
        assert np.array_equal(i[q], order), f"query {q}"
        assert np.array_equal(s[q] * 1024, sign * v[order])


def test_dense_topk_planted_rows_rank_first():
    w = synth.dense_retrieval(seed=0, device=DEV, nq=512, n=300_000, dim=512, k=10, n_planted=200)
    s, i = hpr.dense_ip_topk(w["Q"], w["X"], w["k"])
    pq, pr = w["planted_q"].cpu().numpy(), w["planted_row"].cpu().numpy()
    s, i = s.cpu().numpy(), i.cpu().numpy()
    assert np.array_equal(i[pq, 0], pr)
    assert np.all(np.abs(s[pq, 0] - w["cosine"]) < 3e-3)
    Qh = _f16(w["Q"][torch.as_tensor(pq[:8])])
    Xh = _f16(w["X"][torch.as_tensor(pr[:8])])
    o = np.sum(Qh * Xh, axis=1)
    assert np.all(np.abs(s[pq[:8], 0] - o) <= REL * np.abs(o))


def test_dense_topk_workspace_and_errors():
    Q, X = _rows(4, 64, 31).to(DEV), _rows(100, 64, 32).to(DEV)
    with pytest.raises(hpr.HprError) as e:
        hpr.dense_ip_topk(Q, X, 101)
    assert e.value.status_name == "HPR_ERR_INVALID_ARG"
    with pytest.raises(hpr.HprError) as e:
        hpr.dense_ip_topk(Q[:, :60].contiguous(), X[:, :60].contiguous(), 5)
    assert e.value.status_name == "HPR_ERR_UNSUPPORTED_SHAPE"
    ws = hpr.dense_workspace(Q, X, 5)
    s1, i1 = hpr.dense_ip_topk(Q, X, 5, ws=ws)
    s2, i2 = hpr.dense_ip_topk(Q, X, 5, ws=ws)
    assert torch.equal(s1, s2) and torch.equal(i1, i2)


@pytest.mark.parametrize("n", [8_000, 20_000, 70_000])
def test_dense_store_all_infinite_and_nan_rows(n):
    """Rows of infinite and NaN scores, in lists held whole, streamed, and streamed in slices: an
    infinity orders as a number, a NaN by its sign above or below all of them, at every size."""
    nq, dim, k = 3, 64, 40
    Q, X = _rows(nq, dim, 71), _rows(n, dim, 72)
    Q[:, 0] = 0.5
    nans, inf, ninf = [17, n - 2], n // 2, n // 3
    special = nans + [inf, ninf]
    X[special] = 0.0
    O = oracle.dense_scores(_f16(Q), _f16(X))
    O[:, special] = -1e6
    X[inf, 0], X[ninf, 0] = float("inf"), float("-inf")
    X[nans, 0] = float("nan")
    s, i = hpr.dense_ip_topk(Q.to(DEV), X.to(DEV), k)
    s, i = s.cpu().numpy(), i.cpu().numpy()
    some, _ = hpr.dense_ip_topk(Q.to(DEV), X[:64].to(DEV), 64)  # the sign this unit gives a NaN
    above = bool(torch.isnan(some[0, 0]).item())
    lead = (nans if above else []) + [inf]
    for q in range(nq):
        assert i[q, :len(lead)].tolist() == lead
        assert np.isnan(s[q]).sum() == len(lead) - 1 and s[q, len(lead) - 1] == np.inf
        check_topk(s[q, len(lead):], i[q, len(lead):], O[q], k - len(lead), rel=REL)
