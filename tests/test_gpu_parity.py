"""GPU parity: every entry point of the HIP library against the fp64 oracle on seeded inputs.

Tolerances (scores and loss): |gpu - oracle| <= 2e-3 * max(|oracle|, 1e-3), the stated bound
for bf16 inputs with fp32 accumulation; a 20x tighter check (1e-4) is also asserted on
MaxSim scores because bf16 x bf16 products are exact in fp32 and only the fp32 summation differs
from the oracle.  Gradients: relative L2 error <= 2e-3 per tensor and per row (tests/grad_check.py:
a row's bound widens only by what argmax near-ties may legitimately move).  Top-k lists: the rules of
tests/topk_check.py.  Integer outputs (argmax-dependent structure, indices of clear winners)
are compared exactly.
"""

import math

import numpy as np
import pytest
import torch

import oracle
import paper_2505_04846_amd as hpr
import synth
from grad_check import check_rows, conditioning_allowance, near_tie_allowance
from topk_check import check_topk

pytestmark = pytest.mark.gpu

REL = 2e-3
DEV = "cuda:0"


def _bf(t):
    return oracle.decode_bf16(t.detach().cpu().contiguous().view(torch.int16).numpy())


def _assert_close(g, o, rel=REL, what=""):
    g = np.asarray(g, dtype=np.float64)
    o = np.asarray(o, dtype=np.float64)
    err = np.abs(g - o)
    lim = rel * np.maximum(np.abs(o), 1e-3)
    bad = err > lim
    assert not bad.any(), (f"{what}: {bad.sum()} of {bad.size} outside rel {rel}; worst "
                           f"{(err / lim).max():.3g}x the bound")


def _rel_l2(g, o):
    g = np.asarray(g, dtype=np.float64)
    o = np.asarray(o, dtype=np.float64)
    return float(np.linalg.norm(g - o) / max(np.linalg.norm(o), 1e-300))


def _ragged(seed, nq, lq, lens, dim):
    g = torch.Generator().manual_seed(seed)
    lens = torch.tensor(lens, dtype=torch.int64)
    off = synth.csr_offsets(lens)
    Q = synth.unit_rows(nq * lq, dim, g, "cpu", torch.bfloat16).reshape(nq, lq, dim)
    D = synth.unit_rows(int(off[-1]), dim, g, "cpu", torch.bfloat16)
    return Q, D, off


def _to_dev(*ts):
    return [t.to(DEV) for t in ts]


# ------------------------------------------------------------------------------ MaxSim scores

def test_tiny_maxsim_scores_match_oracle():
    w = synth.tiny_maxsim(seed=0)
    Q, D, off = _to_dev(w["Q"], w["D"], w["off"])
    S = hpr.maxsim_score(Q, D, off).cpu().numpy()
    O = oracle.maxsim_scores(_bf(w["Q"]), _bf(w["D"]), w["off"].numpy())
    _assert_close(S, O, what="scores")
    _assert_close(S, O, rel=1e-4, what="scores (tight)")
    # quantisation effect of rounding the fp32 tokens to bf16, reported against the fp32 oracle
    O32 = oracle.maxsim_scores(w["Q_f32"].numpy().astype(np.float64),
                               w["D_f32"].numpy().astype(np.float64), w["off"].numpy())
    _assert_close(S, O32, what="scores vs fp32-token oracle")


@pytest.mark.parametrize("nq,lq,lens,dim", [
    (1, 1, [1], 8),
    (3, 1, [1, 2, 3, 16, 17], 16),
    (2, 3, [5, 1, 31, 32, 33], 64),
    (5, 17, [15, 16, 17, 100, 1, 300], 128),
    (9, 32, [513, 7, 64, 200], 128),
    (4, 100, [40, 41], 64),
    (3, 64, [20, 260, 3], 128),
    (3, 100, [40, 300, 7], 128),
    (2, 128, [70, 33, 1], 128),
    (5, 96, [64, 65], 120),
    (2, 128, [9, 70], 48),
    (6, 64, [33, 1, 90], 256),
    (2, 33, [50, 17], 192),
    (17, 8, list(range(1, 40)), 32),
])
def test_maxsim_scores_edge_shapes(nq, lq, lens, dim):
    Q, D, off = _ragged(100 + nq + lq + dim, nq, lq, lens, dim)
    S = hpr.maxsim_score(*_to_dev(Q, D, off)).cpu().numpy()
    O = oracle.maxsim_scores(_bf(Q), _bf(D), off.numpy())
    _assert_close(S, O, what="scores")
    _assert_close(S, O, rel=1e-4, what="scores (tight)")


@pytest.mark.parametrize("nq,lq,dim,n_docs", [
    (1, 32, 128, 5000),   # one block per wave: three idle waves per workgroup
    (4, 32, 128, 3000),   # one block per wave, every wave active
    (8, 32, 128, 3000),   # two blocks per wave
    (2, 40, 128, 2000),   # a 64-slot query needs two blocks whatever the slot count
    (1, 8, 64, 4000),
    (3, 20, 256, 2000),
    (6, 16, 32, 2500),
])
def test_maxsim_scores_few_queries(nq, lq, dim, n_docs):
    # few query slots select the variants with fewer query blocks per wave and more resident
    # workgroups; many documents give many short ranges
    g = torch.Generator().manual_seed(nq * 1000 + lq)
    lens = torch.randint(1, 300, (n_docs,), generator=g)
    Q, D, off = _ragged(nq + lq + dim, nq, lq, lens.tolist(), dim)
    S = hpr.maxsim_score(*_to_dev(Q, D, off)).cpu().numpy()
    O = oracle.maxsim_scores(_bf(Q), _bf(D), off.numpy())
    _assert_close(S, O, rel=1e-4, what="scores")
    s, i = hpr.maxsim_topk(*_to_dev(Q, D, off), 50)
    s, i = s.cpu().numpy(), i.cpu().numpy()
    for q in range(nq):
        check_topk(s[q], i[q], O[q], 50)


@pytest.mark.parametrize("nq,lq,dim,n_docs,ld_max", [
    (1, 32, 128, 1, 127),       # one range
    (1, 32, 128, 130, 2),       # 128-token ranges of many documents each
    (16, 32, 128, 50, 300),     # four blocks per wave cut to one to fill the chip
    (10, 64, 128, 20, 300),     # ... to two, a 64-slot query's least
    (3, 96, 128, 9, 100),       # three blocks per query: not cut
    (5, 33, 256, 30, 64),
    (1, 32, 128, 3000, 380),    # about one resident round: own ranges
    (40, 32, 128, 1100, 380),   # between one and two rounds: cut to whole ones
    (2, 32, 128, 9000, 380),    # several rounds: the partition table
    (12, 32, 128, 4000, 200), (20, 30, 96, 4000, 200), (9, 96, 128, 2500, 200),  # three blocks per
    (11, 32, 64, 4000, 200), (10, 25, 32, 4000, 200), (12, 32, 80, 3000, 200),   # wave, every staging
])
def test_maxsim_small_grids(nq, lq, dim, n_docs, ld_max):
    # the plans of calls that do not fill the chip with ranges of 1,024 tokens; the no-workspace
    # entry point takes the same plan, and the plan changes no score's bits
    g = torch.Generator().manual_seed(nq + n_docs)
    lens = torch.randint(1, ld_max + 1, (n_docs,), generator=g).tolist()
    Q, D, off = _ragged(7 + nq + n_docs, nq, lq, lens, dim)
    args = _to_dev(Q, D, off)
    S = hpr.maxsim_score(*args)
    O = oracle.maxsim_scores(_bf(Q), _bf(D), off.numpy())
    _assert_close(S.cpu().numpy(), O, rel=1e-4, what="scores")
    assert torch.equal(S, hpr.maxsim_score_noalloc(*args))
    half = (nq + 1) // 2
    assert torch.equal(S[:half], hpr.maxsim_score(args[0][:half].contiguous(), *args[1:]))


@pytest.mark.parametrize("nq,lq,dim", [
    (100, 20, 128), (70, 40, 128), (33, 33, 64), (200, 5, 128), (130, 16, 96), (70, 17, 256),
    (600, 24, 128), (2100, 42, 128),  # the last one: persistent passes
])
def test_maxsim_packed_queries(nq, lq, dim):
    # many queries whose length is no multiple of 32 share blocks of query slots; a call of few
    # queries gives each blocks of its own, and the scores must have the same bits
    g = torch.Generator().manual_seed(nq + lq)
    lens = torch.randint(1, 90, (230,), generator=g).tolist()
    Q, D, off = _ragged(nq * lq, nq, lq, lens, dim)
    Qd, Dd, od = _to_dev(Q, D, off)
    S = hpr.maxsim_score(Qd, Dd, od)
    pick = [0, 1, nq // 2, nq - 2, nq - 1]
    O = oracle.maxsim_scores(_bf(Q[pick]), _bf(D), off.numpy())
    _assert_close(S[pick].cpu().numpy(), O, rel=1e-4, what="scores")
    for q in range(0, nq, max(1, nq // 16)):
        assert torch.equal(S[q:q + 1], hpr.maxsim_score(Qd[q:q + 1].contiguous(), Dd, od))


@pytest.mark.parametrize("dim", [64, 88, 96, 104, 256])
@pytest.mark.parametrize("nq,lq", [(40, 32), (30, 20)])
def test_directly_staged_dims(dim, nq, lq):
    # dims 64, 96 and 256 stage their tiles straight into LDS when the queries are many (their
    # neighbours do not); documents ending at every row of a tile, scores and loss
    lens = list(range(1, 71))
    Q, D, off = _ragged(dim + nq, nq, lq, lens, dim)
    S = hpr.maxsim_score(*_to_dev(Q, D, off))
    O = oracle.maxsim_scores(_bf(Q), _bf(D), off.numpy())
    _assert_close(S.cpu().numpy(), O, rel=1e-4, what="scores")
    pos = torch.arange(nq, dtype=torch.int32) % len(lens)
    _loss_parity(Q, D, off, pos, 1.5625)


@pytest.mark.parametrize("nq,lq,dim", [(30, 20, 128), (50, 7, 64), (40, 21, 32)])
def test_loss_packed_queries(nq, lq, dim):
    g = torch.Generator().manual_seed(nq + lq)
    lens = torch.randint(1, 90, (61,), generator=g).tolist()
    Q, D, off = _ragged(nq * lq + 1, nq, lq, lens, dim)
    pos = torch.randint(0, len(lens), (nq,), generator=g, dtype=torch.int32)
    _loss_parity(Q, D, off, pos, 1.5625)
    Qd, Dd, od, pd = _to_dev(Q, D, off, pos)
    r = hpr.coltrast_loss_fwd_bwd(Qd, Dd, od, pd, 2.0, return_scores=True)
    assert torch.equal(r["scores"], hpr.maxsim_score(Qd, Dd, od))


@pytest.mark.parametrize("nq,n_docs,ld_max", [(3, 5, 40), (24, 48, 300), (100, 800, 40)])
def test_loss_small_grids(nq, n_docs, ld_max):
    # argmax ranges below 1,024 tokens, and a grid cut to one whole round (13 query groups)
    g = torch.Generator().manual_seed(nq)
    lens = torch.randint(1, ld_max + 1, (n_docs,), generator=g).tolist()
    Q, D, off = _ragged(nq, nq, 32, lens, 128)
    pos = torch.randint(0, n_docs, (nq,), generator=g, dtype=torch.int32)
    _loss_parity(Q, D, off, pos, 1.5625)


def test_maxsim_many_ranges_and_query_groups():
    # enough documents and queries for several document ranges and query workgroups
    g = torch.Generator().manual_seed(7)
    lens = torch.randint(1, 200, (3000,), generator=g)
    Q, D, off = _ragged(8, 70, 32, lens.tolist(), 128)
    S = hpr.maxsim_score(*_to_dev(Q, D, off)).cpu().numpy()
    O = oracle.maxsim_scores(_bf(Q), _bf(D), off.numpy())
    _assert_close(S, O, rel=1e-4, what="scores")


def test_maxsim_persistent_passes_match_oracle():
    # 1,024 queries of 64 tokens: 128 query groups of 8, two passes of the persistent grid (one
    # document range per XCD, checkpoint counters after the range table); the result must not
    # depend on the plan: the no-allocation entry point (its scratch holds the same table and
    # counters) gives the same bits
    g = torch.Generator().manual_seed(11)
    lens = torch.randint(1, 90, (420,), generator=g)
    Q, D, off = _ragged(12, 1024, 64, lens.tolist(), 128)
    Qd, Dd, od = _to_dev(Q, D, off)
    S = hpr.maxsim_score(Qd, Dd, od)
    S2 = hpr.maxsim_score_noalloc(Qd, Dd, od)
    assert torch.equal(S, S2)
    O = oracle.maxsim_scores(_bf(Q), _bf(D), off.numpy())
    _assert_close(S.cpu().numpy(), O, what="scores")
    # the tight diagnostic at 2e-4: over 430,080 scores the fp32 accumulation tail reaches 1e-4
    _assert_close(S.cpu().numpy(), O, rel=2e-4, what="scores (tight)")
    s, i = hpr.maxsim_topk(Qd, Dd, od, 40)
    s, i = s.cpu().numpy(), i.cpu().numpy()
    for q in (0, 7, 8, 511, 512, 1023):
        check_topk(s[q], i[q], O[q], 40)


def test_maxsim_document_token_order_is_bit_invariant():
    Q, D, off = _ragged(21, 6, 32, [70, 33, 128], 128)
    S1 = hpr.maxsim_score(*_to_dev(Q, D, off))
    perm = torch.cat([torch.randperm(int(off[d + 1] - off[d]),
                                     generator=torch.Generator().manual_seed(d)) + off[d]
                      for d in range(3)])
    S2 = hpr.maxsim_score(*_to_dev(Q, D[perm].contiguous(), off))
    S3 = hpr.maxsim_score(*_to_dev(Q, D, off))
    assert torch.equal(S1, S2), "permuting a document's tokens changed its score bits"
    assert torch.equal(S1, S3), "repeated call is not bit-identical"


def test_maxsim_doc_equal_to_query_scores_sum_of_squared_norms():
    Q, D, off = _ragged(22, 2, 32, [10], 128)
    D = torch.cat([Q[0], D, Q[1][:5]])        # doc 0 = query 0's tokens; doc 1 = noise + part of q1
    off = torch.tensor([0, 32, 32 + 15], dtype=torch.int64)
    S = hpr.maxsim_score(*_to_dev(Q, D, off)).cpu().numpy()
    q0 = _bf(Q[0])
    want = float(np.sum(q0 * q0))
    assert abs(S[0, 0] - want) <= 1e-4 * want
    assert abs(want - 32) < 32 * 2 ** -6


# ------------------------------------------------------------------------------ top-k

def test_tiny_maxsim_topk():
    w = synth.tiny_maxsim(seed=0)
    s, i = hpr.maxsim_topk(*_to_dev(w["Q"], w["D"], w["off"]), w["k"])
    O = oracle.maxsim_scores(_bf(w["Q"]), _bf(w["D"]), w["off"].numpy())
    s, i = s.cpu().numpy(), i.cpu().numpy()
    exact = 0
    for q in range(O.shape[0]):
        r = check_topk(s[q], i[q], O[q], w["k"])
        exact += r["exact"]
    assert exact == O.shape[0]


@pytest.mark.parametrize("n_docs,k", [(1, 1), (7, 7), (300, 1), (300, 300), (2500, 1000),
                                      (5000, 1024)])
def test_maxsim_topk_edges(n_docs, k):
    g = torch.Generator().manual_seed(n_docs + k)
    lens = torch.randint(1, 40, (n_docs,), generator=g)
    Q, D, off = _ragged(n_docs, 3, 8, lens.tolist(), 64)
    s, i = hpr.maxsim_topk(*_to_dev(Q, D, off), k)
    O = oracle.maxsim_scores(_bf(Q), _bf(D), off.numpy())
    s, i = s.cpu().numpy(), i.cpu().numpy()
    for q in range(3):
        check_topk(s[q], i[q], O[q], k)


def test_topk_duplicate_documents_lower_index_first():
    Q, D, off = _ragged(31, 2, 16, [20, 30, 25], 128)
    # docs 0, 2, 4 identical (bit-equal scores); docs 1, 3 other
    toks = [D[0:20], D[20:50], D[0:20], D[50:75], D[0:20]]
    D2 = torch.cat(toks)
    off2 = synth.csr_offsets(torch.tensor([20, 30, 20, 25, 20]))
    S = hpr.maxsim_score(*_to_dev(Q, D2, off2))
    assert torch.equal(S[:, 0], S[:, 2]) and torch.equal(S[:, 0], S[:, 4])
    s, i = hpr.maxsim_topk(*_to_dev(Q, D2, off2), 5)
    for q in range(2):
        pos = [int(x) for x in i[q].tolist()]
        assert pos.index(0) < pos.index(2) < pos.index(4)
        # exact order under (score desc, idx asc) using the GPU's own scores
        Sq = S[q].cpu().numpy()
        assert pos == sorted(range(5), key=lambda d: (-Sq[d], d))


def test_topk_all_equal_scores_returns_lowest_indices():
    Q, D, off = _ragged(32, 1, 4, [3], 32)
    D2 = torch.cat([D] * 50)
    off2 = synth.csr_offsets(torch.full((50,), 3))
    s, i = hpr.maxsim_topk(*_to_dev(Q, D2, off2), 17)
    assert i[0].tolist() == list(range(17))
    assert torch.all(s[0] == s[0, 0])



@pytest.mark.parametrize("n_docs,k", [(9000, 10), (20000, 100), (40000, 1000)])
def test_topk_streaming_select_long_rows(n_docs, k):
    # rows longer than the LDS candidate list: sampled threshold, one streaming pass
    g = torch.Generator().manual_seed(n_docs + k)
    lens = torch.randint(1, 6, (n_docs,), generator=g)
    Q, D, off = _ragged(n_docs + k, 3, 4, lens.tolist(), 32)
    s, i = hpr.maxsim_topk(*_to_dev(Q, D, off), k)
    O = oracle.maxsim_scores(_bf(Q), _bf(D), off.numpy())
    s, i = s.cpu().numpy(), i.cpu().numpy()
    for q in range(3):
        check_topk(s[q], i[q], O[q], k)


def test_topk_long_row_of_equal_scores_takes_exact_path():
    # every entry ties with the sampled threshold, so the candidate list overflows and the row
    # is selected by the exact multi-pass path: the lowest indices win
    Q, D, off = _ragged(33, 1, 4, [3], 32)
    n = 20000
    D2 = torch.cat([D] * n)
    off2 = synth.csr_offsets(torch.full((n,), 3))
    s, i = hpr.maxsim_topk(*_to_dev(Q, D2, off2), 1000)
    assert i[0].tolist() == list(range(1000))
    assert torch.all(s[0] == s[0, 0])


def test_topk_unrepresentative_sample_takes_exact_path():
    # the documents the sampler reads (nr = ceil(n / 4096) runs of 64 starting at 16-byte
    # vector r * (n / 4) / nr of the row, which is 16-byte aligned here) score highest and are
    # the only high ones: the threshold then admits fewer than k candidates and the exact path
    # runs
    n, k, lq, dim = 300_000, 1000, 4, 32
    nv, nr = n // 4, min(256, (n + 4095) // 4096)
    sampled = np.array(sorted({4 * ((u >> 4) * nv // nr + (u & 15)) + c
                               for u in range(16 * nr) for c in range(4)}))
    g = torch.Generator().manual_seed(5)
    Q = synth.unit_rows(lq, dim, g, "cpu", torch.bfloat16).reshape(1, lq, dim)
    D = synth.unit_rows(n, dim, g, "cpu", torch.float32)
    noise = synth.unit_rows(sampled.size, dim, g, "cpu", torch.float32)
    qsum = Q[0].float().sum(0)
    D[torch.as_tensor(sampled)] = synth._normalise(qsum[None] / qsum.norm() + 0.3 * noise)
    D = D.to(torch.bfloat16)
    off = synth.csr_offsets(torch.ones(n, dtype=torch.int64))
    s, i = hpr.maxsim_topk(*_to_dev(Q, D, off), k)
    # one token per document: the MaxSim score is <sum_i q_i, d> (the pinned Ld = 1 closed form)
    O = oracle.dense_scores(_bf(Q)[0].sum(0)[None], _bf(D))
    check_topk(s.cpu().numpy()[0], i.cpu().numpy()[0], O[0], k)
    assert set(i.cpu().numpy()[0].tolist()) <= set(sampled.tolist())

# ------------------------------------------------------------------------------ InfoNCE loss

def _loss_parity(Q, D, off, pos, scale, rel_grad=REL, max_allowed=0.5):
    r = hpr.coltrast_loss_fwd_bwd(*_to_dev(Q, D, off, pos), scale, return_scores=True)
    Qo, Do = _bf(Q), _bf(D)
    o = oracle.coltrast_li_loss(Qo, Do, off.numpy(), pos.numpy(), scale)
    _assert_close(r["scores"].cpu().numpy(), o["S"], rel=1e-4, what="scores")
    _assert_close(r["loss"].cpu().numpy()[0], o["loss"], what="loss")
    dq, dd = r["dq"].cpu().numpy(), r["dd"].cpu().numpy()
    e_dq = _rel_l2(dq, o["dQ"])
    e_dd = _rel_l2(dd, o["dD"])
    assert e_dq <= rel_grad, f"dQ rel L2 {e_dq:.3g}"
    assert e_dd <= rel_grad, f"dD rel L2 {e_dd:.3g}"
    # every row on its own: rel L2 2e-3, widened only by what argmax near-ties may move
    aq, ad, _ = near_tie_allowance(Qo, Do, off.numpy(), o["G"])
    cq, cd = conditioning_allowance(Qo, Do, off.numpy(), o["G"], o["A"],
                                    r["scores"].cpu().numpy() - o["S"], scale)
    fq = check_rows(dq, o["dQ"], aq, "dQ rows", rel_grad, cond=cq)
    fd = check_rows(dd, o["dD"], ad, "dD rows", rel_grad, cond=cd)
    assert fq <= max_allowed and fd <= max_allowed, (fq, fd)
    return r, o


@pytest.mark.parametrize("scale", [50.0, 1.5625])
def test_coltrast_step_loss_and_grads(scale):
    w = synth.coltrast_step(seed=0)
    r, o = _loss_parity(w["Q"], w["D"], w["off"], w["pos"], scale)
    if scale == 1.5625:
        assert abs(o["loss"] - 0.6385) < 0.01   # the recipe's expected magnitude
    # rows the oracle's argmax never selects are zero on the GPU too, except where a near-tie
    # (within fp32 rounding of the two dot products) sent the selection to another token
    zero_rows = ~np.any(o["dD"] != 0, axis=1)
    assert zero_rows.any()
    g_rows = r["dd"].cpu().numpy()[zero_rows]
    moved = np.any(g_rows != 0, axis=1)
    assert moved.sum() <= 1e-3 * zero_rows.sum(), f"{moved.sum()} unselected rows non-zero"
    assert np.linalg.norm(g_rows) <= 2e-3 * np.linalg.norm(o["dD"])


@pytest.mark.parametrize("nq,lq,lens,dim,scale", [
    (1, 1, [1, 1], 8, 1.0),
    (3, 5, [4, 9, 1, 17], 16, 2.0),
    (4, 17, [33, 16, 5, 70, 8], 64, 0.7),
    (6, 32, [100, 1, 47, 256, 300, 12, 64], 128, 10.0),
    (2, 32, [20, 21, 22], 256, 3.0),
    (3, 64, [70, 5, 33], 128, 2.0),
])
def test_loss_small_shapes(nq, lq, lens, dim, scale):
    Q, D, off = _ragged(nq * 7 + lq, nq, lq, lens, dim)
    g = torch.Generator().manual_seed(nq)
    pos = torch.randint(0, len(lens), (nq,), generator=g, dtype=torch.int32)
    _loss_parity(Q, D, off, pos, scale)


def test_loss_over_thousands_of_short_documents():
    # 40 queries x 4,000 documents of 1-6 tokens: InfoNCE rows of 4,000 scores, argmax ranges
    # of hundreds of documents, dD over many tiny documents
    nq, lq = 40, 8
    g = torch.Generator().manual_seed(41)
    lens = torch.randint(1, 7, (4000,), generator=g).tolist()
    Q, D, off = _ragged(41, nq, lq, lens, 64)
    pos = torch.randint(0, len(lens), (nq,), generator=g, dtype=torch.int32)
    _loss_parity(Q, D, off, pos, 2.0)


def test_loss_dim128_documents_ending_at_every_row_of_a_tile():
    # at dim 128 the argmax kernel stages four tiles per stage straight into LDS: documents of
    # 1-160 tokens end at every row of a tile and at every tile of a stage, and a stage holds
    # tiles of several documents
    nq, lq = 12, 32
    g = torch.Generator().manual_seed(43)
    lens = list(range(1, 161)) + torch.randint(1, 200, (60,), generator=g).tolist()
    Q, D, off = _ragged(43, nq, lq, lens, 128)
    pos = torch.randint(0, len(lens), (nq,), generator=g, dtype=torch.int32)
    _loss_parity(Q, D, off, pos, 5.0)


@pytest.mark.parametrize("nq,lq", [(200, 32), (470, 32)])
def test_loss_many_query_tokens(nq, lq):
    # 6,400 and 15,040 (query, token) entries: the dD kernel's LDS no longer fits two 512-thread
    # workgroups per CU, so it takes its 256-thread form with more than 64 KiB of dynamic LDS;
    # 15,040 entries is close to the largest size the host accepts (about 15,300 at nq = 470)
    Q, D, off = _ragged(nq + lq, nq, lq, [40, 300, 7, 129, 64, 250, 33, 1, 90, 180, 256, 12], 128)
    pos = torch.randint(0, 12, (nq,), generator=torch.Generator().manual_seed(nq),
                        dtype=torch.int32)
    _loss_parity(Q, D, off, pos, 1.5625)


@pytest.mark.parametrize("dim", [32, 128, 256])
def test_loss_argmax_ties_go_to_the_lowest_token(dim):
    # Bit-identical copies of one token sit in the same lane (rows 1 and 9), in the other
    # half-wave (row 5), in later tiles (rows 33, 62) and at the document's last row (69, whose
    # copies also fill the padding of the partial last tile).  Document 0's copies hold query
    # token 0's and 1's maximum with a positive product; document 1's hold query token 2's and
    # 3's maximum with every product of the document negative (the sign-flipped argmax keys).
    # The whole subgradient must reach the lowest copy, row 1, and nothing the other copies.
    g = torch.Generator().manual_seed(dim)
    L = 70
    copies = [1, 5, 9, 33, 62, 69]

    def unit(x):
        return x / x.norm(dim=-1, keepdim=True)

    t0 = unit(torch.randn(dim, generator=g))
    t1 = unit(torch.randn(dim, generator=g))
    q = torch.stack([unit(t0 + 0.1 * torch.randn(dim, generator=g)),
                     unit(t0 + 0.1 * torch.randn(dim, generator=g)),
                     unit(-t1 + 0.1 * torch.randn(dim, generator=g)),
                     unit(-t1 + 0.1 * torch.randn(dim, generator=g))])
    # document 0: random tokens far from t0 (products with q[0], q[1] near 0)
    d0 = unit(torch.randn(L, dim, generator=g))
    # document 1: tokens close to -q[2], -q[3] (products near -1), and copies of a token whose
    # products with q[2], q[3] are negative but larger
    d1 = unit(-(q[2] + q[3])[None] + 0.05 * torch.randn(L, dim, generator=g))
    c1 = unit(0.5 * t1 + unit(torch.randn(dim, generator=g)))
    d2 = unit(torch.randn(L, dim, generator=g))
    D = torch.cat([d0, d1, d2]).to(torch.bfloat16)
    c0b, c1b = t0.to(torch.bfloat16), c1.to(torch.bfloat16)
    for r in copies:
        D[r] = c0b
        D[L + r] = c1b
    Q = q.to(torch.bfloat16)[None]
    off = synth.csr_offsets(torch.full((3,), L, dtype=torch.int64))
    pos = torch.tensor([2], dtype=torch.int32)
    o = oracle.coltrast_li_loss(_bf(Q), _bf(D), off.numpy(), pos.numpy(), 1.0)
    # the constructed maxima: document 0's copies for tokens 0, 1, document 1's for 2, 3
    assert list(o["A"][0, :2, 0]) == [1, 1] and list(o["A"][0, 2:, 1]) == [1, 1]
    qd = _bf(Q)[0, 2:] @ _bf(D)[L:2 * L].T  # every product behind document 1's maxima < 0
    assert np.all(qd < 0)
    r = hpr.coltrast_loss_fwd_bwd(*_to_dev(Q, D, off, pos), 1.0)
    dd = r["dd"].cpu().numpy()
    for base in (0, L):
        assert np.any(dd[base + 1] != 0), "the lowest copy received no gradient"
        for c in copies[1:]:
            assert not np.any(dd[base + c] != 0), f"copy at row {c} of doc {base // L} chosen"
    assert _rel_l2(dd, o["dD"]) <= REL and _rel_l2(r["dq"].cpu().numpy(), o["dQ"]) <= REL


def test_loss_ranges_inside_a_long_document_and_over_many_tiny_ones():
    # The argmax kernel splits the tokens into equal ranges and each workgroup searches the
    # offsets for the documents that start in its range.  A 20,000-token document among short
    # ones leaves ~18 of 28 ranges without a document; 20,000 documents of one or two tokens
    # take three rounds of the search.
    g = np.random.default_rng(7)
    lens_a = g.integers(1, 300, 30).tolist() + [20_000] + g.integers(1, 300, 30).tolist()
    lens_b = g.integers(1, 3, 20_000).tolist()
    for seed, lens in ((1, lens_a), (2, lens_b)):
        Q, D, off = _ragged(seed, 2, 32, lens, 64)
        pos = torch.tensor([0, len(lens) - 1], dtype=torch.int32)
        _loss_parity(Q, D, off, pos, 2.0)


@pytest.mark.parametrize("dim", [8, 128])  # tiles staged through VGPRs / straight into LDS
def test_loss_document_length_limit(dim):
    # 65,536 tokens is the longest document whose argmax offsets fit 16 bits: such a document
    # is scored exactly; one token more and its scores, and hence the loss, are NaN.
    Q, D, off = _ragged(3, 2, 4, [10, 65_536, 10], dim)
    pos = torch.tensor([0, 2], dtype=torch.int32)
    _loss_parity(Q, D, off, pos, 1.0)
    Q, D, off = _ragged(4, 2, 4, [10, 65_537, 10], dim)
    r = hpr.coltrast_loss_fwd_bwd(*_to_dev(Q, D, off, pos), 1.0, return_scores=True)
    s = r["scores"].cpu().numpy()
    assert np.all(np.isnan(s[:, 1])) and math.isnan(float(r["loss"].item()))
    o = oracle.maxsim_scores(_bf(Q), _bf(D), off.numpy())
    _assert_close(s[:, [0, 2]], o[:, [0, 2]], rel=1e-4, what="scores")


@pytest.mark.parametrize("nq,lq,dim", [(12, 32, 128), (3, 20, 128), (9, 64, 128), (6, 17, 64),
                                       (5, 32, 32), (4, 30, 256)])
def test_loss_scores_equal_maxsim_score_bits(nq, lq, dim):
    # The loss's argmax kernel and the score kernel take each tile's maximum in a different
    # order but of the same fp32 products, and sum the query slots in the same fixed order: the
    # scores the loss returns are maxsim_score's, bit for bit (different staging variants
    # included: at dim 128 the first case takes the score kernel's directly staged one)
    g = torch.Generator().manual_seed(nq * 1000 + lq + dim)
    lens = torch.randint(1, 300, (57,), generator=g).tolist()
    Q, D, off = _ragged(nq + dim, nq, lq, lens, dim)
    pos = torch.randint(0, len(lens), (nq,), generator=g, dtype=torch.int32)
    Qd, Dd, od, pd = _to_dev(Q, D, off, pos)
    r = hpr.coltrast_loss_fwd_bwd(Qd, Dd, od, pd, 2.0, return_scores=True)
    assert torch.equal(r["scores"], hpr.maxsim_score(Qd, Dd, od))


def test_loss_grads_optional_and_deterministic():
    w = synth.coltrast_step(seed=1, nq=8, n_neg=3, ld=64)
    args = _to_dev(w["Q"], w["D"], w["off"], w["pos"])
    full = hpr.coltrast_loss_fwd_bwd(*args, 1.5625)
    again = hpr.coltrast_loss_fwd_bwd(*args, 1.5625)
    for key in ("loss", "dq", "dd"):
        assert torch.equal(full[key], again[key]), f"{key} not bit-reproducible"
    only_q = hpr.coltrast_loss_fwd_bwd(*args, 1.5625, need_dd=False)
    only_d = hpr.coltrast_loss_fwd_bwd(*args, 1.5625, need_dq=False)
    assert only_q["dd"] is None and only_d["dq"] is None
    assert torch.equal(only_q["dq"], full["dq"]) and torch.equal(only_d["dd"], full["dd"])
    assert torch.equal(only_q["loss"], full["loss"])


def test_loss_bad_positive_gives_nan():
    w = synth.coltrast_step(seed=2, nq=4, n_neg=1, ld=32)
    pos = w["pos"].clone()
    pos[1] = 10_000
    args = _to_dev(w["Q"], w["D"], w["off"], pos)
    r = hpr.coltrast_loss_fwd_bwd(*args, 1.0, return_scores=True)
    assert math.isnan(float(r["loss"].item()))
    # the scores are still returned whole, the bad row's included
    assert torch.equal(r["scores"], hpr.maxsim_score(*args[:3]))
    # the bad row's G is zero: its query tokens get no MaxSim gradient
    assert not bool(r["dq"][1].any())


def test_autograd_function_matches_fwd_bwd_and_scales():
    w = synth.coltrast_step(seed=3, nq=4, n_neg=3, ld=32)
    Q = w["Q"].to(DEV).requires_grad_(True)
    D = w["D"].to(DEV).requires_grad_(True)
    off, pos = _to_dev(w["off"], w["pos"])
    loss = hpr.coltrast_loss(Q, D, off, pos, 1.5625)
    (3.0 * loss).backward()
    ref = hpr.coltrast_loss_fwd_bwd(Q.detach(), D.detach(), off, pos, 1.5625)
    assert torch.allclose(Q.grad.float(), (3.0 * ref["dq"]).bfloat16().float())
    assert torch.allclose(D.grad.float(), (3.0 * ref["dd"]).bfloat16().float())
    assert float(loss.detach()) == float(ref["loss"][0])


@pytest.mark.parametrize("n_q,n_d,shift", [(8, 0, 0), (0, 40, 0), (64, 8 * 300_007, 0),
                                           (7, 1000, 0), (64, 64, 1)])
def test_scaled_gradients_equal_a_rounded_product(n_q, n_d, shift):
    # the vector path, one array only, more values than one round of workgroups, and the
    # value-by-value path (odd lengths, an unaligned array), with the specials bf16 rounding meets
    g = torch.Generator().manual_seed(n_q + n_d)
    special = torch.tensor([0.0, -0.0, float("inf"), float("-inf"), float("nan"), 1e-45, -3e-39,
                            3.4e38, 1.00390625, 1.01171875, -1e-20])
    scale = torch.tensor(0.37, device=DEV)

    def grad(n):
        x = torch.randn(n + shift, generator=g)
        m = min(n, special.numel())
        x[shift:shift + m] = special[:m]
        return x.to(DEV)[shift:] if n else None

    dq, dd = grad(n_q), grad(n_d)
    for src, out in zip((dq, dd), hpr._scaled_grads(dq, dd, scale)):
        if src is None:
            assert out is None
            continue
        ref = (src * scale).to(torch.bfloat16)
        assert torch.equal(out.view(torch.int16), ref.view(torch.int16))


@pytest.mark.parametrize("n", [1, 5, 1_000_003])
def test_scale_in_place(n):
    g = torch.Generator().manual_seed(n)
    x = torch.randn(n, generator=g).to(DEV)
    scale = torch.tensor([-0.37], device=DEV)
    ref = x * scale
    assert hpr.scale_(x, scale) is x and torch.equal(x, ref)


def test_autograd_second_backward_over_a_retained_graph():
    # each backward scales the forward's gradients by its own upstream gradient (the saved
    # tensors are not scaled in place, which would compound the two upstream gradients)
    w = synth.coltrast_step(seed=3, nq=4, n_neg=3, ld=32)
    Q = w["Q"].to(DEV).requires_grad_(True)
    D = w["D"].to(DEV).requires_grad_(True)
    off, pos = _to_dev(w["off"], w["pos"])
    ref = hpr.coltrast_loss_fwd_bwd(Q.detach(), D.detach(), off, pos, 1.5625)
    ref_t = hpr.coltrast_total_loss_fwd_bwd(Q.detach(), D.detach(), off, pos, 1.5625, 0.05)
    for fn, r in ((lambda: hpr.coltrast_loss(Q, D, off, pos, 1.5625), ref),
                  (lambda: hpr.coltrast_total_loss(Q, D, off, pos, 1.5625, 0.05), ref_t)):
        loss = fn()
        gq1, gd1 = torch.autograd.grad(5.0 * loss, (Q, D), retain_graph=True)
        gq2, gd2 = torch.autograd.grad(-3.0 * loss, (Q, D))
        assert torch.equal(gq1, (5.0 * r["dq"]).bfloat16())
        assert torch.equal(gd1, (5.0 * r["dd"]).bfloat16())
        assert torch.equal(gq2, (-3.0 * r["dq"]).bfloat16())
        assert torch.equal(gd2, (-3.0 * r["dd"]).bfloat16())


def test_autograd_saved_gradients_through_hooks():
    # saved-tensor hooks that keep the gradients in 16 bits, or transposed, or on the host
    w = synth.coltrast_step(seed=3, nq=4, n_neg=3, ld=32)
    Q = w["Q"].to(DEV).requires_grad_(True)
    D = w["D"].to(DEV).requires_grad_(True)
    off, pos = _to_dev(w["off"], w["pos"])
    r = hpr.coltrast_loss_fwd_bwd(Q.detach(), D.detach(), off, pos, 1.5625)
    hooks = [(lambda t: t.to(torch.bfloat16), lambda t: t),
             (lambda t: t.transpose(0, 1).contiguous(), lambda t: t.transpose(0, 1)),
             (lambda t: t.cpu(), lambda t: t.to(DEV))]
    for pack, unpack in hooks:
        with torch.autograd.graph.saved_tensors_hooks(pack, unpack):
            loss = hpr.coltrast_loss(Q, D, off, pos, 1.5625)
        got = torch.autograd.grad(3.0 * loss, (Q, D))
        for g, ref in zip(got, (r["dq"], r["dd"])):
            kept = unpack(pack(ref)).float()
            assert torch.equal(g, (3.0 * kept).bfloat16())


# ------------------------------------------------------------------------------ plumbing

def test_calls_on_a_non_default_stream():
    w = synth.tiny_maxsim(seed=4)
    Q, D, off = _to_dev(w["Q"], w["D"], w["off"])
    ref = hpr.maxsim_score(Q, D, off)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        out = hpr.maxsim_score(Q, D, off)
    s.synchronize()
    assert torch.equal(ref, out)


def test_calibrate_on_the_current_device():
    low, rand, read = hpr.calibrate(device="cuda", mfma_iters=200, read_bytes=1 << 26, reps=1)
    assert low > 0 and rand > 0 and read > 0


def test_concurrent_calls_on_two_streams_with_separate_workspaces():
    # two streams, each with its own workspace, run different calls at the same time; the
    # results equal those of the same calls made one after the other on the default stream
    w1 = synth.tiny_maxsim(seed=7, n_docs=3000, ld=48)
    c = synth.coltrast_step(seed=8, nq=16, n_neg=7, ld=64)
    Q1, D1, off1 = _to_dev(w1["Q"], w1["D"], w1["off"])
    Q2, D2, off2, pos2 = _to_dev(c["Q"], c["D"], c["off"], c["pos"])
    ref_s, ref_i = hpr.maxsim_topk(Q1, D1, off1, 50)
    ref_l = hpr.coltrast_loss_fwd_bwd(Q2, D2, off2, pos2, 1.5625)
    ref_sc = hpr.maxsim_score(Q2, D2, off2)
    torch.cuda.synchronize()
    sa, sb = torch.cuda.Stream(), torch.cuda.Stream()
    ws_a = torch.empty(hpr.lib().maxsim_topk_workspace_size(8, 32, 3000, D1.shape[0], 128, 50),
                       dtype=torch.uint8, device=DEV)
    ws_b = hpr.coltrast_workspace(Q2, D2, off2)
    outs = []
    for rep in range(3):
        with torch.cuda.stream(sa):
            ta = hpr.maxsim_topk(Q1, D1, off1, 50, ws=ws_a)
            sc = hpr.maxsim_score(Q2, D2, off2)
        with torch.cuda.stream(sb):
            lb = hpr.coltrast_loss_fwd_bwd(Q2, D2, off2, pos2, 1.5625, ws=ws_b)
        outs.append((ta, sc, lb))
    torch.cuda.synchronize()
    for ta, sc, lb in outs:
        assert torch.equal(ta[0], ref_s) and torch.equal(ta[1], ref_i)
        assert torch.equal(sc, ref_sc)
        for key in ("loss", "dq", "dd"):
            assert torch.equal(lb[key], ref_l[key]), key


def test_validate_env_rejects_a_bad_csr_before_the_call(monkeypatch):
    Q, D, off = _ragged(5, 2, 4, [3, 5, 2], 16)
    bad = off.clone()
    bad[2] = bad[1]  # an empty document
    monkeypatch.setenv("HPR_VALIDATE", "1")
    with pytest.raises(hpr.HprError) as e:
        hpr.maxsim_score(*_to_dev(Q, D, bad))
    assert e.value.status_name == "HPR_ERR_EMPTY_DOC"
    S = hpr.maxsim_score(*_to_dev(Q, D, off)).cpu().numpy()  # a valid CSR passes
    _assert_close(S, oracle.maxsim_scores(_bf(Q), _bf(D), off.numpy()), what="scores")


def test_csr_validate():
    good = torch.tensor([0, 3, 4, 9], dtype=torch.int64, device=DEV)
    assert hpr.csr_validate(good, 9) == ("HPR_OK", -1)
    empty = torch.tensor([0, 3, 3, 9], dtype=torch.int64, device=DEV)
    assert hpr.csr_validate(empty, 9) == ("HPR_ERR_EMPTY_DOC", 1)
    dec = torch.tensor([0, 5, 4, 9], dtype=torch.int64, device=DEV)
    assert hpr.csr_validate(dec, 9) == ("HPR_ERR_BAD_CSR", 1)
    end = torch.tensor([0, 5, 8], dtype=torch.int64, device=DEV)
    assert hpr.csr_validate(end, 9) == ("HPR_ERR_BAD_CSR", 1)
    start = torch.tensor([1, 5, 9], dtype=torch.int64, device=DEV)
    assert hpr.csr_validate(start, 9) == ("HPR_ERR_BAD_CSR", 0)


def test_loss_call_replays_correctly_in_a_hip_graph():
    # every library launch of the call is captured; replays with eager work and synchronisation
    # in between must reproduce the eager result bit for bit each time
    w = synth.coltrast_step(seed=5, nq=16, n_neg=7, ld=64)
    Q, D, off, pos = _to_dev(w["Q"], w["D"], w["off"], w["pos"])
    ws = hpr.coltrast_workspace(Q, D, off)
    out = {"loss": torch.empty(1, device=DEV), "dq": torch.empty(Q.shape, device=DEV),
           "dd": torch.empty(D.shape, device=DEV)}
    eager = hpr.coltrast_loss_fwd_bwd(Q, D, off, pos, 1.5625)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        hpr.coltrast_loss_fwd_bwd(Q, D, off, pos, 1.5625, ws=ws, out=out)
    torch.cuda.current_stream().wait_stream(side)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        hpr.coltrast_loss_fwd_bwd(Q, D, off, pos, 1.5625, ws=ws, out=out)
    for rep in range(4):
        for key in ("loss", "dq", "dd"):
            out[key].fill_(float("nan"))
        g.replay()
        hpr.maxsim_score(Q, D, off)             # unrelated eager work between replays
        torch.cuda.synchronize()
        for key in ("loss", "dq", "dd"):
            assert torch.equal(out[key], eager[key]), f"replay {rep}: {key} differs"


def test_topk_call_replays_correctly_in_a_hip_graph():
    w = synth.tiny_maxsim(seed=6)
    Q, D, off = _to_dev(w["Q"], w["D"], w["off"])
    ref_s, ref_i = hpr.maxsim_topk(Q, D, off, 10)
    ws = torch.empty(hpr.lib().maxsim_topk_workspace_size(8, 32, 256, D.shape[0], 128, 10),
                     dtype=torch.uint8, device=DEV)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        hpr.maxsim_topk(Q, D, off, 10, ws=ws)
    torch.cuda.current_stream().wait_stream(side)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        s, i = hpr.maxsim_topk(Q, D, off, 10, ws=ws)
    for rep in range(3):
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(s, ref_s) and torch.equal(i, ref_i), f"replay {rep}"
