"""The work that programs have this library do, as cases that can be timed and compared.

A case is a dict of plain values; its "kind" says which public entry points one pass calls:

  score   maxsim_score: late-interaction scores of a few queries over candidate documents
  search  maxsim_topk: exact late-interaction search of a document store
  loss    coltrast_loss_fwd_bwd: L_LI with both gradients into buffers the program keeps
  train   coltrast_loss or coltrast_total_loss and its backward through autograd
  dense   dense_ip_topk over a pooled single-vector store
  eval    dense_ip_topk, then retrieval_metrics on its lists (the retrieval evaluation)
  chunk   semantic_chunk over sentence embeddings

Tokens are unit rows rounded to bf16 (fp16 for pooled rows and sentences).  Queries are noisy
copies of some document's tokens, as relevant documents are in a real store.
"""

import math

import torch

import paper_2505_04846_amd as hpr

DEV = "cuda:0"
CHUNK_ROWS = 1 << 21


def listed():
    return [
        # Reranking: one query's 1,000 first-stage candidates, a call per user query (latency).
        {"name": "rerank", "kind": "score", "nq": 1, "lq": 32, "n_docs": 1000, "dim": 128,
         "lengths": "uniform", "ld_min": 32, "ld_max": 384},
        # Interactive search: one query against a whole store (bound by reading the store).
        {"name": "search_one", "kind": "search", "nq": 1, "lq": 32, "n_docs": 100_000,
         "dim": 128, "lengths": "uniform", "ld_min": 32, "ld_max": 384, "k": 100},
        # A batch of queries against a ragged store (li_retrieval with a tenth of its documents).
        {"name": "search_batch", "kind": "search", "nq": 1024, "lq": 32, "n_docs": 50_000,
         "dim": 128, "lengths": "uniform", "ld_min": 32, "ld_max": 384, "k": 100},
        # The largest batches and lists (li_large with a twentieth of its documents).
        {"name": "search_large", "kind": "search", "nq": 4096, "lq": 64, "n_docs": 50_000,
         "dim": 128, "lengths": "lognormal", "ld_min": 16, "ld_max": 512, "k": 1000},
        # A fine-tuning micro-batch: 24 queries, a positive and a negative each, ragged chunks.
        {"name": "train_micro", "kind": "train", "total": False, "nq": 24, "lq": 32,
         "n_neg": 1, "dim": 128, "lengths": "uniform", "ld_min": 40, "ld_max": 300},
        # The L_LI training step of the benchmark, outputs and workspace kept by the program.
        {"name": "loss_step", "kind": "loss", "nq": 64, "lq": 32, "n_neg": 7, "dim": 128,
         "lengths": "fixed", "ld_min": 256, "ld_max": 256},
        # The same batch under the whole ColTrast loss, through autograd, ragged documents.
        {"name": "train_total", "kind": "train", "total": True, "nq": 64, "lq": 32, "n_neg": 7,
         "dim": 128, "lengths": "uniform", "ld_min": 64, "ld_max": 448},
        # Pooled search of a small collection (one corpus section) at a BERT-sized embedding.
        {"name": "dense_small", "kind": "dense", "nq": 16, "n": 20_011, "dim": 768, "k": 10},
        # Pooled search, one query against a million SFR-sized rows (bound by reading them).
        {"name": "dense_one", "kind": "dense", "nq": 1, "n": 1_000_000, "dim": 4096, "k": 100},
        # Retrieval evaluation: every question against the store, then P@k and MRR@k.
        {"name": "dense_eval", "kind": "eval", "nq": 4096, "n": 1_000_000, "dim": 4096, "k": 100},
        # Chunking papers one by one, as they come out of the parser.
        {"name": "chunk_paper", "kind": "chunk", "papers": 1, "len_min": 200, "len_max": 200,
         "dim": 4096},
        # Chunking a corpus (semantic_chunk of the benchmark with a fifth of its papers).
        {"name": "chunk_corpus", "kind": "chunk", "papers": 2000, "len_min": 50, "len_max": 350,
         "dim": 4096},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _doc_lengths(rng):
    kind = rng.choice(["uniform", "uniform", "lognormal", "fixed"])
    if kind == "lognormal":
        return {"lengths": kind, "ld_min": 16, "ld_max": 512}
    if kind == "fixed":
        ld = _log_int(rng, 48, 384)
        return {"lengths": kind, "ld_min": ld, "ld_max": ld}
    return {"lengths": kind, "ld_min": _log_int(rng, 16, 64), "ld_max": _log_int(rng, 128, 512)}


def draw(rng):
    kind = rng.choice(["score", "search", "search", "loss", "train", "train", "dense", "dense",
                       "eval", "chunk"])
    if kind in ("score", "search"):
        dim = rng.choice([128, 128, 128, 96, 64, 256])
        c = {"kind": kind, "nq": _log_int(rng, 1, 16 if kind == "score" else 4096),
             "lq": rng.choice([32, 32, rng.randint(8, 64)]), "n_docs": 0, "dim": dim}
        c.update(_doc_lengths(rng))
        if kind == "score":
            c["n_docs"] = _log_int(rng, 50, 5000)
            return c
        per_doc = 2.0 * dim * c["nq"] * c["lq"] * 0.5 * (c["ld_min"] + c["ld_max"])
        most = max(1000, min(100_000, int(1.5e14 / per_doc)))  # at most a fifth of search_large
        c["n_docs"] = _log_int(rng, 1000, most) if most > 1000 else most
        c["k"] = _log_int(rng, 1, 1000)
        return c
    if kind in ("loss", "train"):
        c = {"kind": kind, "nq": _log_int(rng, 4, 128), "lq": rng.choice([32, rng.randint(8, 48)]),
             "n_neg": rng.randint(0, 7), "dim": rng.choice([128, 128, 96, 64])}
        if kind == "train":
            c["total"] = rng.random() < 0.5
        c.update(_doc_lengths(rng))
        if c["lengths"] == "fixed" or c["ld_min"] < c["lq"]:  # documents hold the query's tokens
            c["ld_min"] = max(c["ld_min"], c["lq"])
            c["ld_max"] = max(c["ld_max"], c["ld_min"])
        return c
    if kind in ("dense", "eval"):
        dim = rng.choice([384, 768, 1024, 4096])
        n = _log_int(rng, 2000, 1_000_000 if dim <= 1024 else 400_000)
        return {"kind": kind, "nq": min(_log_int(rng, 1, 4096), n // 2), "n": n, "dim": dim,
                "k": _log_int(rng, 1, 1000)}
    return {"kind": "chunk", "papers": _log_int(rng, 1, 2000), "len_min": rng.randint(20, 100),
            "len_max": rng.randint(150, 400), "dim": rng.choice([384, 768, 1024, 4096])}


# ---- inputs --------------------------------------------------------------------------------


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _normalise(x):
    return x / torch.linalg.vector_norm(x, dim=-1, keepdim=True).clamp_min(1e-30)


def _unit_rows(n, dim, gen, dtype):
    out = torch.empty((n, dim), dtype=dtype, device=DEV)
    for r0 in range(0, n, CHUNK_ROWS):
        r1 = min(n, r0 + CHUNK_ROWS)
        raw = torch.randn((r1 - r0, dim), generator=gen, device=DEV)
        out[r0:r1] = _normalise(raw).to(dtype)
    return out


def _spread(n, gen):
    """n values spread evenly over (0, 1), in random order: sizes whose total is the case's own."""
    u = (torch.arange(n, device=DEV, dtype=torch.float64) + 0.5) / n
    return u[torch.randperm(n, generator=gen, device=DEV)]


def _lengths(case, n, gen):
    lo, hi = case["ld_min"], case["ld_max"]
    u = _spread(n, gen)
    if case["lengths"] == "lognormal":
        z = torch.special.ndtri(u)
        return torch.round(torch.exp(math.log(200.0) + 0.5 * z)).to(torch.int64).clamp_(lo, hi)
    return (lo + torch.floor(u * (hi - lo + 1)).to(torch.int64)).clamp_(lo, hi)


def _offsets(lengths):
    off = torch.zeros(lengths.numel() + 1, dtype=torch.int64, device=DEV)
    off[1:] = torch.cumsum(lengths, 0)
    return off


def _store(case, seed):
    """A token store and queries, each query token a noisy copy of a token of one document."""
    g = _gen(seed)
    lengths = _lengths(case, case["n_docs"], g)
    off = _offsets(lengths)
    D = _unit_rows(int(off[-1].item()), case["dim"], g, torch.bfloat16)
    nq, lq, dim = case["nq"], case["lq"], case["dim"]
    doc = torch.randint(0, case["n_docs"], (nq, 1), generator=g, device=DEV)
    u = torch.rand((nq, lq), generator=g, device=DEV, dtype=torch.float64)
    rows = off[doc] + torch.floor(u * lengths[doc]).to(torch.int64)
    noise = torch.randn((nq, lq, dim), generator=g, device=DEV) / math.sqrt(dim)
    Q = _normalise(D[rows].float() + 0.75 * noise).to(torch.bfloat16)
    return {"Q": Q, "D": D, "off": off}


def _batch(case, seed):
    """An in-batch training set: doc (n_neg + 1) q + h holds, in lq random slots, noisy copies of
    query q's tokens, the positive (h = 0) closer ones than the hard negatives."""
    g = _gen(seed)
    nq, lq, dim, per_q = case["nq"], case["lq"], case["dim"], case["n_neg"] + 1
    n_docs = nq * per_q
    lengths = _lengths(case, n_docs, g).clamp_min(lq)
    off = _offsets(lengths)
    n_tok = int(off[-1].item())
    q_raw = torch.randn((nq, lq, dim), generator=g, device=DEV)
    D = _unit_rows(n_tok, dim, g, torch.bfloat16)
    most = int(lengths.max().item())
    key = torch.rand((n_docs, most), generator=g, device=DEV)
    key.masked_fill_(torch.arange(most, device=DEV)[None] >= lengths[:, None], 2.0)
    slots = torch.argsort(key, dim=1)[:, :lq] + off[:-1, None]
    h = torch.arange(n_docs, device=DEV) % per_q
    sigma = (0.3 + 0.05 * h.float())[:, None, None]
    eps = torch.randn((n_docs, lq, dim), generator=g, device=DEV)
    near = _normalise(q_raw.repeat_interleave(per_q, 0) + sigma * eps).to(torch.bfloat16)
    D[slots.reshape(-1)] = near.reshape(-1, dim)
    return {"Q": _normalise(q_raw).to(torch.bfloat16), "D": D, "off": off,
            "pos": torch.arange(0, n_docs, per_q, dtype=torch.int32, device=DEV)}


def _pooled(case, seed):
    """A pooled store with one relevant row (cosine 0.95) for every query."""
    g = _gen(seed)
    nq, n, dim = case["nq"], case["n"], case["dim"]
    Q = _unit_rows(nq, dim, g, torch.float16)
    X = _unit_rows(n, dim, g, torch.float16)
    rows = torch.randperm(n, generator=g, device=DEV)[:nq]
    q = _normalise(Q.float())
    u = torch.randn((nq, dim), generator=g, device=DEV)
    u = _normalise(u - (u * q).sum(-1, keepdim=True) * q)
    X[rows] = (0.95 * q + math.sqrt(1.0 - 0.95 ** 2) * u).to(torch.float16)
    return {"Q": Q, "X": X, "positive": rows, "k": min(case["k"], n)}


def _sentences(case, seed):
    """Consecutive papers' sentences; a paper's topic changes about every eight sentences."""
    g = _gen(seed)
    u = _spread(case["papers"], g)
    lo, hi = case["len_min"], case["len_max"]
    off = _offsets((lo + torch.floor(u * (hi - lo + 1)).to(torch.int64)).clamp_(lo, hi))
    n, dim = int(off[-1].item()), case["dim"]
    switch = torch.rand(n, generator=g, device=DEV) < 0.125
    switch[off[:-1]] = True
    topic = torch.cumsum(switch.to(torch.int64), 0) - 1
    topics = _unit_rows(int(topic[-1].item()) + 1, dim, g, torch.float32)
    E = torch.empty((n, dim), dtype=torch.float16, device=DEV)
    for r0 in range(0, n, 1 << 17):
        r1 = min(n, r0 + (1 << 17))
        noise = torch.randn((r1 - r0, dim), generator=g, device=DEV)
        E[r0:r1] = _normalise(topics[topic[r0:r1]] + (0.5 / math.sqrt(dim)) * noise).half()
    return {"E": E, "off": off if case["papers"] > 1 else None}


SCALE, TAU = 1.5625, 0.05  # 1 / (32 x 0.02), and the temperature of the pooled half
THRESHOLD = 0.5


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("score", "search"):
        s = _store(case, seed)
        if kind == "search":
            s["k"] = min(case["k"], case["n_docs"])
    elif kind in ("loss", "train"):
        s = _batch(case, seed)
        if kind == "loss":
            Q, D = s["Q"], s["D"]
            s["ws"] = hpr.coltrast_workspace(Q, D, s["off"])
            s["out"] = {"loss": torch.empty(1, device=DEV),
                        "dq": torch.empty(Q.shape, device=DEV),
                        "dd": torch.empty(D.shape, device=DEV)}
        else:
            s["total"] = case["total"]
            s["Q"].requires_grad_(True)
            s["D"].requires_grad_(True)
    elif kind in ("dense", "eval"):
        s = _pooled(case, seed)
    else:
        s = _sentences(case, seed)
    s["kind"] = kind
    return s


def run(s):
    kind = s["kind"]
    if kind == "score":
        return hpr.maxsim_score(s["Q"], s["D"], s["off"])
    if kind == "search":
        return hpr.maxsim_topk(s["Q"], s["D"], s["off"], s["k"])
    if kind == "loss":
        r = hpr.coltrast_loss_fwd_bwd(s["Q"], s["D"], s["off"], s["pos"], SCALE, ws=s["ws"],
                                      out=s["out"])
        return {"loss": r["loss"], "dq": r["dq"], "dd": r["dd"]}
    if kind == "train":
        if s["total"]:
            loss = hpr.coltrast_total_loss(s["Q"], s["D"], s["off"], s["pos"], SCALE, TAU)
        else:
            loss = hpr.coltrast_loss(s["Q"], s["D"], s["off"], s["pos"], SCALE)
        dq, dd = torch.autograd.grad(loss, (s["Q"], s["D"]))
        return {"loss": loss.detach(), "dq": dq, "dd": dd}
    if kind == "dense":
        return hpr.dense_ip_topk(s["Q"], s["X"], s["k"])
    if kind == "eval":
        scores, idx = hpr.dense_ip_topk(s["Q"], s["X"], s["k"])
        m = hpr.retrieval_metrics(idx, s["positive"])
        return {"scores": scores, "idx": idx, "metrics": m["metrics"], "ranks": m["ranks"]}
    r = hpr.semantic_chunk(s["E"], s["off"], THRESHOLD, return_cos=True)
    return {"seg": r["seg"], "n_segments": r["n_segments"], "cos": r["cos"]}


# ---- what a pass cannot do without ----------------------------------------------------------


def _mean_len(case):
    if case["lengths"] == "lognormal":
        return 223.0  # exp(N(ln 200, 0.5)) clipped to [16, 512]
    return max(0.5 * (case["ld_min"] + case["ld_max"]), 1.0)


def work(case):
    kind = case["kind"]
    if kind in ("score", "search", "loss", "train"):
        nq, lq, dim = case["nq"], case["lq"], case["dim"]
        n_docs = case.get("n_docs") or nq * (case["n_neg"] + 1)
        n_tok = n_docs * _mean_len(case)
        nbytes = 2.0 * dim * (nq * lq + n_tok) + 8.0 * n_docs
        flops = 2.0 * dim * nq * lq * n_tok
        if kind == "score":
            nbytes += 4.0 * nq * n_docs
        elif kind == "search":
            nbytes += 12.0 * nq * min(case["k"], n_docs)
        else:  # gradients out (fp32 buffers, or bf16 like the inputs) and their gather terms
            nbytes += (4.0 if kind == "loss" else 2.0) * dim * (nq * lq + n_tok)
            flops += 4.0 * dim * nq * lq * n_docs
            if case.get("total"):
                flops += 6.0 * dim * nq * n_docs
        return {"bytes": nbytes, "flops": flops}
    if kind in ("dense", "eval"):
        nq, n, dim, k = case["nq"], case["n"], case["dim"], min(case["k"], case["n"])
        return {"bytes": 2.0 * dim * (nq + n) + 12.0 * nq * k, "flops": 2.0 * dim * nq * n}
    n = case["papers"] * 0.5 * (case["len_min"] + case["len_max"])
    return {"bytes": 2.0 * case["dim"] * n + 8.0 * n, "flops": 4.0 * case["dim"] * n}


def tolerance(case):
    kind = case["kind"]
    if kind == "score":
        return {"rel": 4e-7, "max": 1e-5}
    if kind == "search":  # indices: near-equal scores may change places
        return {"rel": 4e-7, "max": 1e-5, "differ": 0.01}
    if kind in ("dense", "eval"):
        return {"rel": 1.5e-6, "max": 1e-5, "differ": 0.01}
    if kind == "loss":  # a near-tie of two tokens moves a gradient term to another row
        return {"rel": 1e-4, "max": 0.5}
    if kind == "train":  # ... and the gradients come back rounded to bf16
        return {"rel": 2e-3, "max": 0.5}
    return {"rel": 4e-7, "max": 1e-5, "differ": 1e-4}


# ---- the same in 64 bits --------------------------------------------------------------------


def _blocks(off, nq_slots):
    """Runs of documents whose padded tables hold at most 2^28 values, or 2^17 tokens."""
    lens = (off[1:] - off[:-1]).tolist()
    d0, most = 0, 0
    for d, n in enumerate(lens):
        grown = max(most, n)
        if d > d0 and (d + 1 - d0) * grown * max(nq_slots, 2048) > (1 << 28):
            yield d0, d, most
            d0, grown = d, n
        most = grown
    yield d0, len(lens), most


def _maxsim64(Q, D, off):
    """Per (query token, document): the largest product and its first token, in 64 bits."""
    nq, lq, dim = Q.shape
    q = Q.detach().reshape(nq * lq, dim).double()
    best = torch.empty((nq * lq, off.numel() - 1), dtype=torch.float64, device=DEV)
    arg = torch.empty(best.shape, dtype=torch.int64, device=DEV)
    for d0, d1, most in _blocks(off, nq * lq):
        j = torch.arange(most, device=DEV)[None]
        lens = (off[d0 + 1:d1 + 1] - off[d0:d1])[:, None]
        rows = off[d0:d1, None] + torch.minimum(j, lens - 1)
        d = D.detach()[rows.reshape(-1)].double()
        sims = (q @ d.t().contiguous()).reshape(nq * lq, d1 - d0, most)
        v, a = sims.max(dim=-1)
        best[:, d0:d1] = v
        arg[:, d0:d1] = torch.gather(rows, 1, a.t()).t()
    return best, arg


def _pool64(x, off):
    lens = (off[1:] - off[:-1]).double()
    doc = torch.repeat_interleave(torch.arange(lens.numel(), device=DEV), off[1:] - off[:-1])
    p = torch.zeros((lens.numel(), x.shape[1]), dtype=torch.float64, device=DEV)
    return p.index_add_(0, doc, x) / lens[:, None]


def _loss64(s, total):
    Q, D, off, pos = s["Q"].detach(), s["D"].detach(), s["off"], s["pos"].long()
    nq, lq, dim = Q.shape
    best, arg = _maxsim64(Q, D, off)
    S = best.reshape(nq, lq, -1).sum(1)
    logp = torch.log_softmax(SCALE * S, dim=1)
    loss = -logp.gather(1, pos[:, None]).mean()
    P = logp.exp()
    P.scatter_(1, pos[:, None], 0.0)
    P.scatter_(1, pos[:, None], -P.sum(1, keepdim=True))
    G = (P * (SCALE / nq)).repeat_interleave(lq, 0)
    q, d = Q.reshape(nq * lq, dim).double(), D.double()
    dq, dd = torch.zeros_like(q), torch.zeros_like(d)
    for c in range(off.numel() - 1):
        dq += G[:, c:c + 1] * d[arg[:, c]]
        dd.index_add_(0, arg[:, c], G[:, c:c + 1] * q)
    if total:
        with torch.enable_grad():
            qg, dg = q.clone().requires_grad_(True), d.clone().requires_grad_(True)
            uq = _normalise(qg.reshape(nq, lq, dim).mean(1))
            ud = _normalise(_pool64(dg, off))
            cos = torch.log_softmax((uq @ ud.t().contiguous()) / TAU, dim=1)
            lc = -cos.gather(1, pos[:, None]).mean()
            gq, gd = torch.autograd.grad(lc, (qg, dg))
        loss, dq, dd = 0.5 * (loss + lc.detach()), 0.5 * (dq + gq), 0.5 * (dd + gd)
    return loss, dq.reshape(nq, lq, dim), dd


def exact(case, seed):
    if work(case)["flops"] > 2.5e14:
        return None
    s = prepare(case, seed)
    kind = case["kind"]
    if kind in ("score", "search"):
        best, _ = _maxsim64(s["Q"], s["D"], s["off"])
        S = best.reshape(case["nq"], case["lq"], -1).sum(1)
        return S if kind == "score" else (torch.topk(S, s["k"], dim=1).values, None)
    if kind in ("loss", "train"):
        loss, dq, dd = _loss64(s, bool(case.get("total")))
        return {"loss": loss.reshape(1) if kind == "loss" else loss, "dq": dq, "dd": dd}
    if kind in ("dense", "eval"):
        q, top = s["Q"].double(), None
        for r0 in range(0, case["n"], 1 << 16):
            v = q @ s["X"][r0:r0 + (1 << 16)].double().t().contiguous()
            top = v if top is None else torch.cat([top, v], 1)
            top = torch.topk(top, min(s["k"], top.shape[1]), dim=1).values
        if kind == "dense":
            return top, None
        return {"scores": top, "idx": None, "metrics": None, "ranks": None}
    E, off = s["E"], s["off"]
    n = E.shape[0]
    cos = torch.full((n,), float("nan"), dtype=torch.float64, device=DEV)
    for r0 in range(1, n, 1 << 16):
        r1 = min(n, r0 + (1 << 16))
        a, b = E[r0 - 1:r1 - 1].double(), E[r0:r1].double()
        cos[r0:r1] = (a * b).sum(1) / (a.norm(dim=1) * b.norm(dim=1))
    if off is not None:
        cos[off[:-1][off[:-1] < n]] = float("nan")
    return {"seg": None, "n_segments": None, "cos": cos}
