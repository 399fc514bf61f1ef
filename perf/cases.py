"""The workloads this library is measured on: what a reranking service has it do, through the Python entry points.

Every case is a plain dict.  `kind` says which calls one pass makes:

  score     Model.score on resident documents (f32 models: and the per-query top-k of the scores)
  plan      Plan.run, the fixed-shape form of the same call that serving loops keep
  cold      the candidates' pages arrive from pinned host memory in 4-bit records, then Model.score
  prefill   Model.doc_prefill: documents run through the model once, their K/V stored in pool pages
  ingest    KVPool.write of documents whose K/V were computed elsewhere, and KVPool.read of them all

Models are the shapes of workloads.MODELS with random weights (one fixed draw per shape, as a service keeps one model);
documents, queries, candidate lists and page placement come from the seed.  Lengths are drawn per document and per
query between the bounds of the case (prefill, ingest: the same ones for every seed)."""

import functools
import math

import numpy as np
import torch

from paper_2504_02921_amd import binding as hb
from paper_2504_02921_amd import workloads as wlmod

DEV = "cuda:0"
POOL_BYTES_MOST = 56e9            # three states of a case and the models fit the card


def _case(kind, model, kv, queries, cands, docs, query, pool_docs=0, **more):
    """docs, query: (shortest, longest).  pool_docs: candidates are drawn from this many documents by popularity, 0: every
    pair has a document of its own.  prefill / ingest: `cands` documents, no queries."""
    return dict(kind=kind, model=model, kv=kv, queries=queries, cands=cands, doc_lo=docs[0], doc_hi=docs[1],
                query_lo=query[0], query_hi=query[1], pool_docs=pool_docs, **more)


def listed():
    return [
        # a small fp32 model (exact scores for regression checks), one query, best candidates picked
        _case("score", "tiny", "f32", 1, 8, (128, 128), (16, 16), name="tiny_f32"),
        # the shortest request a service sees: one query, the retriever's five candidates, ragged passages
        _case("score", "qwen2_0p5b", "bf16", 1, 5, (100, 300), (13, 13), name="request5_0p5b"),
        # the ordinary request of a latency-bound serving loop: one query, 20 candidates, fixed shape
        _case("plan", "qwen2_0p5b", "bf16", 1, 20, (512, 512), (32, 32), name="request20_0p5b"),
        # the same with the large model
        _case("score", "llama3_8b", "bf16", 1, 20, (256, 256), (32, 32), name="request20_8b"),
        # throughput: many queries batched, 0.5B shape
        _case("score", "qwen2_0p5b", "bf16", 32, 20, (512, 512), (32, 32), name="batch_0p5b"),
        # throughput, ragged lengths, popular documents shared between queries
        _case("score", "qwen2_0p5b", "bf16", 64, 100, (64, 1024), (8, 64), 4096, name="ragged_0p5b"),
        # throughput, 8B shape
        _case("score", "llama3_8b", "bf16", 8, 50, (256, 256), (32, 32), name="batch_8b"),
        # long documents in an 8-bit pool, 8B shape: the largest
        _case("score", "llama3_8b", "fp8", 4, 100, (2048, 2048), (64, 64), name="long_fp8_8b"),
        # candidates that are not resident: 4-bit pages over the bus, then the request
        _case("cold", "qwen2_0p5b", "bf16", 1, 20, (512, 512), (32, 32), name="cold20_0p5b"),
        # indexing a corpus on the device
        _case("prefill", "qwen2_0p5b", "bf16", 0, 128, (512, 512), (0, 0), name="prefill_0p5b"),
        _case("prefill", "llama3_8b", "bf16", 0, 32, (100, 700), (0, 0), name="prefill_8b"),
        # documents whose K/V come from another producer, and their way back to a storage tier
        _case("ingest", "qwen2_0p5b", "bf16", 0, 16, (64, 1024), (0, 0), name="ingest_0p5b"),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _span(rng, lo, hi, fixed):
    """Bounds of a length: one value, or a range up to it."""
    top = _log_int(rng, lo, hi)
    return (top, top) if rng.random() < fixed else (_log_int(rng, max(1, lo // 2), top), top)


def draw(rng):
    most = max(_cost(c) for c in listed())
    while True:
        what = rng.choice(("score", "score", "score", "score", "plan", "cold", "prefill", "ingest", "f32"))
        big = rng.random() < 0.4
        model = "llama3_8b" if big else "qwen2_0p5b"
        kv = "fp8" if rng.random() < 0.3 else "bf16"
        if what == "f32":
            c = _case("score", "tiny", "f32", rng.randint(1, 4), _log_int(rng, 5, 50), _span(rng, 16, 512, 0.5), _span(rng, 4, 64, 0.5))
        elif what == "score":
            queries, cands = _log_int(rng, 1, 8 if big else 64), _log_int(rng, 5, 100)
            pool = queries * cands * rng.randint(1, 3) if queries > 1 and rng.random() < 0.4 else 0
            c = _case("score", model, kv, queries, cands, _span(rng, 64, 2048, 0.4), _span(rng, 8, 64, 0.5), max(pool, cands) if pool else 0)
        elif what == "plan":
            c = _case("plan", model, kv, rng.randint(1, 4), _log_int(rng, 5, 20), _span(rng, 64, 1024, 0.6), _span(rng, 8, 64, 0.6))
        elif what == "cold":
            c = _case("cold", "qwen2_0p5b", "bf16", rng.randint(1, 2), _log_int(rng, 5, 40), _span(rng, 64, 1024, 0.4), _span(rng, 8, 64, 0.6))
        elif what == "prefill":
            c = _case("prefill", model, "bf16", 0, _log_int(rng, 1, 32 if big else 128), _span(rng, 64, 1024, 0.4), (0, 0))
        else:
            c = _case("ingest", model, kv, 0, _log_int(rng, 1, 16), _span(rng, 64, 1024, 0.3), (0, 0))
        if _cost(c) <= most and _pool_bytes(c) <= POOL_BYTES_MOST:
            return c


# ---- sizes --------------------------------------------------------------------------------------------------------
def _mean(lo, hi):
    return 0.5 * (lo + hi)


def _docs(c):
    """(documents in the pool, distinct documents one pass reads, expected)."""
    pairs = c["queries"] * c["cands"]
    if c["kind"] in ("prefill", "ingest"):
        return c["cands"], c["cands"]
    if not c["pool_docs"]:
        return pairs, pairs
    p = np.arange(1, c["pool_docs"] + 1, dtype=np.float64) ** -1.1
    hit = 1.0 - np.exp(-c["cands"] * p / p.sum())                 # per query, candidates without replacement: about this
    scale = min(1.0, c["cands"] / hit.sum())
    return c["pool_docs"], float((1.0 - (1.0 - hit * scale) ** c["queries"]).sum())


def _doc_token_bytes(c):
    m = wlmod.MODELS[c["model"]]
    return m.kv_bytes_per_token(c["kv"])


def _pool_bytes(c):
    return _docs(c)[0] * (_mean(c["doc_lo"], c["doc_hi"]) + 16) * _doc_token_bytes(c)


def work(case):
    """What one pass cannot do without: layer weights once, each distinct document's K/V once, the projections of the
    tokens whose results are used (only a pair's last token is needed behind the last layer's K/V), scores of every
    visible key."""
    c = case
    m = wlmod.MODELS[c["model"]]
    L, H, d, F = m.n_layers, m.hidden, m.head_dim, m.ffn
    nq, nqkv = m.n_q_heads * d, m.qkv_out
    esz = 4 if m.dtype == "f32" else 2
    doc = _mean(c["doc_lo"], c["doc_hi"])
    weights = L * (H * nqkv + nq * H + 3 * H * F) * esz
    kv_tok = _doc_token_bytes(c)
    n_docs = _docs(c)[1]
    rest = nq * H + 3 * H * F
    if c["kind"] == "ingest":                                     # source read, pages written; pages read, copies written
        return {"bytes": 4.0 * n_docs * doc * kv_tok, "flops": 0.0}
    if c["kind"] == "prefill":
        T = n_docs * doc
        pairs2 = n_docs * (doc * doc + (c["doc_hi"] - c["doc_lo"]) ** 2 / 12.0) / 2.0       # causal (token, key) pairs
        flops = 2.0 * T * (L * H * nqkv + (L - 1) * rest) + 4.0 * (L - 1) * pairs2 * nq
        return {"bytes": float(weights + T * kv_tok + T * H * esz), "flops": flops}
    P = c["queries"] * c["cands"]
    q = _mean(c["query_lo"], c["query_hi"])
    T = P * q
    keys = doc + q / 2.0
    flops = 2.0 * T * L * H * nqkv + 2.0 * ((L - 1) * T + P) * rest + 4.0 * ((L - 1) * T + P) * keys * nq
    nbytes = weights + n_docs * doc * kv_tok + T * H * esz
    if c["kind"] == "cold":
        nbytes += n_docs * doc * kv_tok * (1.0 + 1.0 / 3.2)       # records read, pages written
    return {"bytes": float(nbytes), "flops": flops}


def _cost(c):
    w = work(c)
    return w["flops"] / 1e15 + w["bytes"] / 4e12


# ---- models: one fixed draw of weights per shape --------------------------------------------------------------------
class _Weights:
    """Random-init matrices N(0, 0.02^2) and unit gains: windows of one long normal vector, another window for every
    matrix, so that an 8B-shaped model is up in seconds."""

    STRIDE = 100003                # no multiple of a row length: no two matrices share a row

    def __init__(self, m):
        self.m = m
        most = max(int(np.prod(m.shape(k))) for k in ("wq", "wo", "wg", "wd"))
        rng = np.random.Generator(np.random.PCG64(20))
        self.base = rng.standard_normal(most + self.STRIDE * (8 * m.n_layers + 1), dtype=np.float32)
        self.base *= np.float32(0.02)

    def get(self, kind, layer=-1):
        shape = self.m.shape(kind)
        if len(shape) == 1:
            return np.ones(shape, np.float32)
        if kind == "embedding":
            return np.resize(self.base, shape)
        at = self.STRIDE * (7 * layer + ("wq", "wk", "wv", "wo", "wg", "wu", "wd").index(kind))
        return self.base[at:at + int(np.prod(shape))].reshape(shape)


@functools.lru_cache(maxsize=None)
def _model(name):
    m = wlmod.MODELS[name]
    return hb.Model(m, _Weights(m), DEV)


# ---- inputs ---------------------------------------------------------------------------------------------------------
def _doc_kv(m, kv, n_tokens, gen):
    """One document's K/V as a stage-one pass leaves them: bell-shaped around the size RMS-1 rows and N(0, 0.02^2)
    projections give; fp8: codes with a scale per (layer, page, kv head)."""
    shape = (2, m.n_layers, n_tokens, m.n_kv_heads, m.head_dim)
    sigma = wlmod.synthetic_kv_sigma(m)
    if kv == "fp8":
        x = torch.randn(shape, generator=gen, device=DEV, dtype=torch.bfloat16).mul_(96.0).clamp_(-448.0, 448.0)
        codes = x.to(torch.float8_e4m3fn).view(torch.uint8)
        n_pages = (n_tokens + hb.PAGE_TOKENS - 1) // hb.PAGE_TOKENS
        s = torch.rand((2, m.n_layers, n_pages, m.n_kv_heads), generator=gen, device=DEV).sub_(0.5).exp2_().mul_(sigma / 96.0)
        return codes[0], codes[1], s[0], s[1]
    dt = torch.float32 if kv == "f32" else torch.bfloat16
    x = torch.randn(shape, generator=gen, device=DEV, dtype=dt).mul_(sigma)
    return x[0], x[1], None, None


def _pool(m, kv, n_pages):
    return hb.KVPool(m.n_layers, m.n_kv_heads, m.head_dim, n_pages, kv, DEV)


def prepare(case, seed):
    c = case
    m = wlmod.MODELS[c["model"]]
    gen = torch.Generator(DEV)
    gen.manual_seed(seed)
    if c["kind"] in ("prefill", "ingest"):
        # the corpus' lengths belong to the case (the outputs' shapes follow from them), its contents and pages to the seed
        lens = np.random.default_rng(c["cands"]).integers(c["doc_lo"], c["doc_hi"] + 1, c["cands"])
        rng = np.random.default_rng([seed, 1])
        n_pages = (lens + hb.PAGE_TOKENS - 1) // hb.PAGE_TOKENS
        place = rng.permutation(int(n_pages.sum())).astype(np.int32)
        pages = np.split(place, np.cumsum(n_pages)[:-1])
        st = {"kind": c["kind"], "pool": _pool(m, c["kv"], len(place)), "all_pages": place, "pages": pages, "lens": [int(n) for n in lens]}
        if c["kind"] == "prefill":
            st["model"] = _model(c["model"])
            st["tokens"] = [rng.integers(0, m.vocab, n).astype(np.int32) for n in lens]
            data = m.n_layers * len(place) * m.n_kv_heads * 2 * hb.PAGE_TOKENS * m.head_dim * 2
            st["stored"] = st["pool"].mem[:data].view(torch.float16)
        else:
            st["kv"] = [_doc_kv(m, c["kv"], n, gen) for n in st["lens"]]
        return st

    span = lambda lo, hi: lo if lo == hi else (lo, hi)  # noqa: E731
    wl = wlmod.make_workload(wlmod.WorkloadCfg("case", m, c["queries"], c["cands"], span(c["doc_lo"], c["doc_hi"]),
                                               span(c["query_lo"], c["query_hi"]), c["kv"], c["pool_docs"] or None,
                                               1.1 if c["pool_docs"] else None, seed))
    model = _model(c["model"])
    pool = _pool(m, c["kv"], wl.num_pages)
    for doc in np.unique(wl.pair_doc):
        pool.write(int(wl.pool_doc_lens[doc]), wl.pool_doc_pages[doc], *_doc_kv(m, c["kv"], int(wl.pool_doc_lens[doc]), gen))
    st = {"kind": c["kind"], "model": model, "pool": pool,
          "inputs": (wl.page_table, wl.doc_lens, wl.query_tokens, wl.query_lens)}
    if c["kind"] == "plan":
        st["plan"] = hb.Plan(model, pool, wl.doc_lens, wl.query_lens, wl.page_table.shape[1])
        st["plan"].set_inputs(wl.page_table, wl.query_tokens)
        st["scores"] = torch.empty(wl.n_pairs, dtype=torch.float32, device=DEV)
    if c["kind"] == "cold":
        st["all_pages"] = np.concatenate(wl.pool_doc_pages)
        st["records"] = torch.empty(len(st["all_pages"]) * pool.page_record4_bytes, dtype=torch.uint8, pin_memory=True)
        pool.pages_out4(st["all_pages"], st["records"])
        torch.cuda.synchronize()
    if c["kv"] == "f32":
        st["segments"] = np.arange(0, wl.n_pairs + 1, c["cands"])
    return st


def run(state):
    kind, pool = state["kind"], state["pool"]
    if kind == "plan":
        return state["plan"].run(state["scores"])
    if kind == "prefill":
        pool.free(state["all_pages"])
        state["model"].doc_prefill(pool, state["tokens"], state["pages"])
        return state["stored"]
    if kind == "ingest":
        pool.free(state["all_pages"])
        for n, pages, kv in zip(state["lens"], state["pages"], state["kv"]):
            pool.write(n, pages, *kv)
        return [pool.read(n, pages) for n, pages in zip(state["lens"], state["pages"])]
    if kind == "cold":
        pool.free(state["all_pages"])
        pool.pages_in4(state["all_pages"], state["records"])
    scores = state["model"].score(pool, *state["inputs"])
    if "segments" in state:
        return scores, hb.rerank_topk(scores, state["segments"], 5)
    return scores


def tolerance(case):
    if case["kind"] == "ingest":
        return "exact"
    if case["kv"] == "f32":
        return {"rel": 2e-5, "max": 1e-4, "differ": 0.01}
    # 16-bit operands: every activation is rounded to 11 significant bits once per layer, and the layers amplify it
    return {"rel": 1e-2, "max": 8e-2}
