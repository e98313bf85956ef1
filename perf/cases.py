"""The work that users of this library have it do, as measurable cases.

Seven kinds of work, each through the public entry points of `paper_2210_15748_amd`, with the handle, the workspace and the
output buffers that a serving or indexing program keeps from call to call:

  search   queries against every document (`search` without candidates)
  rerank   queries against candidate lists (`search` with candidates), batches down to one query set
  sweep    the synthetic experiment of the paper's Sec. 6.1: 1000 documents of m vectors, queries as long as the documents,
           8 tables of log2(m) + 1 hashes
  build    index building (`build_index`): hashing all document vectors, int8 with +-1 projections or fp16 with Gaussian ones
  phi      `scores` of every document with one of the Sec. 4 aggregations and weighted query vectors
  filter   the whole query of Sec. 5 (`filter_search`): probe the centroid index, count, keep filter_k, score, top-k
  train    making the filter: k-means on a sample of the vectors (`filter_kmeans`), then `filter_build`

Vectors are normalised mixture samples (1024 centres), documents have about 70 vectors (rounded normal, 8 to 180) unless stated,
query vectors are noisy copies of vectors of planted documents.  App. B of the paper walks L over 16 to 128 and C over 4 to 8.
"""
import math

import numpy as np
import torch

import paper_2210_15748_amd as dz

CHUNK = 1 << 21      # vectors made at a time
CENTRES = 1024
SIGMA, SIGMA_Q = 0.3, 0.2


# ---- the cases ----------------------------------------------------------------------------------------------------------
def listed():
    return [
        # the smallest call: ten short query sets over a collection that fits a cache; launches and host time count
        dict(name="search_tiny", kind="search", docs=1000, lens="const32", d=128, L=16, C=6, B=10, q=8, q_ragged=False, k=10),
        # every document of a mid-sized collection for a batch of token-embedding queries
        dict(name="search_mid", kind="search", docs=100_000, lens="uniform", d=128, L=32, C=7, B=64, q=32, q_ragged=False, k=100),
        # the headline: candidate rerank for a batch, the paper's low-latency setting
        dict(name="rerank_batch", kind="rerank", docs=1_000_000, lens="tokens", d=128, L=32, C=7, B=256, q=32, q_ragged=False,
             cand=4096, cand_ragged=False, k=10),
        # rerank for recall: long lists of unequal length, queries of unequal length, 1000 results, 64 tables
        dict(name="rerank_recall", kind="rerank", docs=300_000, lens="tokens", d=128, L=64, C=7, B=32, q=40, q_ragged=True,
             cand=16384, cand_ragged=True, k=1000),
        # one point of the synthetic experiment, 16-bit codes
        dict(name="sweep_m256", kind="sweep", m=256, L=8, C=9, d=128, B=16, k=10),
        # index building, the main configuration
        dict(name="build_i8", kind="build", dtype="i8", docs=200_000, lens="tokens", d=128, L=32, C=7),
        # index building from fp16 embeddings of 256 dimensions, Gaussian projections
        dict(name="build_f16", kind="build", dtype="f16", docs=30_000, lens="tokens", d=256, L=64, C=8),
        # the synthetic experiment's index from 200-dimensional word vectors: 1000 documents of 1024 vectors, 11 hashes a table
        dict(name="build_words", kind="build", dtype="f16", docs=1000, lens="const1024", d=200, L=8, C=11),
        # a Sec. 4 aggregation: mean of the debiased sigmoid over the document, weighted query vectors
        dict(name="phi_mean", kind="phi", docs=20_000, lens="tokens", d=128, L=32, C=7, B=8, q=32, q_ragged=False,
             transform=dz.SCORE_MEAN_SIGMOID_Q16, weighted=True),
        # the paper's unit of latency: one query set through filter, scoring and top-k
        dict(name="filter_one", kind="filter", docs=1_000_000, lens="tokens", d=128, L=32, C=7, K=65_536, B=1, q=32,
             q_ragged=False, probe=1, fk=4096, k=10),
        # a batch in the paper's high-recall setting (4 probes, 8192 candidates, 1000 results)
        dict(name="filter_batch", kind="filter", docs=500_000, lens="tokens", d=128, L=32, C=6, K=32_768, B=128, q=32,
             q_ragged=False, probe=4, fk=8192, k=1000),
        # making the filter for a collection of 4M vectors
        dict(name="train", kind="train", docs=60_000, lens="tokens", d=128, K=16_384, sample=1 << 19, iters=2),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["search", "rerank", "sweep", "build", "phi", "filter", "train"])
    L = rng.choice([8, 16, 24, 32, 48, 64, 96, 128])
    C = rng.randint(4, 8)
    d = rng.choice([64, 128, 256])
    q = rng.randint(5, 70)
    ragged = rng.random() < 0.4
    lens = rng.choice(["tokens", "uniform"])
    if kind == "search":
        docs = _log(rng, 1000, 100_000)
        B = _log(rng, 1, 64)
        while docs * B * q * L > 100_000 * 64 * 32 * 32:
            docs, B = max(1000, docs * 2 // 3), max(1, B * 2 // 3)
        return dict(kind=kind, docs=docs, lens=lens, d=d, L=L, C=C, B=B, q=q, q_ragged=ragged, k=min(docs, _log(rng, 1, 1000)))
    if kind == "rerank":
        cand = _log(rng, 256, 16384)
        B = _log(rng, 1, 256)
        while cand * B * q * L > 256 * 4096 * 32 * 32:
            B = max(1, B * 2 // 3)
        return dict(kind=kind, docs=_log(rng, 20_000, 300_000), lens=lens, d=d, L=L, C=C, B=B, q=q, q_ragged=ragged, cand=cand,
                    cand_ragged=rng.random() < 0.4, k=min(cand, _log(rng, 1, 1000)))
    if kind == "sweep":
        e = rng.randint(1, 9)
        return dict(kind=kind, m=1 << e, L=8, C=e + 1, d=rng.choice([64, 100, 128, 200]), B=_log(rng, 1, 16), k=rng.randint(1, 100))
    if kind == "build":
        dtype = rng.choice(["i8", "f16"])
        d = rng.choice([50, 64, 96, 128, 200, 256, 300])
        C = rng.choice([4, 5, 6, 7, 8, 10, 12])
        docs = _log(rng, 100, 60_000)
        while docs * d * L * C > 30_000 * 256 * 64 * 8:
            docs = docs * 2 // 3
        return dict(kind=kind, dtype=dtype, docs=docs, lens=lens, d=d, L=L, C=C)
    if kind == "phi":
        docs = _log(rng, 500, 20_000)
        B = _log(rng, 1, 16)
        while docs * B * q * L > 20_000 * 8 * 32 * 32:
            docs, B = max(500, docs * 2 // 3), max(1, B * 2 // 3)
        return dict(kind=kind, docs=docs, lens=lens, d=d, L=L, C=C, B=B, q=q, q_ragged=ragged,
                    transform=rng.randint(dz.SCORE_EQ1_Q16, dz.SCORE_MEAN_SIGMOID_Q16), weighted=rng.random() < 0.5)
    if kind == "filter":
        fk = _log(rng, 256, 16384)
        B = _log(rng, 1, 128)
        while fk * B * q * L > 128 * 8192 * 32 * 32:
            B = max(1, B * 2 // 3)
        return dict(kind=kind, docs=_log(rng, 30_000, 300_000), lens=lens, d=rng.choice([64, 128]), L=L, C=C,
                    K=_log(rng, 2000, 32_768), B=B, q=q, q_ragged=ragged, probe=rng.choice([1, 2, 3, 4, 8]), fk=fk,
                    k=min(fk, _log(rng, 1, 1000)))
    docs = _log(rng, 2000, 40_000)
    return dict(kind="train", docs=docs, lens="tokens", d=rng.choice([64, 128]), K=_log(rng, 500, 16_384),
                sample=docs * rng.randint(4, 12), iters=rng.randint(1, 2))


# ---- inputs -------------------------------------------------------------------------------------------------------------
def _lengths(law, n, rng):
    """Document lengths: the same ones for every seed, so that arrays have the same shapes, in an order of the seed's own."""
    if law.startswith("const"):
        return np.full(n, int(law[5:]), np.uint32)
    drawn = np.random.default_rng(n)
    if law == "uniform":
        return rng.permutation(drawn.integers(16, 129, n).astype(np.uint32))
    return rng.permutation(np.clip(np.rint(drawn.normal(70.0, 25.0, n)), 8, 180).astype(np.uint32))


def _quantize(v, dtype):
    v = v / v.norm(dim=1, keepdim=True).clamp_min(1e-12)
    return (v * 127.0).round_().clamp_(-127, 127).to(torch.int8) if dtype == "i8" else v.to(torch.float16)


def _vectors(n, d, dtype, centres, g, dev):
    c = torch.randint(0, centres.shape[0], (n,), generator=g, device=dev)
    return _quantize(centres[c] + (SIGMA / math.sqrt(d)) * torch.randn(n, d, generator=g, device=dev), dtype)


def _noisy(v, dtype, g):
    v = v.float()
    v = v / v.norm(dim=1, keepdim=True).clamp_min(1e-12)
    return _quantize(v + (SIGMA_Q / math.sqrt(v.shape[1])) * torch.randn(v.shape, generator=g, device=v.device), dtype)


def _projection(L, C, d, dtype, seed, dev):
    g = torch.Generator(device=dev)
    g.manual_seed(7 * seed + 5)
    if dtype == "i8":
        return (torch.randint(0, 2, (L * C, d), generator=g, device=dev) * 2 - 1).to(torch.int8)
    return torch.randn(L * C, d, generator=g, device=dev)


def _make(case, seed, keep_vectors=False, index=True):
    """Lengths, projection, queries and (index=True) a handle with the index of the case's documents."""
    dev = torch.device("cuda", torch.cuda.current_device())
    rng = np.random.default_rng(seed)
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    dtype, d, L, C = case.get("dtype", "i8"), case["d"], case["L"], case["C"]
    if case["kind"] == "sweep":
        lens = np.full(1000, case["m"], np.uint32)
    else:
        lens = _lengths(case["lens"], case["docs"], rng)
    off = np.zeros(lens.size + 1, np.int64)
    np.cumsum(lens, out=off[1:])
    n = int(off[-1])
    s = dict(kind=case["kind"], lens=lens, off=off, n=n, dtype=dtype, d=d, L=L, C=C)
    s["proj"] = _projection(L, C, d, dtype, seed, dev)
    s["ix"] = dz.create(d, L, C, dtype=dz.I8 if dtype == "i8" else dz.F16,
                        proj_kind=dz.PROJ_RADEMACHER_I8 if dtype == "i8" else dz.PROJ_GAUSSIAN_F32, proj=s["proj"])
    # query rows: each query set is a noisy copy of vectors of one document
    rows = None
    if "B" in case:
        B, q = case["B"], case.get("q", case.get("m"))
        q_lens = rng.integers(max(1, q // 3), q + 1, B) if case.get("q_ragged") else np.full(B, q)
        s["q_lens"] = q_lens.astype(np.uint32)
        planted = rng.integers(0, lens.size, B)
        rows = np.concatenate([off[p] + rng.integers(0, lens[p], m) if case["kind"] != "sweep" else off[p] + np.arange(m)
                               for p, m in zip(planted, q_lens)])
        s["planted"] = planted
    centres = torch.randn(CENTRES, d, generator=g, device=dev) / math.sqrt(d)
    tdt = torch.int8 if dtype == "i8" else torch.float16
    src = torch.empty(0 if rows is None else rows.size, d, dtype=tdt, device=dev)
    docs = torch.empty(n, d, dtype=tdt, device=dev) if keep_vectors else None
    codes = torch.empty(n, L, dtype=dz.code_dtype(s["ix"]), device=dev) if index else None
    for lo in range(0, n, CHUNK):
        hi = min(n, lo + CHUNK)
        v = _vectors(hi - lo, d, dtype, centres, g, dev)
        if docs is not None:
            docs[lo:hi] = v
        if index:
            dz.hash(s["ix"], v, codes[lo:hi])
        if rows is not None:
            at = np.nonzero((rows >= lo) & (rows < hi))[0]
            if at.size:
                src[torch.from_numpy(at).to(dev)] = v[torch.from_numpy(rows[at] - lo).to(dev)]
    if rows is not None:
        s["queries"] = _noisy(src, dtype, g)
    if index:
        dz.attach_index(s["ix"], codes, torch.from_numpy(off).to(dev), int(lens.max()))
    s["docs"], s["codes"], s["g"], s["dev"], s["rng"] = docs, codes, g, dev, rng
    return s


def _result_buffers(s, B, k):
    s["ids"] = torch.empty(B, k, dtype=torch.uint32, device=s["dev"])
    s["scores"] = torch.empty(B, k, dtype=torch.int32, device=s["dev"])
    s["k"] = k


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("search", "sweep", "phi"):
        s = _make(case, seed)
        B, N = case["B"], s["lens"].size
        k = case.get("k", 0)
        s["ws"] = torch.empty(dz.workspace_bytes(s["ix"], B, s["queries"].shape[0], B * N, k), dtype=torch.uint8, device=s["dev"])
        if kind == "phi":
            dz.set_score_transform(s["ix"], case["transform"])
            s["weights"] = None
            if case["weighted"]:
                s["weights"] = torch.randint(0, 65537, (s["queries"].shape[0],), generator=s["g"], device=s["dev"], dtype=torch.int32)
                dz.set_query_weights(s["ix"], s["weights"])
            s["scores"] = torch.empty(B * N, dtype=torch.int32, device=s["dev"])
        else:
            _result_buffers(s, B, k)
        return s
    if kind == "rerank":
        s = _make(case, seed)
        B, N, n = case["B"], s["lens"].size, case["cand"]
        # distinct ids: one of each of n equal ranges of documents, shuffled; the planted document takes the first slot
        step = N / n
        lists, sizes = [], s["rng"].integers(n // 4, n + 1, B) if case["cand_ragged"] else np.full(B, n)
        ids = ((torch.arange(n, device=s["dev"]) + torch.rand(B, n, generator=s["g"], device=s["dev"], dtype=torch.float64)) * step)
        ids = ids.long().clamp_(max=N - 1)
        ids = ids.gather(1, torch.rand(B, n, generator=s["g"], device=s["dev"]).argsort(dim=1)).to(torch.int32)
        ids[:, 0] = torch.from_numpy(s["planted"]).to(s["dev"]).to(torch.int32)
        for b in range(B):
            lists.append(ids[b, : int(sizes[b])])
        s["cand"] = torch.cat(lists).contiguous()
        s["cand_off"] = np.concatenate([[0], np.cumsum(sizes)]).astype(np.uint64)
        s["ws"] = torch.empty(dz.workspace_bytes(s["ix"], B, s["queries"].shape[0], int(s["cand_off"][-1]), case["k"]),
                              dtype=torch.uint8, device=s["dev"])
        _result_buffers(s, B, case["k"])
        return s
    if kind == "build":
        s = _make(case, seed, keep_vectors=True, index=False)
        s["codes"] = torch.empty(s["n"], case["L"], dtype=dz.code_dtype(s["ix"]), device=s["dev"])
        s["offsets"] = torch.empty(s["lens"].size + 1, dtype=torch.int64, device=s["dev"])
        return s
    if kind == "filter":
        s = _make(case, seed, keep_vectors=True)
        cent = s["docs"][torch.randint(0, s["n"], (case["K"],), generator=s["g"], device=s["dev"])].contiguous()
        dz.filter_build(s["ix"], cent, s["docs"])
        s["docs"] = None
        s["probe"], s["fk"] = case["probe"], case["fk"]
        nbytes = dz.lib().dessert_filter_search_workspace_bytes(s["ix"].handle, case["B"], s["queries"].shape[0],
                                                                int(s["q_lens"].max()), case["probe"], case["fk"], case["k"])
        s["ws"] = torch.empty(int(nbytes), dtype=torch.uint8, device=s["dev"])
        _result_buffers(s, case["B"], case["k"])
        return s
    s = _make(dict(case, L=32, C=7), seed, keep_vectors=True)
    pick = torch.randint(0, s["n"], (case["sample"] + case["K"],), generator=s["g"], device=s["dev"])
    s["sample"] = s["docs"][pick[: case["sample"]]].contiguous()
    s["start"] = s["docs"][pick[case["sample"]:]].contiguous()
    s["iters"] = case["iters"]
    return s


def run(s):
    kind, ix = s["kind"], s["ix"]
    if kind in ("search", "sweep"):
        return dz.search(ix, s["queries"], s["q_lens"], s["k"], workspace=s["ws"], out_ids=s["ids"], out_scores=s["scores"])
    if kind == "rerank":
        return dz.search(ix, s["queries"], s["q_lens"], s["k"], cand_ids=s["cand"], cand_offsets=s["cand_off"], workspace=s["ws"],
                         out_ids=s["ids"], out_scores=s["scores"])
    if kind == "build":
        codes, offsets = dz.build_index(ix, s["docs"], s["lens"], s["codes"], s["offsets"])
        return codes if s["C"] <= 8 else codes.view(torch.int16), offsets      # torch does little with uint16
    if kind == "phi":
        return dz.scores(ix, s["queries"], s["q_lens"], workspace=s["ws"], out=s["scores"])
    if kind == "filter":
        return dz.filter_search(ix, s["queries"], s["q_lens"], s["probe"], s["fk"], s["k"], workspace=s["ws"], out_ids=s["ids"],
                                out_scores=s["scores"])
    centroids = dz.filter_kmeans(ix, s["sample"], s["start"], s["iters"])
    assign, starts, _ = dz.filter_build(ix, centroids, s["docs"])   # the documents inside a bucket are in no particular order
    return centroids, assign, starts


# ---- what the work is ---------------------------------------------------------------------------------------------------
def _mean_len(case):
    if case["kind"] == "sweep":
        return case["m"]
    law = case["lens"]
    return int(law[5:]) if law.startswith("const") else 72 if law == "uniform" else 70


def work(case):
    """bytes: every input once and every output once.  flops: multiply-adds of projections and distances as two, and one for
    each comparison of two codes."""
    kind = case["kind"]
    N = 1000 if kind == "sweep" else case["docs"]
    d, m = case["d"], _mean_len(case)
    if kind == "train":
        V = N * m
        pairs = (case["sample"] * case["iters"] + V) * case["K"]
        return {"bytes": (case["sample"] * case["iters"] + V) * (d + 4.0) + 2.0 * case["K"] * d, "flops": 2.0 * pairs * d}
    L, C = case["L"], case["C"]
    row = L * (1 if C <= 8 else 2)
    if kind == "build":
        w = 1 if case["dtype"] == "i8" else 2
        return {"bytes": N * m * (d * w + row) + 8.0 * N, "flops": 2.0 * N * m * d * L * C}
    B, q = case["B"], case.get("q", case.get("m"))
    q = q * 2 / 3 if case.get("q_ragged") else q
    hashing = 2.0 * B * q * d * L * C
    if kind in ("search", "sweep", "phi"):
        out = 4.0 * B * N if kind == "phi" else 8.0 * B * case["k"]
        return {"bytes": N * (m * row + 8.0) + B * q * d + out, "flops": hashing + float(B) * q * N * m * L}
    scored = B * (case["fk"] if kind == "filter" else case["cand"] * (0.625 if case["cand_ragged"] else 1.0))
    distinct = N * -math.expm1(-scored / N)
    flops = hashing + scored * q * m * L
    nbytes = distinct * (m * row + 8.0) + B * q * d + 4.0 * scored + 8.0 * B * case["k"]
    if kind == "filter":
        flops += 2.0 * B * q * case["K"] * d
        nbytes += case["K"] * (d + 4.0) + 4.0 * B * q * case["probe"] * N * m / case["K"]
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # Integers throughout, except the fp32 projections of fp16 vectors: a sign bit may turn where a projection is within the
    # rounding of its sum of zero.  2.4e-7 to 3.1e-7 of the codes are seen to differ from those of 64-bit projections; two such
    # computations may differ by twice that, and a small array's share moves in steps of one code.
    if case["kind"] == "build" and case["dtype"] == "f16":
        n = case["docs"] * _mean_len(case) * case["L"]
        return {"rel": 0.0, "differ": max(2.5e-6, 3.0 / n)}
    return "exact"


# ---- the same in 64 bits, from the vectors on ---------------------------------------------------------------------------
def _codes64(v, proj, L, C):
    out = torch.empty(v.shape[0], L, dtype=torch.int32, device=v.device)
    P = proj.double().t().contiguous()
    bit = (1 << torch.arange(C, device=v.device)).to(torch.int32)
    for lo in range(0, v.shape[0], 1 << 18):
        p = v[lo:lo + (1 << 18)].double() @ P
        out[lo:lo + (1 << 18)] = ((p >= 0).view(-1, L, C).to(torch.int32) * bit).sum(-1, dtype=torch.int32)
    return out


def _phi64(transform, L, C):
    """Table entries round(65536 * phi(count / L)), half away from zero."""
    t = [0]
    for c in range(1, L + 1):
        x = c / L
        if transform == dz.SCORE_EQ1_Q16:
            y = math.exp(math.log(x) / C)
        elif transform in (dz.SCORE_MAX_IDENTITY_Q16, dz.SCORE_MEAN_IDENTITY_Q16):
            y = x
        elif transform in (dz.SCORE_MAX_EXPM1_Q16, dz.SCORE_MEAN_EXPM1_Q16):
            y = math.exp(x) - 1.0
        else:
            y = 1.0 / (1.0 + math.exp(-x)) - 0.5
        t.append(int(math.floor(65536.0 * y + 0.5)))
    return t


def _scores64(codes, starts, counts, qc, table, mean, w):
    """Scores of the documents (starts, counts: rows of `codes`) against one query set's codes."""
    dev = codes.device
    out = torch.zeros(starts.numel(), dtype=torch.int64, device=dev)
    for lo in range(0, starts.numel(), 4096):
        st, ct = starts[lo:lo + 4096], counts[lo:lo + 4096]
        doc = torch.repeat_interleave(torch.arange(st.numel(), device=dev), ct)
        rows = torch.arange(doc.numel(), device=dev) - (torch.cumsum(ct, 0) - ct)[doc] + st[doc]
        x = codes[rows]
        cnt = torch.zeros(rows.numel(), qc.shape[0], dtype=torch.int64, device=dev)
        for t in range(codes.shape[1]):
            cnt += x[:, t, None] == qc[None, :, t]
        if table is not None:
            cnt = table[cnt]
        agg = torch.zeros(st.numel(), qc.shape[0], dtype=torch.int64, device=dev)
        agg.scatter_reduce_(0, doc[:, None].expand_as(cnt), cnt, "sum" if mean else "amax", include_self=True)
        if mean:
            agg = (agg + (ct // 2)[:, None]) // ct.clamp(min=1)[:, None]
        if w is not None:
            agg = (agg * w[None, :] + 32768) >> 16
        out[lo:lo + 4096] = agg.sum(1)
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind in ("filter", "train"):
        return None      # 64-bit distances of all vectors to all centroids take too long
    if kind != "build" and work(case)["flops"] > 1e11:
        return None
    s = _make(case, seed, keep_vectors=True, index=False) if kind != "rerank" and kind != "phi" else prepare(case, seed)
    if kind == "build":
        return _codes64(s["docs"], s["proj"], case["L"], case["C"]), torch.from_numpy(s["off"])
    docs = s["docs"] if s["docs"] is not None else _make(case, seed, keep_vectors=True, index=False)["docs"]
    codes = _codes64(docs, s["proj"], case["L"], case["C"])
    qcodes = _codes64(s["queries"], s["proj"], case["L"], case["C"])
    dev = s["dev"]
    starts, counts = torch.from_numpy(s["off"][:-1]).to(dev), torch.from_numpy(s["lens"].astype(np.int64)).to(dev)
    table, mean, w = None, False, None
    if kind == "phi":
        table = torch.tensor(_phi64(case["transform"], case["L"], case["C"]), device=dev)
        mean = case["transform"] >= dz.SCORE_MEAN_IDENTITY_Q16
        w = None if s["weights"] is None else s["weights"].long()
    ids, scores, at = [], [], 0
    for b, m in enumerate(s["q_lens"].tolist()):
        take = None
        if kind == "rerank":
            take = s["cand"][int(s["cand_off"][b]):int(s["cand_off"][b + 1])].long()
        sc = _scores64(codes, starts if take is None else starts[take], counts if take is None else counts[take],
                       qcodes[at:at + m], table, mean, None if w is None else w[at:at + m])
        at += m
        if kind == "phi":
            scores.append(sc)
            continue
        names = torch.arange(sc.numel(), device=dev) if take is None else take
        best = torch.argsort(sc * (1 << 32) + ((1 << 32) - 1 - names), descending=True)[: case["k"]]
        i = torch.full((case["k"],), 0xFFFFFFFF, dtype=torch.int64, device=dev)
        v = torch.full((case["k"],), -1, dtype=torch.int64, device=dev)
        i[: best.numel()], v[: best.numel()] = names[best], sc[best]
        ids.append(i)
        scores.append(v)
    if kind == "phi":
        return torch.stack(scores)
    return torch.stack(ids), torch.stack(scores)
