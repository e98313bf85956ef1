"""Chunk pairs of the mask-table kernel (query sets of more than 32 vectors, both masks of an entry from one set) under
DESSERT_SCORE_AUTO, bit for bit against the single-chunk forms of DESSERT_SCORE_MASKLUT and, for one set, the oracle."""
import re

import numpy as np
import pytest
import torch

import paper_2210_15748_amd as dz
from oracle import oracle as orc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
EMPTY = 0xFFFFFFFF


def launched(ix):
    m = re.fullmatch(r"score_masklut_kernel<(\d+), (\d+), (\d+), (\d+), (\d+), (true|false)>", dz.last_score_kernel(ix))
    assert m, dz.last_score_kernel(ix)
    return int(m.group(5)), m.group(6) == "true", int(m.group(4))


def paired(L, Cb, mode, form):
    """Whether the batches below are for chunk pairs: not with 64 tables (the single form is the rotated one), with 32 tables of up to
    5 bits only for lists that make 1536 workgroups; with weights no lists at up to 6 bits, and with 32 tables of 7 bits 1536
    workgroups."""
    if form == "weighted" and (Cb <= 6 and mode != "all split" or L == 32 and Cb <= 7 and mode == "lists split"):
        return False
    return L < 64 and not (L == 32 and Cb <= 5 and mode != "lists")


# every shape whose paired table fits.  Query sets of 33, 63, 64, 65, 96, 97 and 128 vectors: full and nearly empty second chunks, odd and
# even chunk counts; some of at most 32 among them.  Lists with empty slots, repeats, one of no ids and lengths that end inside a block;
# documents of no vectors
@pytest.mark.parametrize("form", ["raw", "eq1", "weighted"])
@pytest.mark.parametrize("mode", ["lists", "lists split", "all split"])
@pytest.mark.parametrize("L,Cb", [(8, 6), (8, 8), (8, 9), (8, 10), (16, 7), (16, 8), (16, 9), (32, 5), (32, 7), (32, 8), (64, 6)])
def test_chunk_pairs(L, Cb, mode, form):
    print("[case]", L, Cb, mode, form, flush=True)
    rng = np.random.default_rng(L * 100 + Cb)
    d = 64
    lens = np.concatenate([[0, 1, 7, 8, 9, 31, 33, 64, 65, 0, 180], rng.integers(0, 30, 1500)])
    pool = rng.integers(-100, 101, (9, d))
    near = lambda n, s: np.clip(pool[rng.integers(0, 9, n)] + rng.integers(-s, s + 1, (n, d)), -127, 127).astype(np.int8)
    if mode == "lists":
        q_lens = np.array([33, 64, 63, 40, 5, 64, 50, 48] * 8, dtype=np.int64)
    else:
        q_lens = np.array([128, 97, 65, 33, 128, 100, 120, 32, 96] * (3 if mode == "lists split" else 4), dtype=np.int64)
    X, Q = near(int(lens.sum()), 12), near(int(q_lens.sum()), 8)
    R = (rng.integers(0, 2, (L * Cb, d)) * 2 - 1).astype(np.int8)
    ix = dz.create(d, L, Cb, proj=torch.from_numpy(R).to(DEV))
    dz.build_index(ix, torch.from_numpy(X).to(DEV), lens)
    w = None
    if form != "raw":
        dz.set_score_transform(ix, dz.SCORE_EQ1_Q16 if form == "eq1" else dz.SCORE_MAX_SIGMOID_Q16)
    if form == "weighted":
        w = rng.integers(0, 65537, Q.shape[0]).astype(np.uint32)
        dz.set_query_weights(ix, torch.from_numpy(w.view(np.int32)).to(DEV))
    flat = co = None
    if mode != "all split":
        sizes = [1500, 1400, 1499, 1537, 1500, 1500, 1500, 1500] * 8 if mode == "lists" else [1001, 1000, 0, 1500, 1500, 999, 1501, 1500, 1300] * 3
        cands = [rng.integers(0, len(lens), n) for n in sizes]
        for c in cands:
            c[rng.random(len(c)) < 0.02] = EMPTY
        co = np.concatenate([[0], np.cumsum(sizes)])
        flat = torch.from_numpy(np.concatenate(cands).astype(np.uint32).view(np.int32)).to(DEV)
    got = {}
    for algo in (dz.SCORE_AUTO, dz.SCORE_MASKLUT):
        dz.set_algo(ix, dz.HASH_AUTO, algo)
        got[algo] = dz.scores(ix, torch.from_numpy(Q).to(DEV), q_lens, cand_ids=flat, cand_offsets=co).cpu().numpy().reshape(-1)
        W, split, remap = launched(ix)
        if algo == dz.SCORE_AUTO:
            assert W == (2 if paired(L, Cb, mode, form) else 1) and (W == 1 or split == (mode != "lists")), dz.last_score_kernel(ix)
            # instantiations of their own, told from pairs of sets
            assert remap == (5 if W == 2 else 0) + ["raw", "eq1", "weighted"].index(form)
        else:
            assert W == 1
    assert np.array_equal(got[dz.SCORE_AUTO], got[dz.SCORE_MASKLUT])
    b = 3
    qo, off = np.concatenate([[0], np.cumsum(q_lens)]), np.concatenate([[0], np.cumsum(lens)])
    dc, qc = orc.hash_i8(X, R, L, Cb), orc.hash_i8(Q[qo[b]:qo[b + 1]], R, L, Cb)
    sel = None if co is None else np.where(cands[b] == EMPTY, 0, cands[b]).astype(np.int64)
    if form == "raw":
        want = orc.scores(dc, off, qc, sel)
    elif form == "eq1":
        want = orc.scores_eq1(dc, off, qc, Cb, sel)
    else:
        want = orc.scores_general(dc, off, qc, orc.PHI_SIGMOID, orc.SIGMA_MAX, weights=w[qo[b]:qo[b + 1]], doc_ids=sel)
    mine = got[dz.SCORE_AUTO].reshape(len(q_lens), -1)[b] if co is None else got[dz.SCORE_AUTO][co[b]:co[b + 1]]
    assert np.array_equal(mine, want if co is None else np.where(cands[b] == EMPTY, -1, want))


# Where chunk pairs are the slower form although the paired table fits: 64 tables; 32 tables with few codes unless many lists; five chunks
# with tables of 64 KB; 16-byte rows of 8 tables in large batches of lists; three chunks
@pytest.mark.parametrize("L,Cb,q,n_sets,n_cand,want", [(64, 6, 64, 64, 1000, False), (64, 4, 128, 12, 0, False), (32, 4, 128, 64, 0, False),
                                                       (32, 5, 128, 8, 4096, False), (32, 4, 64, 64, 1600, True), (32, 6, 128, 64, 0, True),
                                                       (32, 8, 160, 64, 500, False), (32, 8, 128, 64, 500, True), (8, 10, 160, 64, 500, False),
                                                       (8, 10, 64, 64, 1000, True), (8, 10, 64, 256, 1100, False), (8, 9, 64, 256, 1100, True),
                                                       (16, 8, 96, 64, 500, False), (16, 8, 160, 64, 500, True)])
def test_which_batches_take_chunk_pairs(L, Cb, q, n_sets, n_cand, want):
    print("[case]", L, Cb, q, n_sets, n_cand, flush=True)
    rng = np.random.default_rng(q)
    lens = rng.integers(1, 5, 2000)
    ix = dz.create(64, L, Cb, seed=2)
    dz.build_index(ix, torch.from_numpy(rng.integers(-127, 128, (int(lens.sum()), 64)).astype(np.int8)).to(DEV), lens)
    Q = torch.from_numpy(rng.integers(-127, 128, (n_sets * q, 64)).astype(np.int8)).to(DEV)
    kw = {}
    if n_cand:
        kw = dict(cand_ids=torch.from_numpy(rng.integers(0, 2000, n_sets * n_cand).astype(np.int32)).to(DEV),
                  cand_offsets=np.arange(n_sets + 1) * n_cand)
    got = {}
    for algo in (dz.SCORE_AUTO, dz.SCORE_MASKLUT):
        dz.set_algo(ix, dz.HASH_AUTO, algo)
        got[algo] = dz.scores(ix, Q, np.full(n_sets, q), **kw).cpu().numpy()
        assert (launched(ix)[2] >= 5) == (want and algo == dz.SCORE_AUTO), dz.last_score_kernel(ix)
    assert np.array_equal(got[dz.SCORE_AUTO], got[dz.SCORE_MASKLUT])
