"""Every document scored for four query sets per workgroup (large batches under DESSERT_SCORE_AUTO), and blocks of documents that make whole
rounds over the chip: bit for bit against the forms of DESSERT_SCORE_MASKLUT and, for one set, the oracle."""
import re

import numpy as np
import pytest
import torch

import paper_2210_15748_amd as dz
from oracle import oracle as orc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def launched(ix):
    m = re.fullmatch(r"score_masklut_kernel<(\d+), (\d+), (\d+), (\d+), (\d+), (true|false)>", dz.last_score_kernel(ix))
    assert m, dz.last_score_kernel(ix)
    return int(m.group(5))


# every shape that has the form, and some that have not.  Documents of no, one and many vectors, more of them than one block holds and a
# number that fills no block; sets of one chunk, of two, and of unequal numbers of chunks; batches whose last workgroup lacks a set
@pytest.mark.parametrize("form", ["raw", "eq1", "weighted"])
@pytest.mark.parametrize("n_sets,q", [(4, "even"), (7, "ragged"), (16, "even"), (23, "long"), (16, "unequal"), (5, "even")])
@pytest.mark.parametrize("L,Cb", [(8, 5), (8, 7), (8, 8), (8, 9), (16, 6), (16, 7), (16, 8), (32, 6), (32, 7), (32, 8), (64, 6), (128, 6)])
def test_four_sets(L, Cb, n_sets, q, form):
    print("[case]", L, Cb, n_sets, q, form, flush=True)
    rng = np.random.default_rng(L * 100 + Cb + n_sets)
    d, groups = 64, (n_sets + 3) // 4
    n_docs = 256 * ((256 + groups - 1) // groups) + 3
    lens = rng.integers(0, 4, n_docs)
    lens[:8] = [0, 1, 260, 7, 9, 65, 0, 3]
    lens[-2:] = [33, 0]
    q_lens = {"even": np.full(n_sets, 9), "ragged": rng.integers(1, 33, n_sets), "long": rng.integers(33, 65, n_sets),
              "unequal": np.where(np.arange(n_sets) % 3 == 1, 40, 5)}[q]
    pool = rng.integers(-100, 101, (9, d))
    near = lambda n, s: np.clip(pool[rng.integers(0, 9, n)] + rng.integers(-s, s + 1, (n, d)), -127, 127).astype(np.int8)
    X, Q = near(int(lens.sum()), 25), near(int(q_lens.sum()), 20)
    R = (rng.integers(0, 2, (L * Cb, d)) * 2 - 1).astype(np.int8)
    ix = dz.create(d, L, Cb, proj=torch.from_numpy(R).to(DEV))
    dz.build_index(ix, torch.from_numpy(X).to(DEV), lens)
    w = None
    if form != "raw":
        dz.set_score_transform(ix, dz.SCORE_EQ1_Q16)
    if form == "weighted":
        w = rng.integers(0, 65537, Q.shape[0]).astype(np.uint32)
        dz.set_query_weights(ix, torch.from_numpy(w.view(np.int32)).to(DEV))
    got = {}
    for algo in (dz.SCORE_AUTO, dz.SCORE_MASKLUT):
        dz.set_algo(ix, dz.HASH_AUTO, algo)
        got[algo] = dz.scores(ix, torch.from_numpy(Q).to(DEV), q_lens).cpu().numpy().reshape(n_sets, n_docs)
        fits = L <= 32 and (L << max(Cb, 6)) * 16 <= 65536
        four = algo == dz.SCORE_AUTO and fits and form != "weighted" and q != "unequal" and n_sets != 5
        assert (launched(ix) == 4) == four, dz.last_score_kernel(ix)
    assert np.array_equal(got[dz.SCORE_AUTO], got[dz.SCORE_MASKLUT])
    b = n_sets - 1
    qo, off = np.concatenate([[0], np.cumsum(q_lens)]), np.concatenate([[0], np.cumsum(lens)])
    dc, qc = orc.hash_i8(X, R, L, Cb), orc.hash_i8(Q[qo[b]:qo[b + 1]], R, L, Cb)
    if form == "raw":
        want = orc.scores(dc, off, qc, None)
    elif form == "eq1":
        want = orc.scores_eq1(dc, off, qc, Cb, None)
    else:
        want = orc.scores_general(dc, off, qc, orc.PHI_EQ1, orc.SIGMA_MAX, weights=w[qo[b]:qo[b + 1]], eq1_C=Cb)
    assert np.array_equal(got[dz.SCORE_AUTO][b], want)


# four chunks of one set per workgroup: 8 tables, sets of four and more chunks, the last four of two, three or four of them; long documents,
# some empty or short; every document scored and lists with empty slots; one call with the chunks split over workgroups
@pytest.mark.parametrize("lists", [False, True])
@pytest.mark.parametrize("n_sets,q,want", [(8, 100, True), (16, 128, True), (16, 224, True), (8, 256, True), (60, 190, True), (16, 160, False), (2, 128, False)])
@pytest.mark.parametrize("Cb", [5, 7, 8, 9])
def test_four_chunks(Cb, n_sets, q, want, lists):
    print("[case]", Cb, n_sets, q, lists, flush=True)
    rng = np.random.default_rng(Cb * 1000 + q + n_sets)
    d, L, n_docs = 64, 8, 900
    lens = rng.integers(50, 110, n_docs)
    lens[:6] = [0, 1, 260, 7, 0, 65]
    lens[-1] = 0
    pool = rng.integers(-100, 101, (9, d))
    near = lambda n, s: np.clip(pool[rng.integers(0, 9, n)] + rng.integers(-s, s + 1, (n, d)), -127, 127).astype(np.int8)
    X, Q = near(int(lens.sum()), 25), near(n_sets * q, 20)
    R = (rng.integers(0, 2, (L * Cb, d)) * 2 - 1).astype(np.int8)
    ix = dz.create(d, L, Cb, proj=torch.from_numpy(R).to(DEV))
    dz.build_index(ix, torch.from_numpy(X).to(DEV), lens)
    kw, sel = {}, [None] * n_sets
    if lists:
        sizes = rng.integers(700, 1001, n_sets)
        sizes[-1] = 1000
        sel = [rng.integers(0, n_docs, n).astype(np.uint32) for n in sizes]
        for c in sel:
            c[rng.random(len(c)) < 0.02] = 0xFFFFFFFF
        kw = dict(cand_ids=torch.from_numpy(np.concatenate(sel).view(np.int32)).to(DEV), cand_offsets=np.concatenate([[0], np.cumsum(sizes)]))
    got = {}
    for algo in (dz.SCORE_AUTO, dz.SCORE_MASKLUT):
        dz.set_algo(ix, dz.HASH_AUTO, algo)
        got[algo] = dz.scores(ix, torch.from_numpy(Q).to(DEV), np.full(n_sets, q), **kw).cpu().numpy().reshape(-1)
        assert (launched(ix) == 4) == (want and algo == dz.SCORE_AUTO), dz.last_score_kernel(ix)
    assert np.array_equal(got[dz.SCORE_AUTO], got[dz.SCORE_MASKLUT])
    b, off = n_sets - 1, np.concatenate([[0], np.cumsum(lens)])
    dc, qc = orc.hash_i8(X, R, L, Cb), orc.hash_i8(Q[b * q:], R, L, Cb)
    ids = None if sel[b] is None else np.where(sel[b] == 0xFFFFFFFF, 0, sel[b]).astype(np.int64)
    expect = orc.scores(dc, off, qc, ids)
    if ids is not None:
        expect = np.where(sel[b] == 0xFFFFFFFF, -1, expect)
    assert np.array_equal(got[dz.SCORE_AUTO][-len(expect):], expect)
