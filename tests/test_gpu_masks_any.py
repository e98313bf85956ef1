"""The mask-table kernel for any number of tables and for sigma = mean of any phi (DESSERT_SCORE_AUTO where the fixed-size kernel
does not apply) against the oracle and against the code-compare kernel, bit for bit."""
import numpy as np
import pytest
import torch

import paper_2210_15748_amd as dz
from oracle import oracle as orc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

KINDS = {dz.SCORE_EQ1_Q16: (orc.PHI_EQ1, orc.SIGMA_MAX), dz.SCORE_MAX_SIGMOID_Q16: (orc.PHI_SIGMOID, orc.SIGMA_MAX),
         dz.SCORE_MEAN_IDENTITY_Q16: (orc.PHI_IDENTITY, orc.SIGMA_MEAN), dz.SCORE_MEAN_EXPM1_Q16: (orc.PHI_EXPM1, orc.SIGMA_MEAN),
         dz.SCORE_MEAN_SIGMOID_Q16: (orc.PHI_SIGMOID, orc.SIGMA_MEAN)}


def case(seed, L, Cb, lens, q_lens):
    """Codes that collide often: vectors near a few pool vectors."""
    rng = np.random.default_rng(seed)
    d = 64
    pool = rng.integers(-100, 101, (9, d))
    near = lambda n, s: np.clip(pool[rng.integers(0, 9, n)] + rng.integers(-s, s + 1, (n, d)), -127, 127).astype(np.int8)
    X, Q = near(int(lens.sum()), 12), near(int(q_lens.sum()), 8)
    R = (rng.integers(0, 2, (L * Cb, d)) * 2 - 1).astype(np.int8)
    ix = dz.create(d, L, Cb, proj=torch.from_numpy(R).to(DEV))
    dz.build_index(ix, torch.from_numpy(X).to(DEV), lens)
    return rng, ix, X, Q, R


def check(ix, Q, q_lens, transform, weights, cands, X, R, L, Cb, lens, tag):
    Qd = torch.from_numpy(Q).to(DEV)
    dz.set_score_transform(ix, transform)
    dz.set_query_weights(ix, None if weights is None else torch.from_numpy(weights.view(np.int32)).to(DEV))
    flat = co = None
    if cands is not None:
        co = np.concatenate([[0], np.cumsum([len(c) for c in cands])])
        flat = torch.from_numpy(np.concatenate(cands).astype(np.uint32).view(np.int32)).to(DEV)
    got = {}
    for algo in (dz.SCORE_AUTO, dz.SCORE_BYTECMP):
        dz.set_algo(ix, dz.HASH_AUTO, algo)
        got[algo] = dz.scores(ix, Qd, q_lens, cand_ids=flat, cand_offsets=co).cpu().numpy().reshape(-1)
        name = dz.last_score_kernel(ix)
        assert name.startswith("score_bytecmp_kernel_masks<" if algo == dz.SCORE_AUTO else "score_bytecmp_kernel<"), name
    assert np.array_equal(got[dz.SCORE_AUTO], got[dz.SCORE_BYTECMP]), tag
    # and the oracle, for one query set
    b, off = len(q_lens) - 1, np.concatenate([[0], np.cumsum(lens)])
    qo = np.concatenate([[0], np.cumsum(q_lens)])
    dc, qc = orc.hash_i8(X, R, L, Cb), orc.hash_i8(Q[qo[b]:qo[b + 1]], R, L, Cb)
    sel = None if cands is None else np.where(cands[b] == 0xFFFFFFFF, 0, cands[b]).astype(np.int64)
    if transform == dz.SCORE_RAW_COUNTS:
        want = orc.scores(dc, off, qc, sel)
    else:
        phi, sigma = KINDS[transform]
        want = orc.scores_general(dc, off, qc, phi, sigma, weights=None if weights is None else weights[qo[b]:qo[b + 1]], doc_ids=sel, eq1_C=Cb)
    if sel is not None:
        want = np.where(cands[b] == 0xFFFFFFFF, -1, want)
    mine = got[dz.SCORE_AUTO][co[b]:co[b + 1]] if cands is not None else got[dz.SCORE_AUTO].reshape(len(q_lens), -1)[b]
    assert np.array_equal(mine, want), tag


# every remainder of L mod 16 (groups of 4, 8, 12 and 16 tables), every instantiation (L <= 16, 32, 64, 128; both code widths),
# tables of 256 bytes to 128 KB (all three workgroup sizes), query sets of one vector up to several chunks of 32
@pytest.mark.parametrize("L,Cb", [(4, 4), (12, 5), (20, 7), (24, 8), (28, 3), (36, 6), (44, 8), (48, 7), (60, 5), (72, 6), (96, 8), (100, 7), (124, 8),
                                  (4, 13), (12, 11), (16, 11), (24, 10), (28, 9), (48, 9), (32, 10), (64, 9)])
def test_any_table_count(L, Cb):
    print("[case]", L, Cb, flush=True)
    head = np.array([0, 1, 7, 8, 9, 70, 0, 31, 33, 64, 65, 2, 300])
    lens = np.concatenate([head, np.random.default_rng(L).integers(0, 40, 300)])
    q_lens = np.array([1, 32, 33, 70, 7], dtype=np.int64)
    rng, ix, X, Q, R = case(L * 100 + Cb, L, Cb, lens, q_lens)
    w = rng.integers(0, 65537, Q.shape[0]).astype(np.uint32)
    w[:3] = [65536, 0, 1]
    cands = [rng.integers(0, len(lens), n) for n in (50, 1, 257, 8, 129)]
    cands[4][7] = cands[2][0] = 0xFFFFFFFF
    for transform, weights in ((dz.SCORE_RAW_COUNTS, None), (dz.SCORE_EQ1_Q16, w), (dz.SCORE_MAX_SIGMOID_Q16, None), (dz.SCORE_MEAN_EXPM1_Q16, w),
                               (dz.SCORE_MEAN_SIGMOID_Q16, None)):
        for c in (None, cands):
            check(ix, Q, q_lens, transform, weights, c, X, R, L, Cb, lens, (transform, c is not None))
    if L & (L - 1):      # a power of two has the fixed-size kernel's form of this mean
        check(ix, Q, q_lens, dz.SCORE_MEAN_IDENTITY_Q16, w, None, X, R, L, Cb, lens, "mean identity")


@pytest.mark.parametrize("L,Cb", [(8, 6), (16, 8), (32, 7), (64, 8), (128, 7), (8, 11), (32, 9)])
@pytest.mark.parametrize("transform", [dz.SCORE_MEAN_EXPM1_Q16, dz.SCORE_MEAN_SIGMOID_Q16])
def test_mean_of_other_phi_at_the_fixed_table_counts(L, Cb, transform):
    """Long candidate lists (grouped by id range) and a grid of many workgroups; documents up to several hundred vectors."""
    print("[case]", L, Cb, transform, flush=True)
    rng0 = np.random.default_rng(L + Cb)
    lens = np.concatenate([rng0.integers(0, 30, 3000), [500, 0, 64]])
    q_lens = np.array([32, 5, 40, 8, 1, 31, 16, 64], dtype=np.int64)
    rng, ix, X, Q, R = case(L * 10 + Cb, L, Cb, lens, q_lens)
    check(ix, Q, q_lens, transform, None, None, X, R, L, Cb, lens, "all")
    check(ix, Q, q_lens, transform, rng.integers(0, 65537, Q.shape[0]).astype(np.uint32), [rng.integers(0, len(lens), 1500) for _ in q_lens], X, R, L,
          Cb, lens, "lists")


def test_mean_falls_back_where_32_bit_sums_do_not_fit():
    """phi(1) = e - 1 in Q16 is 112609: 38 140 of them and the rounding term 19 070 are below 2^32, 38 141 and 19 070 are not."""
    for m, masks in ((38140, True), (38141, False)):
        lens = np.array([5, m, 3])
        q_lens = np.array([40], dtype=np.int64)                # enough query vectors for the mask table where it can be taken
        rng, ix, X, Q, R = case(m, 32, 4, lens, q_lens)
        X[5:] = X[5]                                          # every vector of the long document collides in every table
        Q[:] = X[5]
        dz.build_index(ix, torch.from_numpy(X).to(DEV), lens)
        dz.set_score_transform(ix, dz.SCORE_MEAN_EXPM1_Q16)
        got = dz.scores(ix, torch.from_numpy(Q).to(DEV), q_lens).cpu().numpy()[0]
        assert dz.last_score_kernel(ix).startswith("score_bytecmp_kernel_masks<" if masks else "score_bytecmp_kernel<")
        dc, qc = orc.hash_i8(X, R, 32, 4), orc.hash_i8(Q, R, 32, 4)
        want = orc.scores_general(dc, np.concatenate([[0], np.cumsum(lens)]), qc, orc.PHI_EXPM1, orc.SIGMA_MEAN, eq1_C=4)
        assert np.array_equal(got, want)


# A few query vectors against few or long documents are for the code-compare kernel (a wave per document, query vectors one by one),
# more of them for the mask table (eight lanes per document, 32 query vectors at once)
@pytest.mark.parametrize("L,Cb,N,m,n_sets,q,transform,masks",
                         [(4, 4, 20, 3000, 1, 1, dz.SCORE_MEAN_SIGMOID_Q16, False), (4, 4, 20, 600, 1, 4, dz.SCORE_MEAN_SIGMOID_Q16, False),
                          (4, 4, 20, 600, 1, 64, dz.SCORE_MEAN_SIGMOID_Q16, True), (96, 8, 200, 1, 1, 1, dz.SCORE_RAW_COUNTS, False),
                          (96, 8, 1500, 120, 64, 8, dz.SCORE_RAW_COUNTS, True), (128, 7, 1500, 120, 64, 1, dz.SCORE_MEAN_EXPM1_Q16, True),
                          (12, 7, 1500, 30, 8, 16, dz.SCORE_RAW_COUNTS, True), (64, 9, 20, 120, 8, 2, dz.SCORE_RAW_COUNTS, False)])
def test_which_kernel_takes_a_few_query_vectors(L, Cb, N, m, n_sets, q, transform, masks):
    print("[case]", L, Cb, N, m, n_sets, q, transform, flush=True)
    rng = np.random.default_rng(L + N)
    ix = dz.create(64, L, Cb, seed=4)
    dz.build_index(ix, torch.from_numpy(rng.integers(-127, 128, (N * m, 64)).astype(np.int8)).to(DEV), np.full(N, m))
    Q = torch.from_numpy(rng.integers(-127, 128, (n_sets * q, 64)).astype(np.int8)).to(DEV)
    dz.set_score_transform(ix, transform)
    got = {}
    for algo in (dz.SCORE_AUTO, dz.SCORE_BYTECMP):
        dz.set_algo(ix, dz.HASH_AUTO, algo)
        got[algo] = dz.scores(ix, Q, np.full(n_sets, q)).cpu().numpy()
        mask_kernel = dz.last_score_kernel(ix).startswith("score_bytecmp_kernel_masks<")
        assert mask_kernel == (masks and algo == dz.SCORE_AUTO), dz.last_score_kernel(ix)
    assert np.array_equal(got[dz.SCORE_AUTO], got[dz.SCORE_BYTECMP])


# grids that make whole rounds over the chip: block sizes that are no power of two, a last block that is not full, tables of every thread count
@pytest.mark.parametrize("transform", [dz.SCORE_RAW_COUNTS, dz.SCORE_MEAN_SIGMOID_Q16])
@pytest.mark.parametrize("L,Cb,n_docs,n_sets", [(12, 5, 22_003, 3), (24, 7, 17_001, 4), (36, 6, 66_001, 1), (96, 7, 13_005, 5), (96, 8, 33_001, 1), (24, 9, 17_003, 4)])
def test_whole_rounds(L, Cb, n_docs, n_sets, transform):
    print("[case]", L, Cb, n_docs, n_sets, transform, flush=True)
    rng = np.random.default_rng(L + n_docs)
    lens = rng.integers(0, 4, n_docs)
    lens[:4], lens[-2:] = [0, 300, 1, 9], [17, 0]
    pool = rng.integers(-100, 101, (9, 64))
    near = lambda n, s: np.clip(pool[rng.integers(0, 9, n)] + rng.integers(-s, s + 1, (n, 64)), -127, 127).astype(np.int8)
    ix = dz.create(64, L, Cb, seed=3)
    dz.build_index(ix, torch.from_numpy(near(int(lens.sum()), 25)).to(DEV), lens)
    dz.set_score_transform(ix, transform)
    q_lens = rng.integers(20, 33, n_sets)
    Q = torch.from_numpy(near(int(q_lens.sum()), 20)).to(DEV)
    got = {}
    for algo in (dz.SCORE_AUTO, dz.SCORE_BYTECMP):
        dz.set_algo(ix, dz.HASH_AUTO, algo)
        got[algo] = dz.scores(ix, Q, q_lens).cpu().numpy()
        assert dz.last_score_kernel(ix).startswith("score_bytecmp_kernel_masks") == (algo == dz.SCORE_AUTO), dz.last_score_kernel(ix)
    assert np.array_equal(got[dz.SCORE_AUTO], got[dz.SCORE_BYTECMP])
