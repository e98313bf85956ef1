"""What the query-hashing launch carries along (the join of the probe lists, the clearing of scores that partial sums are added to), and the
filter's per-slab rows for counts above 126: against the oracle and the forms that do without."""
import numpy as np
import pytest
import torch

import paper_2210_15748_amd as dz
from oracle import oracle as orc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# 126, 130, 134, 138 and 254 to 257 bins, of which rows hold 256 at most (and the last two cases count to 255, a byte's largest, and beyond).  A
# set of equal vectors reaches the largest count.  A workspace without room for the wide rows is accepted; a timed call hashes in its own stage.
@pytest.mark.parametrize("n_sets", [2, 9])
@pytest.mark.parametrize("max_q,probe", [(31, 4), (32, 4), (33, 4), (34, 4), (63, 4), (127, 2), (255, 1), (128, 2)])
def test_counts_of_several_probes(max_q, probe, n_sets):
    print("[case]", max_q, probe, n_sets, flush=True)
    rng = np.random.default_rng(max_q)
    d, K, L, Cb, n_docs, filter_k, k = 128, 37, 32, 7, 70_001, 600, 50
    lens = rng.integers(0, 5, n_docs)
    lens[:3], lens[-2:] = [150, 0, 150], [150, 0]
    off = np.concatenate([[0], np.cumsum(lens)])
    pool = rng.integers(-100, 101, (K, d))
    Cn = np.clip(pool + rng.integers(-4, 5, (K, d)), -127, 127).astype(np.int8)
    X = np.clip(pool[rng.integers(0, K, off[-1])] + rng.integers(-50, 51, (off[-1], d)), -127, 127).astype(np.int8)
    R = (rng.integers(0, 2, (L * Cb, d)) * 2 - 1).astype(np.int8)
    q_lens = rng.integers(1, max_q + 1, n_sets)
    q_lens[0] = max_q
    qo = np.concatenate([[0], np.cumsum(q_lens)])
    Q = np.clip(Cn[rng.integers(0, K, qo[-1])].astype(np.int64) + rng.integers(-60, 61, (qo[-1], d)), -127, 127).astype(np.int8)
    Q[:max_q] = Q[0]
    ix = dz.create(d, L, Cb, proj=torch.from_numpy(R).to(DEV))
    dz.build_index(ix, torch.from_numpy(X).to(DEV), lens)
    dz.filter_build(ix, torch.from_numpy(Cn).to(DEV), torch.from_numpy(X).to(DEV))
    Qd = torch.from_numpy(Q).to(DEV)
    obo, obd = orc.inverted_index(orc.assign_centroids(X, Cn), off, K)
    dc, qc = orc.hash_i8(X, R, L, Cb), orc.hash_i8(Q, R, L, Cb)
    ids, cnt = (t.cpu().numpy() for t in dz.filter_query(ix, Qd, q_lens, probe, filter_k))
    assert cnt[0].max() == probe * max_q
    full = int(dz.lib().dessert_filter_search_workspace_bytes(ix.handle, n_sets, int(qo[-1]), max_q, probe, filter_k, k))
    got = []
    wide = 128 < probe * max_q + 2 <= 256
    if wide:   # rows of 256 counters per set and slab of 32 768 documents, not of 128
        narrow = dz.lib().dessert_filter_search_workspace_bytes(ix.handle, n_sets, int(qo[-1]), 126 // probe, probe, filter_k, k)
        assert full - int(narrow) >= n_sets * 3 * 128 * 4
    for nbytes in (full, full - 256) if wide else (full,):
        for timed in (False, True):
            ws = torch.full((nbytes,), 0x5A, dtype=torch.uint8, device=DEV)
            dz.enable_timing(ix, timed)
            got.append([t.cpu().numpy() for t in dz.filter_search(ix, Qd, q_lens, probe, filter_k, k, workspace=ws)])
    for b in range(n_sets):
        want, want_cnt = orc.filter_query(Q[qo[b]:qo[b + 1]], Cn, obo, obd, n_docs, probe, filter_k)
        assert np.array_equal(ids[b], want) and np.array_equal(cnt[b], want_cnt), b
        real = want[want != 0xFFFFFFFF].astype(np.int64)
        want_ids, want_sc = orc.topk(orc.scores(dc, off, qc[qo[b]:qo[b + 1]], real), k, real)
        for i, (a, s) in enumerate(got):
            assert np.array_equal(a[b], want_ids) and np.array_equal(s[b], want_sc), (b, i)


# long query sets over few documents: chunks split over workgroups that add into scores, which hold something else before each call
@pytest.mark.parametrize("lists", [False, True])
@pytest.mark.parametrize("L,Cb,transform,kernel", [(8, 9, dz.SCORE_RAW_COUNTS, "score_masklut_kernel<"), (32, 7, dz.SCORE_RAW_COUNTS, "score_masklut_kernel<"),
                                                   (64, 7, dz.SCORE_RAW_COUNTS, "score_masklut_kernel<"),
                                                   (32, 7, dz.SCORE_MEAN_SIGMOID_Q16, "score_bytecmp_kernel_masks<")])
def test_scores_cleared_while_hashing(L, Cb, transform, kernel, lists):
    print("[case]", L, Cb, transform, lists, flush=True)
    rng = np.random.default_rng(L + Cb)
    d, n_docs, q_lens = 128, 301, np.array([200, 130, 199])
    lens = rng.integers(0, 60, n_docs)
    pool = rng.integers(-100, 101, (9, d))
    near = lambda n, s: np.clip(pool[rng.integers(0, 9, n)] + rng.integers(-s, s + 1, (n, d)), -127, 127).astype(np.int8)
    ix = dz.create(d, L, Cb, seed=5)
    dz.build_index(ix, torch.from_numpy(near(int(lens.sum()), 25)).to(DEV), lens)
    dz.set_score_transform(ix, transform)
    Q = torch.from_numpy(near(int(q_lens.sum()), 20)).to(DEV)
    kw = dict(cand_ids=torch.from_numpy(rng.integers(0, n_docs, 600).astype(np.int32)).to(DEV), cand_offsets=np.array([0, 250, 255, 600])) if lists else {}
    got = {}
    for algo in (dz.SCORE_AUTO, dz.SCORE_AUTO, dz.SCORE_BYTECMP):
        dz.set_algo(ix, dz.HASH_AUTO, algo)
        ws = torch.full((1 << 20,), 0x5A, dtype=torch.uint8, device=DEV)
        ids, sc = dz.search(ix, Q, q_lens, 100, workspace=ws, **kw)
        if algo == dz.SCORE_AUTO:
            name = dz.last_score_kernel(ix)
            assert name.startswith(kernel) and ("masklut" not in kernel or name.endswith(", true>")), name   # chunks are split
        got.setdefault(algo, []).append((ids.cpu().numpy(), sc.cpu().numpy()))
    want = got[dz.SCORE_BYTECMP][0]
    for a, s in got[dz.SCORE_AUTO]:
        assert np.array_equal(a, want[0]) and np.array_equal(s, want[1])
