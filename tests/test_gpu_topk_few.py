"""The selection of a few results (k <= 16) from lists of at most 4096 scores against the oracle: list lengths either side of a wave's 512
and of a workgroup's 4096 scores, lists shorter than k, heavy ties, repeated ids, empty slots; the longer lists beside them."""
import numpy as np
import pytest
import torch

import paper_2210_15748_amd as dz
from oracle import oracle as orc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("k", [1, 2, 7, 8, 15, 16, 17])
@pytest.mark.parametrize("N,lens_of_lists", [(60, [1, 5, 60, 33, 0]), (700, [511, 512, 513, 700, 3]), (5000, [4096, 4095, 1025, 1024, 31]),
                                             (5000, [4097, 5000, 64, 1, 2])])
def test_few_results(N, lens_of_lists, k):
    print("[case]", N, lens_of_lists, k, flush=True)
    rng = np.random.default_rng(N + k)
    d, L, Cb = 64, 4, 2                                    # scores of few values: large groups of ties
    lens = rng.integers(1, 3, N)
    X = rng.integers(-127, 128, (int(lens.sum()), d)).astype(np.int8)
    R = (rng.integers(0, 2, (L * Cb, d)) * 2 - 1).astype(np.int8)
    ix = dz.create(d, L, Cb, proj=torch.from_numpy(R).to(DEV))
    dz.build_index(ix, torch.from_numpy(X).to(DEV), lens)
    q_lens = np.array([2, 1, 3, 2, 4], dtype=np.int64)
    Q = rng.integers(-127, 128, (12, d)).astype(np.int8)
    qo, off = np.concatenate([[0], np.cumsum(q_lens)]), np.concatenate([[0], np.cumsum(lens)])
    dc, qc = orc.hash_i8(X, R, L, Cb), orc.hash_i8(Q, R, L, Cb)
    Qd = torch.from_numpy(Q).to(DEV)
    scores = [orc.scores(dc, off, qc[qo[b]:qo[b + 1]]) for b in range(5)]
    ids, sc = (t.cpu().numpy() for t in dz.search(ix, Qd, q_lens, k))
    for b in range(5):
        want_ids, want_sc = orc.topk(scores[b], k)
        assert np.array_equal(ids[b], want_ids) and np.array_equal(sc[b], want_sc), b
    cands = [rng.integers(0, N, n) for n in lens_of_lists]
    if len(cands[2]) > 4:
        cands[2][2] = cands[2][0]                          # an id listed twice appears twice
    co = np.concatenate([[0], np.cumsum(lens_of_lists)])
    flat = np.concatenate(cands).astype(np.uint32)
    hole = rng.random(len(flat)) < 0.05
    flat_dev = torch.from_numpy(np.where(hole, 0xFFFFFFFF, flat).astype(np.uint32).view(np.int32)).to(DEV)
    ids, sc = (t.cpu().numpy() for t in dz.search(ix, Qd, q_lens, k, cand_ids=flat_dev, cand_offsets=co))
    for b in range(5):
        c = cands[b][~hole[co[b]:co[b + 1]]]
        order = np.lexsort((c, -scores[b][c].astype(np.int64)))[:k]
        want_ids, want_sc = np.full(k, 0xFFFFFFFF, np.uint32), np.full(k, -1, np.int32)
        want_ids[:len(order)], want_sc[:len(order)] = c[order], scores[b][c][order]
        assert np.array_equal(ids[b], want_ids) and np.array_equal(sc[b], want_sc), b


def test_few_results_of_a_list_cut_into_slices():
    """One query set over 40 000 documents: four slices of 10 000, a list that the selection of a few results leaves to the general
    one and its merge."""
    rng = np.random.default_rng(1)
    d, L, Cb, N = 64, 8, 3, 40_000
    X = rng.integers(-127, 128, (N, d)).astype(np.int8)
    ix = dz.create(d, L, Cb, seed=5)
    R = dz.get_projection(ix).cpu().numpy()
    dz.build_index(ix, torch.from_numpy(X).to(DEV), np.ones(N, dtype=np.int64))
    Q = rng.integers(-127, 128, (7, d)).astype(np.int8)
    dc, qc = orc.hash_i8(X, R, L, Cb), orc.hash_i8(Q, R, L, Cb)
    for k in (1, 10, 16):
        ids, sc = (t.cpu().numpy() for t in dz.search(ix, torch.from_numpy(Q).to(DEV), [7], k))
        want_ids, want_sc = orc.topk(orc.scores(dc, np.arange(N + 1), qc), k)
        assert np.array_equal(ids[0], want_ids) and np.array_equal(sc[0], want_sc)


@pytest.mark.parametrize("k", [17, 1000, 5000])
def test_lists_that_stay_in_registers(k):
    """Lists either side of 4096 and of 16 384 scores, the lengths at which the selection changes its workgroup."""
    rng = np.random.default_rng(k)
    d, L, Cb, N = 64, 4, 2, 20_000
    X = rng.integers(-127, 128, (N, d)).astype(np.int8)
    ix = dz.create(d, L, Cb, seed=3)
    R = dz.get_projection(ix).cpu().numpy()
    dz.build_index(ix, torch.from_numpy(X).to(DEV), np.ones(N, dtype=np.int64))
    Q = rng.integers(-127, 128, (6, d)).astype(np.int8)
    dc, qc = orc.hash_i8(X, R, L, Cb), orc.hash_i8(Q, R, L, Cb)
    score = orc.scores(dc, np.arange(N + 1), qc[:2])
    for n in (4096, 4097, 8191, 16384, 16385):
        print("[case]", n, k, flush=True)
        lists = [rng.integers(0, N, n), rng.integers(0, N, n // 2), rng.integers(0, N, 3)]
        co = np.concatenate([[0], np.cumsum([len(c) for c in lists])])
        flat = torch.from_numpy(np.concatenate(lists).astype(np.int32)).to(DEV)
        ids, sc = (t.cpu().numpy() for t in dz.search(ix, torch.from_numpy(np.concatenate([Q[:2]] * 3)).to(DEV), [2, 2, 2], k, cand_ids=flat, cand_offsets=co))
        for b, c in enumerate(lists):
            order = np.lexsort((c, -score[c].astype(np.int64)))[:k]
            want_ids, want_sc = np.full(k, 0xFFFFFFFF, np.uint32), np.full(k, -1, np.int32)
            want_ids[:len(order)], want_sc[:len(order)] = c[order], score[c][order]
            assert np.array_equal(ids[b], want_ids) and np.array_equal(sc[b], want_sc), (n, b)
