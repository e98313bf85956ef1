"""The passes around the filter's GEMM where their paths branch: bucket building for documents either side of the LDS set's limits,
scans over several parts, merges of the per-range lists, against the oracle."""
import numpy as np
import pytest
import torch

import paper_2210_15748_amd as dz
from oracle import oracle as orc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def index(rng, lens, d=64, L=8, Cb=4):
    X = rng.integers(-127, 128, (int(lens.sum()), d)).astype(np.int8)
    R = (rng.integers(0, 2, (L * Cb, d)) * 2 - 1).astype(np.int8)
    ix = dz.create(d, L, Cb, proj=torch.from_numpy(R).to(DEV))
    dz.build_index(ix, torch.from_numpy(X).to(DEV), lens)
    return ix, X


def buckets_equal(starts, docs, want_starts, want_docs):
    assert np.array_equal(starts, want_starts)
    for c in range(len(starts) - 1):
        assert np.array_equal(np.sort(docs[starts[c]:starts[c + 1]]), np.sort(want_docs[starts[c]:starts[c + 1]])), c


# few centroids: nearly every vector of a document repeats one; many: nearly none does.  Lengths either side of the set's three sizes
# (96, 192 and 384 vectors fill 3/4 of 128, 256 and 512 slots), of whole passes of 64 and of the fall-back
@pytest.mark.parametrize("K", [1, 2, 33, 700, 5000])
def test_buckets_of_documents_of_every_length_class(K):
    print("[case]", K, flush=True)
    rng = np.random.default_rng(K)
    lens = np.array([0, 1, 63, 64, 65, 95, 96, 97, 128, 129, 191, 192, 193, 256, 257, 383, 384, 385, 449, 1000, 0] + [5] * 40)
    ix, X = index(rng, lens)
    C = X[rng.permutation(X.shape[0])[:K]].copy() if K <= X.shape[0] else rng.integers(-127, 128, (K, 64)).astype(np.int8)
    assign, starts, docs = (t.cpu().numpy() for t in dz.filter_build(ix, torch.from_numpy(C).to(DEV), torch.from_numpy(X).to(DEV)))
    want = orc.assign_centroids(X, C)
    assert np.array_equal(assign.view(np.uint32), want)
    ws, wd = orc.inverted_index(want, np.concatenate([[0], np.cumsum(lens)]), K)
    buckets_equal(starts.view(np.uint32).astype(np.int64), docs.view(np.uint32), np.asarray(ws, dtype=np.int64), np.asarray(wd))


# the scan's parts hold 4096 entries: one part, exactly full, one more entry, several parts
@pytest.mark.parametrize("K", [4095, 4096, 4097, 20_000])
def test_bucket_starts_over_several_scan_parts(K):
    rng = np.random.default_rng(K)
    lens = rng.integers(0, 30, 1500)
    ix, X = index(rng, lens)
    C = rng.integers(-127, 128, (K, 64)).astype(np.int8)
    assign, starts, docs = (t.cpu().numpy() for t in dz.filter_build(ix, torch.from_numpy(C).to(DEV), torch.from_numpy(X).to(DEV)))
    ws, wd = orc.inverted_index(assign.view(np.uint32), np.concatenate([[0], np.cumsum(lens)]), K)
    buckets_equal(starts.view(np.uint32).astype(np.int64), docs.view(np.uint32), np.asarray(ws, dtype=np.int64), np.asarray(wd))


# probes 2, 3, 4, 5 and 8 (every list width, full or not); centroids that repeat (ties to the lower id); tiles of one chunk of eight,
# a chunk and one tile, several ranges; the values themselves decide at the end of a chunk
@pytest.mark.parametrize("K", [9, 32, 256, 257, 290, 3000])
@pytest.mark.parametrize("probe", [2, 3, 4, 5, 8])
@pytest.mark.parametrize("d", [64, 128, 256])
def test_probes_with_ties_over_chunks(d, probe, K):
    print("[case]", d, probe, K, flush=True)
    rng = np.random.default_rng(K + probe)
    lens = rng.integers(1, 12, 400)
    ix, X = index(rng, lens, d=d)
    C = rng.integers(-127, 128, (K, d)).astype(np.int8)
    C[rng.integers(0, K, K // 3)] = C[0]                        # a third of the centroids equal
    C[K - 1] = -128
    q_lens = np.array([5, 40, 1], dtype=np.int64)
    Q = np.concatenate([X[rng.integers(0, X.shape[0], 44)], C[:1], np.full((1, d), 127, np.int8)])
    assign, starts, docs = (t.cpu().numpy() for t in dz.filter_build(ix, torch.from_numpy(C).to(DEV), torch.from_numpy(X).to(DEV)))
    ids, counts = dz.filter_query(ix, torch.from_numpy(Q).to(DEV), q_lens, probe, 60)
    qo = np.concatenate([[0], np.cumsum(q_lens)])
    for b in range(len(q_lens)):
        want_ids, want_counts = orc.filter_query(Q[qo[b]:qo[b + 1]], C, starts.view(np.uint32), docs.view(np.uint32), len(lens), probe, 60)
        assert np.array_equal(counts.cpu().numpy()[b], want_counts)
        assert np.array_equal(ids.cpu().numpy()[b], want_ids)


# n: less than a group's positions, either side of a workgroup's 256 (the form for fewer than 2^17 vectors), several workgroups; one
# cluster for all, clusters that span groups and workgroups, most clusters empty; either side of n = 370 sqrt(K), below which the vectors
# are not ordered.  The smaller workspace of a caller that knows only the older size takes the unordered path always
@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("n,K", [(1, 3), (15, 1), (63, 7), (1023, 5), (1024, 1), (1025, 40), (5000, 900), (3000, 20_000),
                                 (374, 1), (375, 1), (1058, 8), (1059, 8), (1500, 7), (6000, 40), (11_300, 900)])
def test_kmeans_update_with_and_without_room_for_the_order(d, n, K):
    print("[case]", d, n, K, flush=True)
    rng = np.random.default_rng(d + n + K)
    pool = rng.integers(-128, 128, (6, d))
    X = np.clip(pool[rng.integers(0, 6, n)] + rng.integers(-9, 10, (n, d)), -128, 127).astype(np.int8)
    C = rng.integers(-128, 128, (K, d)).astype(np.int8)
    C[: min(K, n)] = X[: min(K, n)]
    R = (rng.integers(0, 2, (8 * 4, d)) * 2 - 1).astype(np.int8)
    ix = dz.create(d, 8, 4, proj=torch.from_numpy(R).to(DEV))
    Xd = torch.from_numpy(X).to(DEV)
    want = orc.kmeans(X, C, 2)
    want = want[0] if isinstance(want, tuple) else want
    assert np.array_equal(dz.filter_kmeans(ix, Xd, torch.from_numpy(C).to(DEV), 2).cpu().numpy(), want)
    full = int(dz.lib().dessert_filter_kmeans_workspace_bytes(ix.handle, n, K))
    order = (n * 4 + 255) // 256 * 256
    cent = torch.from_numpy(C).to(DEV)
    ws = torch.empty(full - order, dtype=torch.uint8, device=DEV)
    assert dz.lib().dessert_filter_kmeans(ix.handle, Xd.data_ptr(), n, cent.data_ptr(), K, 2, ws.data_ptr(), ws.numel()) == dz.OK
    assert np.array_equal(cent.cpu().numpy(), want)


# Samples of 2^17 and more take two pieces per group of lanes, from 2^19 on four: runs that go on from piece to piece, groups whose later
# pieces lie past the sample's end, waves of which one group has work left; against the path that adds every coordinate by itself
@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("n,K", [(131_071, 3), (131_072, 90), (131_077, 1), (131_077, 5000), (524_287, 70), (524_365, 4), (524_365, 20_000)])
def test_kmeans_update_of_large_samples(d, n, K):
    print("[case]", d, n, K, flush=True)
    g = torch.Generator(device=DEV)
    g.manual_seed(d + n + K)
    ix = dz.create(d, 8, 4, seed=1)
    pool = torch.randint(-120, 121, (50, d), generator=g, device=DEV)
    X = (pool[torch.randint(0, 50, (n,), generator=g, device=DEV)] + torch.randint(-8, 9, (n, d), generator=g, device=DEV)).clamp(-128, 127).to(torch.int8)
    C = X[torch.randperm(n, generator=g, device=DEV)[:K]].contiguous()
    full = int(dz.lib().dessert_filter_kmeans_workspace_bytes(ix.handle, n, K))
    up = lambda x: (x + 255) // 256 * 256
    rows = (K + 31) // 32 * 32                          # the centroids' copies come in tiles of 32
    least = up(4 * n) + up(4 * K * d) + up(4 * K) + up(rows * d) + up(4 * rows)   # assignment, sums, counts, centroids, their constants
    order = up(4 * n)
    assert full >= least + order                        # and what assignments by groups take, where they are tried
    got = []
    for nbytes in (full, least + order - 256, least):   # with the order, without
        ws = torch.empty(nbytes, dtype=torch.uint8, device=DEV)
        cent = C.clone()
        assert dz.lib().dessert_filter_kmeans(ix.handle, X.data_ptr(), n, cent.data_ptr(), K, 1, ws.data_ptr(), nbytes) == dz.OK
        got.append(cent.cpu().numpy())
    assert np.array_equal(got[0], got[1]) and np.array_equal(got[0], got[2])
    # the rounded means from an assignment and sums of their own: values below 2^24, exact in fp32
    norm, Ct = (C.int() ** 2).sum(1), C.float().t().contiguous()
    sums, counts = torch.zeros(K, d, dtype=torch.int64, device=DEV), torch.zeros(K, dtype=torch.int64, device=DEV)
    for x in X.split(16384):
        value = 2 * (x.float() @ Ct).int() - norm
        first = torch.where(value == value.max(dim=1, keepdim=True).values, torch.arange(K, device=DEV, dtype=torch.int32), K).min(dim=1).values.long()
        sums.index_add_(0, first, x.long())
        counts.index_add_(0, first, torch.ones_like(first))
    some = counts.clamp(min=1)[:, None]
    means = torch.where(counts[:, None] > 0, (2 * sums + some).div(2 * some, rounding_mode="floor"), C.long())
    assert np.array_equal(got[0], means.to(torch.int8).cpu().numpy())
    # and of a few clusters, from the assignments of the oracle's definition
    if K <= 100:
        first = torch.arange(K, device=DEV)                                  # ties to the lower id
        near = lambda x: (128 * (2 * x @ C.double().T - (C.double() ** 2).sum(1)) - first).argmax(1)
        assign = torch.cat([near(x.double()) for x in X.split(16384)]).cpu().numpy()
        Xh = X.cpu().numpy().astype(np.int64)
        for c in range(min(K, 5)):
            mine = Xh[assign == c]
            want = (2 * mine.sum(0) + len(mine)) // (2 * len(mine)) if len(mine) else C[c].cpu().numpy()
            assert np.array_equal(got[0][c], want), c


# few vectors (up to 160 000, or 80 000 at d = 256): either side of a workgroup's 64 and 128 vectors and of the sizes that change the
# form; fewer centroid tiles than waves, one more than waves, many; centroids that repeat across waves (ties to the lower id); many
# vectors of few centroids, which take the general kernel
@pytest.mark.parametrize("d,n,K", [(64, 1, 1), (64, 63, 33), (64, 65, 520), (128, 64, 257), (128, 129, 4000), (256, 100, 300), (256, 1000, 31),
                                   (64, 32_769, 513), (128, 32_770, 700), (128, 160_000, 90), (128, 160_001, 90), (256, 80_001, 70),
                                   (128, 65_536, 100), (128, 65_537, 1535), (128, 65_537, 1536), (128, 160_000, 1601), (256, 49_152, 40),
                                   (256, 49_153, 1500), (256, 50_001, 1537)])
def test_closest_centroid_of_few_vectors(d, n, K):
    print("[case]", d, n, K, flush=True)
    rng = np.random.default_rng(n + K)
    lens = np.full((n + 6) // 7, 7)
    lens[-1] = n - 7 * (len(lens) - 1)
    ix, X = index(rng, lens, d=d)
    C = rng.integers(-127, 128, (K, d)).astype(np.int8)
    if K > 4:
        C[rng.integers(0, K, K // 2)] = C[K - 1]
        X[: n // 2] = C[K - 1]                                # their closest centroid stands in many tiles
        dz.build_index(ix, torch.from_numpy(X).to(DEV), lens)
    assign, _, _ = dz.filter_build(ix, torch.from_numpy(C).to(DEV), torch.from_numpy(X).to(DEV))
    got = assign.cpu().numpy().view(np.uint32)
    pick = np.unique(np.concatenate([np.arange(min(n, 200)), np.arange(max(0, n - 200), n), rng.integers(0, n, 1000)]))
    assert np.array_equal(got[pick], orc.assign_centroids(X[pick], C).astype(np.uint32))
