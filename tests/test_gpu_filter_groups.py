"""Assignment by groups of centroids (large filter_build and filter_kmeans calls): the same closest centroid, bit for bit, as comparing every
vector with every centroid, whatever the data look like; ties go to the lower centroid id."""
import math

import pytest
import torch

import paper_2210_15748_amd as dz

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def say(*a):
    print(*a, flush=True)


def vectors(n, d, centres, g, spread=0.3):
    v = torch.randn(n, d, generator=g, device=DEV)
    if centres is not None:
        v = centres[torch.randint(0, centres.shape[0], (n,), generator=g, device=DEV)] + spread / math.sqrt(d) * v
    v = v / v.norm(dim=1, keepdim=True)
    return (v * 127).round_().clamp_(-127, 127).to(torch.int8)


def closest(X, C):
    """argmin |x - c|^2, lowest id among equals.  Sums of products of int8 values stay below 2^24: exact in fp32 in any order."""
    Ct, norm = C.float().t().contiguous(), (C.int() ** 2).sum(1)
    ids = torch.arange(C.shape[0], device=DEV, dtype=torch.int32)
    out = torch.empty(X.shape[0], dtype=torch.int32, device=DEV)
    for lo in range(0, X.shape[0], 8192):
        value = 2 * (X[lo:lo + 8192].float() @ Ct).int() - norm[None, :]
        best = value.max(dim=1, keepdim=True).values
        out[lo:lo + 8192] = torch.where(value == best, ids[None, :], C.shape[0]).min(dim=1).values
    return out


def handle(d, n):
    ix = dz.create(d, 8, 4, proj=torch.ones(32, d, dtype=torch.int8, device=DEV))
    lens = [64] * (n // 64) + ([n % 64] if n % 64 else [])
    codes = torch.zeros(n, 8, dtype=torch.uint8, device=DEV)
    off = torch.zeros(len(lens) + 1, dtype=torch.int64, device=DEV)
    off[1:] = torch.cumsum(torch.tensor(lens, device=DEV), 0)
    dz.attach_index(ix, codes, off, 64)
    return ix


# clusters: most vectors need one group.  partly: 45 % of the vectors lie where no centroid does, a list long enough for the kernel for
# many vectors.  all directions / one point: groups are of no use (too near to each other; one group of everything).  wide: groups around
# centroids that are their own only members, next to a few large ones; duplicates: equal centroids, in and out of order.
KINDS = ["clusters", "partly", "all directions", "one point", "wide", "duplicates"]


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("d,K,n", [(128, 8192, 170_000), (64, 8223, 320_003), (256, 8200, 82_001), (128, 16_385, 200_000)])
def test_assignment_by_groups(kind, d, K, n):
    say(f"assignment by groups: {kind} d={d} K={K} n={n}")
    g = torch.Generator(device=DEV)
    g.manual_seed(1000 * KINDS.index(kind) + d + K)
    centres = torch.randn(700, d, generator=g, device=DEV) / math.sqrt(d)
    X = vectors(n, d, None if kind == "all directions" else centres, g)
    pick = torch.randint(0, n, (K,), generator=g, device=DEV)
    C = X[pick].clone()
    if kind == "partly":
        X[: int(0.45 * n)] = vectors(int(0.45 * n), d, torch.randn(900, d, generator=g, device=DEV) / math.sqrt(d), g)
        X = X[torch.randperm(n, generator=g, device=DEV)].contiguous()
    elif kind == "one point":
        C[:] = C[0]
        C[K // 2] = X[5]
    elif kind == "wide":
        C[K // 2:] = vectors(K - K // 2, d, centres[:5], g, spread=0.6)
        C[: K // 16] = vectors(K // 16, d, None, g)
    elif kind == "duplicates":
        C[K // 2:] = C[torch.randint(0, K // 2, (K - K // 2,), generator=g, device=DEV)]
    ix = handle(d, n)
    assign, starts, docs = dz.filter_build(ix, C, X)
    want = closest(X, C)
    assert torch.equal(assign, want), f"{int((assign != want).sum())} of {n} vectors"
    # the buckets are made from it, over the array that held the list of vectors left over
    pairs = torch.unique(assign.long() * (n // 64 + 1) + torch.arange(n, device=DEV) // 64)
    assert torch.equal(torch.bincount(pairs // (n // 64 + 1), minlength=K), starts[1:].long() - starts[:-1].long())
    total = int(starts[-1])
    got = torch.repeat_interleave(torch.arange(K, device=DEV), starts[1:].long() - starts[:-1].long()) * (n // 64 + 1) + docs[:total].long()
    assert torch.equal(torch.sort(got).values, pairs)


def without_groups(n, d, K):
    """Bytes of a k-means workspace before the scratch for groups: assignment, sums, counts, the centroids' copies in tiles of 32 with their
    constants, the vectors' order."""
    up, rows = lambda x: (x + 255) // 256 * 256, (K + 31) // 32 * 32
    return up(4 * n) + up(4 * K * d) + up(4 * K) + up(rows * d) + up(4 * rows) + up(4 * n)


# What the launches decided stands at the start of the scratch: groups, radius, the trial's vectors that needed one group of 4096, the members of
# those, vectors left over.  partly: as above, one round only (the centroids move to the vectors), enough left over for the kernel for many vectors
# at d = 64 and 128.  all directions: one group of everything, or too many
@pytest.mark.parametrize("kind,rounds", [("clusters", 1), ("clusters", 3), ("partly", 1), ("all directions", 1)])
@pytest.mark.parametrize("d,K,n", [(128, 8192, 170_000), (64, 8223, 320_003), (256, 8200, 82_001)])
def test_kmeans_with_and_without_room_for_groups(d, K, n, kind, rounds):
    say(f"k-means by groups: {kind} {rounds} d={d} K={K} n={n}")
    g = torch.Generator(device=DEV)
    g.manual_seed(d + K)
    X = vectors(n, d, None if kind == "all directions" else torch.randn(500, d, generator=g, device=DEV) / math.sqrt(d), g)
    start = X[torch.randint(0, n, (K,), generator=g, device=DEV)].contiguous()
    if kind == "partly":
        X[: int(0.45 * n)] = vectors(int(0.45 * n), d, torch.randn(900, d, generator=g, device=DEV) / math.sqrt(d), g)
        X = X[torch.randperm(n, generator=g, device=DEV)].contiguous()
    ix = handle(d, 64)
    full, before = int(dz.lib().dessert_filter_kmeans_workspace_bytes(ix.handle, n, K)), without_groups(n, d, K)
    assert full >= before + K * d + K // 3 * d, "the workspace has no room for groups: these sizes do not reach them"
    got = []
    for nbytes in (full, full - 256):   # a workspace without room for the groups is accepted
        ws = torch.empty(full, dtype=torch.uint8, device=DEV)
        cent = start.clone()
        assert dz.lib().dessert_filter_kmeans(ix.handle, X.data_ptr(), n, cent.data_ptr(), K, rounds, ws.data_ptr(), nbytes) == dz.OK
        got.append(cent)
        if nbytes == full:
            groups, _, easy, members, rest = ws[before:before + 20].view(torch.int32).tolist()
            say("decided:", groups, easy, members, rest)
    assert torch.equal(got[0], got[1])
    if kind == "clusters":
        assert 100 < groups <= K // 3 and easy > 3000 and easy <= members < 4096 * (K // 75) and rest < 65536 and rest < n // 4
    elif kind == "partly":
        assert 100 < groups <= K // 3 and easy > 1500 and 0.4 * n < rest < 0.6 * n and (rest > 65536) == (d < 256)
    else:
        assert rest == 0 and (easy == 0 or groups > K // 3)


# Many centroids that lead only themselves: some look for their leaders first, from 32 768 centroids on.  Vectors lie close to centroids, so that the
# groups are narrow; apart: all centroids alone, half: every other one beside the one before; no groups are made then.  few: one in four alone
@pytest.mark.parametrize("kind", ["apart", "half", "few"])
@pytest.mark.parametrize("d,K,n", [(64, 40_003, 320_100), (256, 32_768, 262_200)])
def test_assignment_where_centroids_lead_themselves(kind, d, K, n):
    say(f"centroids that lead themselves: {kind} d={d} K={K} n={n}")
    g = torch.Generator(device=DEV)
    g.manual_seed(d + K)
    C = vectors(K, d, None, g)
    step = {"apart": 1, "half": 2, "few": 4}[kind]
    base = C[torch.arange(K, device=DEV) // step * step].int()
    C = (base + torch.randint(-1, 2, (K, d), generator=g, device=DEV)).clamp(-127, 127).to(torch.int8)
    X = (C[torch.randint(0, K, (n,), generator=g, device=DEV)].int() + torch.randint(-2, 3, (n, d), generator=g, device=DEV)).clamp(-127, 127).to(torch.int8)
    assign, _, _ = dz.filter_build(handle(d, n), C, X)
    want = closest(X, C)
    assert torch.equal(assign, want), f"{int((assign != want).sum())} of {n} vectors"


# Rounds of k-means after one whose groups did not pay: of every eight only the first two try in any case
@pytest.mark.parametrize("clusters", [0, 20, 500])
@pytest.mark.parametrize("d,K,n", [(128, 8192, 170_000), (256, 8200, 82_001)])
def test_rounds_of_kmeans_with_and_without_room_for_groups(clusters, d, K, n):
    say(f"rounds of k-means by groups: clusters={clusters} d={d} K={K} n={n}")
    g = torch.Generator(device=DEV)
    g.manual_seed(d + K + clusters)
    X = vectors(n, d, torch.randn(clusters, d, generator=g, device=DEV) / math.sqrt(d) if clusters else None, g)
    start = X[torch.randint(0, n, (K,), generator=g, device=DEV)].contiguous()
    ix = handle(d, 64)
    full = int(dz.lib().dessert_filter_kmeans_workspace_bytes(ix.handle, n, K))
    got = []
    for nbytes in (full, full - 256):
        ws = torch.randint(0, 256, (full,), generator=g, device=DEV, dtype=torch.uint8)   # what it holds from before does not matter
        cent = start.clone()
        assert dz.lib().dessert_filter_kmeans(ix.handle, X.data_ptr(), n, cent.data_ptr(), K, 10, ws.data_ptr(), nbytes) == dz.OK
        got.append(cent)
    assert torch.equal(got[0], got[1])
