"""Device memory that a handle holds for its filter: scratch for assignments by groups of centroids only where a build takes that way."""
import pytest
import torch

import paper_2210_15748_amd as dz

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def test_scratch_is_held_only_where_it_is_used():
    print("[case] filter scratch", flush=True)
    d, K = 256, 40_960
    g = torch.Generator(device=DEV)
    g.manual_seed(1)
    most = 8 * K                                            # the first number of vectors that goes by groups
    X = torch.randint(-127, 128, (most, d), generator=g, device=DEV, dtype=torch.int8)
    C = X[:K].contiguous()
    codes = torch.zeros(most, 8, dtype=torch.uint8, device=DEV)
    assign, docs = (torch.empty(most, dtype=torch.int32, device=DEV) for _ in range(2))
    starts = torch.empty(K + 1, dtype=torch.int32, device=DEV)
    ix = dz.create(d, 8, 4, seed=1)

    few = most - 64
    offsets = {n: torch.arange(0, n + 1, 64, device=DEV, dtype=torch.int64) for n in (few, most)}   # the same id ranges for both sizes
    kept = [torch.empty(most, dtype=torch.int32, device=DEV) for _ in range(4)]

    def build(n, out):
        dz.attach_index(ix, codes[:n], offsets[n], 64)
        assert dz.lib().dessert_filter_build(ix.handle, C.data_ptr(), K, X.data_ptr(), assign.data_ptr(), starts.data_ptr(), docs.data_ptr()) == dz.OK
        out.copy_(assign)
        torch.cuda.synchronize()

    warm = dz.create(d, 8, 4, seed=1)                       # what the first call of a process takes for itself
    dz.attach_index(warm, codes[:64], torch.arange(0, 65, 64, device=DEV), 64)
    dz.filter_build(warm, C[:64].contiguous(), X[:64])
    torch.cuda.synchronize()
    at = [torch.cuda.mem_get_info()[0]]
    for n, out in zip((few, most, few, most), kept):        # torch allocates nothing in here
        build(n, out)
        at.append(torch.cuda.mem_get_info()[0])
    held = [at[0] - x for x in at[1:]]
    centroids = K * d
    assert centroids <= held[0] < 1.9 * centroids           # the copy in another order, tables, sub-bucket counters
    assert held[1] - held[0] > 1.2 * centroids              # rows by groups, leaders
    # given back and taken again; the runtime takes and keeps 2 MiB blocks of its own for small allocations and the ends of large ones
    assert abs(held[2] - held[0]) <= 2 << 20 and abs(held[3] - held[1]) <= 2 << 20
    assert torch.equal(kept[0][:few], kept[1][:few]) and torch.equal(kept[0][:few], kept[2][:few]) and torch.equal(kept[1], kept[3])
