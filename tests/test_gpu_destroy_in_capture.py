"""A handle that is dropped while another one's search is captured (as a garbage collection may do) leaves the capture alone."""
import gc

import numpy as np
import pytest
import torch

import paper_2210_15748_amd as dz

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("own_stream", [False, True])   # the dropped handle's: the default stream or one of its own
def test_dropping_a_handle_leaves_a_capture_alone(own_stream):
    print("[case] a handle dropped during a capture", own_stream, flush=True)
    d, n, B, q, k = 128, 500, 4, 8, 10
    g = torch.Generator(device=DEV)
    g.manual_seed(2)
    X = torch.randint(-127, 128, (n, d), generator=g, device=DEV, dtype=torch.int8)
    Q = torch.randint(-127, 128, (B * q, d), generator=g, device=DEV, dtype=torch.int8)
    lens, ql = np.ones(n, np.uint32), np.full(B, q, np.uint32)
    other = torch.cuda.Stream(device=DEV) if own_stream else torch.cuda.default_stream()
    other.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(other):
        dropped = dz.create(d, 32, 7, seed=1, stream=other)
        dz.build_index(dropped, X, lens)                  # buffers, events and a copy stream of its own
        dz.enable_timing(dropped, 1)
        dz.search(dropped, Q, ql, k)
    torch.cuda.synchronize()
    side = torch.cuda.Stream(device=DEV)
    with torch.cuda.stream(side):
        ix = dz.create(d, 32, 7, seed=1, stream=side)
        dz.build_index(ix, X, lens)
        ws = torch.empty(1 << 20, dtype=torch.uint8, device=DEV)
        out_i = torch.empty(B, k, dtype=torch.uint32, device=DEV)
        out_s = torch.empty(B, k, dtype=torch.int32, device=DEV)
        want_i, want_s = dz.search(ix, Q, ql, k)
    side.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        dz.destroy(dropped)
        del dropped
        gc.collect()
        dz.search(ix, Q, ql, k, workspace=ws, out_ids=out_i, out_scores=out_s)
    for _ in range(3):
        out_i.view(torch.int32).fill_(-1)
        out_s.fill_(-1)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out_i.view(torch.int32), want_i.view(torch.int32)) and torch.equal(out_s, want_s)
        dz.search(ix, Q, ql, k)
        torch.cuda.synchronize()
