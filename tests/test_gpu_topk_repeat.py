"""Selections whose keys several waves sort in LDS, many times over and over many lists: every one is the exact order of its scores.  (A wave that
reads keys which another is still writing shows now and then only.)"""
import numpy as np
import pytest
import torch

import paper_2210_15748_amd as dz

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# lists of one slice, k keys in two waves; every document in several slices, and the merge of their results
@pytest.mark.parametrize("B,docs,cand,k,q", [(256, 20_000, 3000, 300, 8), (256, 20_000, 4096, 900, 8), (142, 60_286, 0, 172, 45), (40, 60_286, 0, 1000, 45)])
def test_repeated_selections(B, docs, cand, k, q):
    print("[case]", B, docs, cand, k, q, flush=True)
    g = torch.Generator(device=DEV)
    g.manual_seed(docs + k)
    ix = dz.create(64, 16, 4, seed=3)
    V = torch.randint(-127, 128, (docs, 64), generator=g, device=DEV, dtype=torch.int8)
    dz.build_index(ix, V, np.ones(docs, np.uint32))
    Q = torch.randint(-127, 128, (B * q, 64), generator=g, device=DEV, dtype=torch.int8)
    ql = np.full(B, q, np.uint32)
    lists = torch.stack([torch.randperm(docs, generator=g, device=DEV)[:cand] for _ in range(B)]).to(torch.int32) if cand else None
    scores = dz.scores(ix, Q, ql, cand_ids=lists).view(B, -1).long()
    ids = lists.long() if cand else torch.arange(docs, device=DEV)[None].expand(B, -1)
    best = torch.sort(scores * 2 ** 32 + (2 ** 32 - 1 - ids), dim=1, descending=True).values[:, :k]
    want_scores, want_ids = best >> 32, 2 ** 32 - 1 - (best & (2 ** 32 - 1))
    for _ in range(30):
        got_ids, got_scores = dz.search(ix, Q, ql, k, cand_ids=lists)
        assert torch.equal(got_scores.long(), want_scores)
        assert torch.equal(got_ids.view(torch.int32).long() & 0xFFFFFFFF, want_ids)
