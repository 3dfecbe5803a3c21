"""NaN and infinite scores reach the output whatever launch runs the chunk: a query
with a score of NaN or +inf gets out = NaN and lse = -inf, and no other query is
touched (a score of -inf is a weight of 0)."""
import numpy as np
import pytest
import torch

import paper_2605_16839_amd as ca
import synth
from _helpers import device_inputs, i32_dev

pytestmark = pytest.mark.gpu

# cached, chunk, heads, dim, group, num_splits
LAUNCHES = [
    ((9000,), 300, (8, 2), 64, 4, 1),
    ((9000,), 300, (8, 2), 128, 4, 2),          # merge of two uniform pieces
    ((9000,), 300, (8, 2), 64, 4, 5),           # all pieces in flight
    ((9000,), 300, (8, 2), 128, 4, 12),         # more pieces than that
    ((40000,), 37, (32, 8), 128, 4, 0),         # equal shares, four waves to a fragment
    ((20000,), 300, (32, 8), 64, 4, 0),         # equal shares, one wave
    ((30000,), 2048, (32, 8), 64, 4, 0),        # two pieces per row, balanced over the XCDs
]


@pytest.mark.parametrize("kind", ["nan", "inf"])
@pytest.mark.parametrize("cached,chunk,heads,dim,group,splits", LAUNCHES)
def test_reaches_the_output(cached, chunk, heads, dim, group, splits, kind):
    nkb = max(-(-(c + chunk) // 64) for c in cached)
    w = synth.Workload(name="nan", seed=3, batch=len(cached), num_q_heads=heads[0],
                       num_kv_heads=heads[1], head_dim=dim, q_block=64, chunk_len=chunk,
                       cached_lens=tuple(cached), max_kv_blocks=nkb, sm_scale=dim ** -0.5)
    d = synth.make_inputs(w)
    x = device_inputs(d)
    p = ca.Problem.from_workload(w)
    G = heads[0] // group
    # block 3 of KV head 0 of sequence 0 holds the key; row 0 lists every block, the
    # others fewer (rows of one length are not cut for the XCDs)
    kept = [np.arange(w.n_kv_blocks(b)) for b in range(w.batch) for _ in range(G)]
    kept[1:] = [r[(r % 5 != 1) | (r >= len(r) - 48)] for r in kept[1:]]
    ip = np.concatenate([[0], np.cumsum([len(r) for r in kept])]).astype(np.int32)
    ix = np.zeros(len(kept) * nkb, dtype=np.int32)
    ix[:ip[-1]] = np.concatenate(kept)
    k = x["k"].clone()
    page = int(d["page_table"][0, 0, 3])
    if kind == "nan":
        k[page, 17, 5] = float("nan")
    else:   # the score is +inf, or -inf where q_0 is negative
        k[page, 17] = 0.0
        k[page, 17, 0] = float("inf")
    ws = torch.empty(max(16, ca.attention_workspace_bytes(p, group, splits)), dtype=torch.uint8,
                     device="cuda")
    lse = torch.full((w.batch, heads[0], chunk), 7.0, device="cuda")
    out, _ = ca.chunk_attention(p, x["q"], (k, x["v"]), x["pt"], (i32_dev(ip), i32_dev(ix)),
                                group, w.sm_scale, num_splits=splits, lse=lse, ws=ws)
    hit = torch.zeros((w.batch, chunk, heads[0]), dtype=torch.bool, device="cuda")
    own = heads[0] // heads[1]      # the query heads of KV head 0
    hit[0, :, :own] = True if kind == "nan" else ~(x["q"][0, :, :own, 0] < 0)
    assert hit.any() and not hit.all()
    assert torch.equal(torch.isnan(out).all(-1), hit)
    assert torch.equal(torch.isnan(out).any(-1), hit)
    assert torch.equal(torch.isneginf(lse).transpose(1, 2), hit)
    assert torch.isfinite(lse.transpose(1, 2)[~hit]).all()
