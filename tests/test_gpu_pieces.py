"""How the attention kernels cut their work into pieces: trailing entries that a
query tile cannot see, and masked pages, at the edges of the kernels' windows."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_16839_amd as ca
import synth
from _helpers import (bf16_host_f64, compare_attention, device_inputs, i32_dev, rows_by_head,
                      tile_rows)

pytestmark = pytest.mark.gpu


def _inputs(cached, chunk, heads=(4, 1), dim=64, seed=31, max_kv_blocks=None):
    nkb = max(-(-(c + chunk) // 64) for c in cached)
    w = synth.Workload(name="pieces", seed=seed, batch=len(cached), num_q_heads=heads[0],
                       num_kv_heads=heads[1], head_dim=dim, q_block=64, chunk_len=chunk,
                       cached_lens=tuple(cached), max_kv_blocks=max_kv_blocks or nkb,
                       sm_scale=dim ** -0.5, poison_tail=True)
    return w, synth.make_inputs(w)


def _tables(w, density, seed, chunk_open=True):
    """Random cached blocks per (b, group) row; every chunk block, or a random
    part of the chunk's blocks too (chunk_open = False)."""
    rng = np.random.default_rng(seed)
    rows = []
    for b in range(w.batch):
        nc, nkb = w.n_cached_blocks(b), w.n_kv_blocks(b)
        for _ in range(w.num_groups):
            keep = rng.random(nkb) < density
            if chunk_open:
                keep[nc:] = True
            rows.append(np.flatnonzero(keep))
    ip = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32)
    ix = np.zeros(len(rows) * w.max_kv_blocks, dtype=np.int32)
    ix[:ip[-1]] = np.concatenate(rows)
    return rows, ip, ix


def _check(w, d, rows_of, gs, out, lse, per_tile=2, every=1):
    rows = tile_rows(w.batch, w.num_q_heads, w.chunk_len, gs, seed=w.seed, per_tile=per_tile)
    rows = rows[::every]
    G = w.num_q_heads // gs
    tab = [[rows_of[b * G + g] for g in range(G)] for b in range(w.batch)]
    ref = np.full((w.batch, w.chunk_len, w.num_q_heads, w.head_dim), np.nan)
    ref_lse = np.full((w.batch, w.num_q_heads, w.chunk_len), np.nan)
    for (b, h), ts in rows_by_head(rows).items():
        o, l = oracle.chunk_attention(d["q"], d["k_pool"], d["v_pool"], d["page_table"],
                                      d["cached_len"], tab, gs, w.sm_scale, heads=[(b, h)],
                                      queries=ts)
        ref[b, ts, h], ref_lse[b, h, ts] = o[b, ts, h], l[b, h, ts]
    compare_attention(bf16_host_f64(out), lse.cpu().numpy().astype(np.float64), ref, ref_lse,
                      rows=rows)


@pytest.mark.parametrize("chunk_open", [True, False])
def test_trailing_entries_past_one_window(chunk_open):
    """A chunk of 71 blocks: the first tiles see none of the last 64 entries, so
    the visible and the masked counts come from more than one 64-entry window."""
    w, d = _inputs((130,), 4500)
    x = device_inputs(d)
    rows, ip, ix = _tables(w, 0.7, 5, chunk_open)
    p = ca.Problem.from_workload(w)
    lse = torch.empty((1, 4, w.chunk_len), dtype=torch.float32, device="cuda")
    out, _ = ca.chunk_attention(p, x["q"], (x["k"], x["v"]), x["pt"], (i32_dev(ip), i32_dev(ix)),
                                4, w.sm_scale, num_splits=1, lse=lse)
    _check(w, d, rows, 4, out, lse)

