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


# Launches that share their pages equally among the CUs, around the edges of the
# schedule: one query tile (32 segments per slab) to 31 tiles (one segment and a
# remainder on one CU), one table row, rows of very different lengths, selected and
# dense tables of both head sizes and V layouts.  (test_launch_choice.py checks that
# the sizes of each list take the launch it names.)
SHARES = [
    # cached, chunk, heads, dim, group, layout, density (None = dense)
    ((40000,), 37, (32, 8), 64, 4, 0, 0.3),
    ((40000,), 1, (32, 8), 128, 4, 1, 0.3),
    ((20000,), 300, (32, 8), 128, 4, 0, 0.4),
    ((9000,), 700, (32, 8), 64, 4, 1, 0.5),
    ((7001,), 1451, (16, 4), 128, 4, 0, 0.6),
    ((9000,), 1984, (16, 4), 128, 4, 1, 0.6),
    ((9000, 37, 30000), 200, (32, 8), 64, 4, 0, 0.4),
    ((6000,), 700, (16, 8), 128, 2, 0, 0.4),
    ((30000,), 999, (4, 1), 64, 4, 0, 0.9),
    ((100, 3000, 0), 777, (16, 4), 128, 4, 0, None),
    ((16384,), 64, (32, 8), 128, 4, 1, None),
    ((8192,), 1200, (32, 8), 64, 4, 0, None),
    ((6000,), 700, (16, 4), 64, 4, 1, None),
    ((20000,), 300, (4, 1), 64, 4, 1, None),
]
# Uniform splits, some of more pieces than the merge holds at once.
UNIFORM = [
    ((6000, 12000), 500, (8, 1), 64, 8, 1, 0.5),
    ((9000,), 512, (32, 8), 64, 4, 1, 0.5),
    ((9000,), 999, (16, 4), 64, 4, 0, None),
    ((30000,), 300, (4, 1), 64, 4, 0, 0.4),
]


@pytest.mark.parametrize("cached,chunk,heads,dim,group,layout,density", SHARES)
def test_equal_shares_match_oracle(cached, chunk, heads, dim, group, layout, density):
    _matches_oracle(cached, chunk, heads, dim, group, layout, density)


@pytest.mark.parametrize("cached,chunk,heads,dim,group,layout,density", UNIFORM)
def test_uniform_splits_match_oracle(cached, chunk, heads, dim, group, layout, density):
    _matches_oracle(cached, chunk, heads, dim, group, layout, density)


@pytest.mark.parametrize("short", [1, 16])
def test_equal_shares_without_their_workspace(short):
    """A workspace too small for the equal shares by a byte, or by its alignment:
    another launch, the same result."""
    _matches_oracle(*SHARES[2], short=short)


def _matches_oracle(cached, chunk, heads, dim, group, layout, density, short=0):
    w, d = _inputs(cached, chunk, heads, dim)
    w = synth.configs.replace(w, group_size=group)
    x = device_inputs(d, layout)
    p = ca.Problem.from_workload(w, v_layout=layout)
    q, kv = x["q"], (x["k"], x["v"])
    rows, ip, ix = _tables(w, 2.0 if density is None else density, 7)
    tables = (i32_dev(ip), i32_dev(ix))
    n = ca.attention_workspace_bytes(p, group, 0)
    lse = torch.empty((w.batch, heads[0], chunk), dtype=torch.float32, device="cuda")

    def run(fill):
        size = max(n - short, 16)
        guarded = torch.full((size + 4096,), fill, dtype=torch.uint8, device="cuda")
        ws = guarded[:size]
        lse.fill_(float("nan"))
        out = torch.full_like(q, float("nan"))
        if density is None:
            ca.dense_paged_chunk_attention(p, q, kv, x["pt"], w.sm_scale, out=out, lse=lse, ws=ws)
        else:
            ca.chunk_attention(p, q, kv, x["pt"], tables, group, w.sm_scale, out=out, lse=lse,
                               ws=ws)
            # the same tables through packed pools
            packed = ca.gather_selected_pages(p, kv, x["pt"], tables, group)
            out2, _ = ca.packed_chunk_attention(p, q, packed, tables, group, w.sm_scale, ws=ws)
            assert torch.equal(out.view(torch.int16), out2.view(torch.int16))
        assert (guarded[size:] == fill).all()     # nothing past the workspace
        return out, lse.clone()

    out, l0 = run(0)
    again, l1 = run(255)     # whatever the workspace held
    assert torch.equal(out.view(torch.int16), again.view(torch.int16)) and torch.equal(l0, l1)
    _check(w, d, rows, group, out, l0, per_tile=2, every=1 if w.batch == 1 else 2)


@pytest.mark.parametrize("chunk", [100, 1300])
def test_equal_shares_sparse_rows(chunk):
    """Tables that leave out chunk blocks, list one block, or list none: every
    output is written (0 and -inf for a query that sees no key)."""
    w, d = _inputs((30000, 8000), chunk, (32, 8))
    x = device_inputs(d)
    p = ca.Problem.from_workload(w)
    rows, _, _ = _tables(w, 0.5, 11, chunk_open=False)
    rows[1], rows[2] = rows[1][:0], rows[2][:1]
    rows[9], rows[15] = rows[9][-1:], rows[15][:0]
    ip = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32)
    ix = np.zeros(len(rows) * w.max_kv_blocks, dtype=np.int32)
    ix[:ip[-1]] = np.concatenate(rows)
    lse = torch.full((2, 32, chunk), float("nan"), device="cuda")
    out = torch.full_like(x["q"], float("nan"))
    ca.chunk_attention(p, x["q"], (x["k"], x["v"]), x["pt"], (i32_dev(ip), i32_dev(ix)), 4,
                       w.sm_scale, out=out, lse=lse)
    _check(w, d, rows, 4, out, lse, every=2)


# Half tiles (128 rows per workgroup): one query up to more tiles than fit the GPU
# at once, partial tiles, group sizes that change the queries per tile, rows that do
# not spread over the XCDs evenly, unaligned lengths, selected and packed tables.
HALF = [
    # cached, chunk, heads, dim, group, layout, density (None = dense)
    ((0,), 2048, (32, 8), 128, 4, 0, None),
    ((0, 500), 1000, (32, 8), 64, 4, 1, None),
    ((3000,), 1024, (32, 8), 64, 4, 1, 0.5),
    ((7001,), 1451, (32, 8), 128, 4, 0, 0.6),
    ((0,), 1, (4, 1), 64, 4, 0, None),
    ((0,), 64, (32, 8), 128, 4, 0, None),
    ((0,), 97, (32, 8), 128, 4, 1, None),
    ((37,), 512, (32, 8), 128, 4, 0, None),
    ((0, 0), 700, (32, 8), 64, 4, 1, None),
    ((100, 0, 300), 333, (12, 3), 128, 4, 0, None),
    ((0,), 2048, (32, 8), 64, 4, 0, None),
    ((0,), 300, (16, 2), 64, 8, 1, None),
    ((500,), 400, (16, 8), 128, 2, 0, 0.5),
    ((64,), 129, (8, 8), 64, 1, 0, 0.5),
    ((3000,), 2048, (32, 8), 64, 4, 0, 0.4),
    ((700, 2100), 2048, (32, 8), 128, 4, 1, 0.3),
]


@pytest.mark.parametrize("cached,chunk,heads,dim,group,layout,density", HALF)
def test_half_tiles_match_oracle(cached, chunk, heads, dim, group, layout, density):
    _matches_oracle(cached, chunk, heads, dim, group, layout, density)


# cached, chunk: short rows, and whole tiles that fill the GPU
SPARSE_HALF = [((900,), 600), ((3000,), 2048)]


@pytest.mark.parametrize("cached,chunk", SPARSE_HALF)
def test_half_tiles_sparse_rows(cached, chunk):
    """Rows that leave out chunk blocks or list nothing; no workspace at all."""
    w, d = _inputs(cached, chunk, (32, 8))
    x = device_inputs(d)
    p = ca.Problem.from_workload(w)
    rows, _, _ = _tables(w, 0.5, 13, chunk_open=False)
    rows[1], rows[2], rows[3] = rows[1][:0], rows[2][:1], rows[3][-1:]
    ip = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32)
    ix = np.zeros(len(rows) * w.max_kv_blocks, dtype=np.int32)
    ix[:ip[-1]] = np.concatenate(rows)
    lse = torch.full((1, 32, chunk), float("nan"), device="cuda")
    out = torch.full_like(x["q"], float("nan"))
    ip_dev, ix_dev = i32_dev(ip), i32_dev(ix)
    st = ca.load().ca_chunk_attention(
        p.ref, x["q"].data_ptr(), x["k"].data_ptr(), x["v"].data_ptr(), x["pt"].data_ptr(),
        ip_dev.data_ptr(), ix_dev.data_ptr(), 4, w.sm_scale, 0, out.data_ptr(),
        lse.data_ptr(), None, 0, torch.cuda.current_stream().cuda_stream)
    assert st == 0
    _check(w, d, rows, 4, out, lse)
