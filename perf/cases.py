"""The work that a program asks of this package, as cases that can be timed and compared.

A program prefills long prompts chunk by chunk.  For every chunk of every
layer it selects KV blocks (``estimate_masks`` or its threshold form), merges
the masks into one block table per execution group (``build_block_tables``, or
both at once with ``estimate_tables``) and attends over the listed pages
(``chunk_attention``); short contexts go through
``dense_paged_chunk_attention``.  It keeps its page pools, page table, block
means, output buffers and workspaces from chunk to chunk, so ``prepare`` makes
them and ``run`` is the calls alone.

Kinds of cases:
  step       estimate_masks -> build_block_tables -> chunk_attention, nothing
             carried over between chunks (every cached block is pooled)
  fused      estimate_tables -> chunk_attention with the block means carried
             over: only the blocks the previous chunk completed are pooled
  attention  chunk_attention over given tables
  dense      dense_paged_chunk_attention
  estimate   estimate_masks alone
  threshold  estimate_masks_threshold with the block means carried over
  tables     build_block_tables alone
"""
import math

import torch

import paper_2605_16839_amd as ca

PAGE = 64
DEVICE = "cuda"
RHO = 0.12          # weight of the query direction shared by one KV group's heads
SINK, LOCAL = 1, 4  # the selector's defaults
ALPHA, TEMPERATURE = 0.06, 4.0   # the threshold selector


def _case(name, kind, cached, chunk, heads=(32, 8), dim=128, group=4, q_block=128,
          layout="token_major", top=0.05, density=0.3, table_blocks=0):
    c = dict(kind=kind, cached=cached, chunk=chunk, q_heads=heads[0], kv_heads=heads[1], dim=dim,
             group=group, q_block=q_block, layout=layout, top=top, density=density,
             table_blocks=table_blocks)
    return dict(name=name, **c) if name else c


def listed():
    return [
        # the smallest call: a short chunk of a small model (one KV head of 64
        # dimensions), all three stages; launches and host calls count
        _case("step_small", "step", "1024", 256, (4, 1), 64, 4, 64, top=0.25),
        # the ragged end of a prompt: the last few tokens after 64K cached
        _case("fused_tail", "fused", "65536", 37, layout="transposed", top=0.08),
        # a 512-token chunk (the smallest chunk size serving systems use) near
        # the end of a 128K prompt, block means carried over
        _case("fused_chunk512", "fused", "129024", 512, top=0.05, table_blocks=2048),
        # the whole step on the last 2048-token chunk of a 128K prompt
        _case("step_chunk2048", "step", "129024", 2048, layout="transposed", top=0.05),
        # 64-dimensional heads, two sequences of different lengths
        _case("attention_dim64", "attention", "30720,12345", 1024, (32, 8), 64, 4, 64,
              density=0.35),
        # four sequences of very different lengths in one pool: the largest call
        _case("attention_batched", "attention", "16384,32768,65536,126976", 2048,
              layout="transposed", density=0.3),
        # a prompt's remainder: neither the cache nor the chunk is a multiple
        # of a block, and the chunk does not fill the GPU evenly
        _case("attention_ragged", "attention", "50001", 1451, density=0.3),
        # grouped queries of 8 heads per KV head, tables for sub-groups of 4
        _case("attention_subgroups", "attention", "129024", 1024, (32, 4), 128, 4,
              layout="transposed", density=0.35),
        # the first chunks of a prompt: too short to select, so dense; one
        # sequence at its very start, one a chunk further
        _case("dense_first_chunk", "dense", "0", 2048),
        # selection over four ragged sequences, everything pooled
        _case("estimate_batched", "estimate", "16384,32768,65536,100001", 2048, q_block=64,
              top=0.08),
        # the threshold selector late in a long prompt, block means carried over
        _case("threshold_long", "threshold", "100001", 1024),
        # tables for four sequences from given masks
        _case("tables_batched", "tables", "16384,32768,65536,126976", 2048, density=0.02),
    ]


# No drawn case costs more than the largest listed one.
_MOST_FLOPS = 4.4e12
_MOST_BYTES = 1.6e9


def draw(rng):
    def spread(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    while True:
        kind = rng.choice(["step", "fused", "attention", "attention", "dense", "estimate",
                           "threshold", "tables"])
        batch = rng.choice([1, 1, 1, 2, 3, 4])
        heads, dim = rng.choice([((4, 1), 64), ((8, 2), 64), ((32, 8), 64), ((32, 8), 128),
                                 ((32, 8), 128), ((32, 8), 128), ((32, 4), 128)])
        lens = [spread(500, 129024) for _ in range(batch)]
        if kind == "dense":
            lens = [spread(64, 16384) - 64 for _ in range(batch)]
        chunk = spread(32, 2048)
        if rng.random() < 0.4:      # block-aligned, as most schedulers keep them
            lens = [n // PAGE * PAGE for n in lens]
            chunk = -(-chunk // PAGE) * PAGE
        c = _case(None, kind, ",".join(str(n) for n in lens), chunk, heads, dim, 4,
                  rng.choice([64, 128]), rng.choice(["token_major", "transposed"]),
                  round(rng.uniform(0.03, 0.12), 3),
                  round(rng.uniform(0.005, 0.04) if kind == "tables" else rng.uniform(0.2, 0.5),
                        3))
        w = work(c)
        if w["flops"] <= _MOST_FLOPS and w["bytes"] <= _MOST_BYTES:
            return c


# ---------------------------------------------------------------------------
# sizes
# ---------------------------------------------------------------------------
class _Sizes:
    def __init__(self, c):
        self.lens = [int(n) for n in c["cached"].split(",")]
        self.B, self.C, self.D = len(self.lens), c["chunk"], c["dim"]
        self.Hq, self.Hkv, self.gs = c["q_heads"], c["kv_heads"], c["group"]
        self.G = self.Hq // self.gs
        self.ratio = self.Hq // self.Hkv
        self.qb = c["q_block"]
        self.nqb = -(-self.C // self.qb)
        self.nc = [n // PAGE for n in self.lens]
        self.nkb = [-(-(n + self.C) // PAGE) for n in self.lens]
        self.max_kv = c["table_blocks"] or max(self.nkb)
        self.words = -(-self.max_kv // 64)
        self.transposed = c["layout"] == "transposed"

    def listed_cached(self, c):
        """Cached blocks that row (b, g) of a given table lists (given tables
        differ in length by up to a quarter, as real selections do)."""
        out = []
        for b in range(self.B):
            for g in range(self.G):
                share = c["density"] * (0.88 + 0.24 * ((b * self.G + g) * 5 % 8) / 7)
                out.append(min(self.nc[b], int(round(share * self.nc[b]))))
        return out


def work(case):
    """What one pass cannot do without: each input read once, each output
    written once, 4 D operations per visible (query, key) pair."""
    s = _Sizes(case)
    kind = case["kind"]
    q_bytes = s.B * s.C * s.Hq * s.D * 2
    out_bytes = q_bytes + s.B * s.Hq * s.C * 4
    masks = s.B * s.Hq * s.nqb * s.words * 8
    n_bytes = flops = 0
    if kind in ("step", "fused", "estimate", "threshold"):
        pooled = sum(s.nkb) if kind in ("step", "estimate") else sum(
            n - _first_block(s) for n in s.nkb)
        n_bytes += s.Hkv * pooled * (PAGE * s.D * 2 + s.D * 4)    # K read, means written
        n_bytes += q_bytes + s.B * s.Hq * s.nqb * s.D * 4
        n_bytes += s.Hkv * (sum(s.nkb) - pooled) * s.D * 4        # carried means read
        n_bytes += s.Hq * s.nqb * sum(s.nc) * 4                   # scores written
        flops += 2 * s.D * s.Hq * s.nqb * sum(s.nc)
        if kind != "fused":
            n_bytes += masks
    if kind == "tables":
        n_bytes += masks
        per_row = 1 - (1 - case["density"]) ** (s.gs * s.nqb)
        n_bytes += 4 * s.G * sum(per_row * s.nc[b] + s.nkb[b] - s.nc[b] for b in range(s.B))
    if kind in ("step", "fused", "attention", "dense"):
        if kind == "attention":
            cached = s.listed_cached(case)
        elif kind == "dense":
            cached = [s.nc[b] for b in range(s.B) for _ in range(s.G)]
        else:
            # the rows of a group agree in part (RHO): their union grows like
            # that of about rows ** 0.47 independent rows
            keep = 1 - (1 - case["top"]) ** ((s.gs * s.nqb) ** 0.47)
            cached = [keep * s.nc[b] for b in range(s.B) for _ in range(s.G)]
        for b in range(s.B):
            tail = s.lens[b] - s.nc[b] * PAGE
            for g in range(s.G):
                n = cached[b * s.G + g]
                flops += 4 * s.D * s.gs * (s.C * (PAGE * n + tail) + s.C * (s.C + 1) / 2)
                # tables of one KV head share the pages they both list
                if kind != "dense" or g % (s.ratio // s.gs) == 0:
                    n_bytes += (n + s.nkb[b] - s.nc[b]) * 2 * PAGE * s.D * 2
        n_bytes += q_bytes + out_bytes
    return {"bytes": int(n_bytes), "flops": int(flops)}


def tolerance(case):
    kind = case["kind"]
    if kind == "tables":
        return "exact"
    if kind in ("estimate", "threshold"):
        # fp32 means and scores; a near tie may fall either way in the masks
        return {"rel": 1e-5, "max": 1e-4, "differ": 1e-3}
    # bf16 weights and outputs (2^-9 each), fp32 sums
    return {"rel": 1e-2, "max": 0.2, "differ": 1e-3}


def _first_block(s):
    """The first block whose mean is not yet final after the previous chunk."""
    return max(0, min(s.nc) - -(-s.C // PAGE))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _inputs(case, seed):
    s = _Sizes(case)
    kind = case["kind"]
    gen = torch.Generator(DEVICE).manual_seed(seed)

    def normal(*shape):
        return torch.randn(*shape, generator=gen, device=DEVICE, dtype=torch.float32)

    d = {}
    if kind == "tables":
        d["masks"] = _random_masks(case, s, gen)
        return d
    # queries share a direction within a KV group, so their selections agree in part
    mu = normal(s.B, 1, s.Hkv, 1, s.D).expand(-1, -1, -1, s.ratio, -1)
    q = normal(s.B, s.C, s.Hkv, s.ratio, s.D) * math.sqrt(1 - RHO * RHO) + RHO * mu
    d["q"] = q.reshape(s.B, s.C, s.Hq, s.D).to(torch.bfloat16)
    pages = s.Hkv * sum(s.nkb)
    d["k_pool"] = _normal_bf16(gen, (pages, PAGE, s.D))
    if kind not in ("estimate", "threshold"):
        d["v_pool"] = _normal_bf16(gen, (pages, s.D, PAGE) if s.transposed else (pages, PAGE, s.D))
    ids = torch.randperm(pages, generator=gen, device=DEVICE).to(torch.int32)
    table = torch.zeros(s.B, s.Hkv, s.max_kv, dtype=torch.int32, device=DEVICE)
    at = 0
    for b in range(s.B):
        n = s.Hkv * s.nkb[b]
        table[b, :, :s.nkb[b]] = ids[at:at + n].view(s.Hkv, s.nkb[b])
        at += n
    d["page_table"] = table
    if kind == "attention":
        d["tables"] = _random_tables(case, s, gen)
    return d


def _normal_bf16(gen, shape):
    out = torch.empty(shape, dtype=torch.bfloat16, device=DEVICE)
    return out.normal_(generator=gen)


def _random_masks(case, s, gen):
    """Random cached blocks at the case's density, the sink, the local window
    and the chunk's causal staircase, 64 blocks to a word."""
    j = torch.arange(s.words * 64, device=DEVICE)
    out = []
    for b in range(s.B):
        bits = torch.rand(s.Hq, s.nqb, s.words * 64, generator=gen, device=DEVICE) < case["density"]
        bits |= (j < SINK) | (j >= s.nc[b] - LOCAL)
        bits &= j < s.nc[b]
        last = torch.arange(1, s.nqb + 1, device=DEVICE) * s.qb
        end = (s.lens[b] + last.clamp(max=s.C) - 1) // PAGE + 1
        bits |= (j >= s.nc[b]) & (j < end[:, None])
        out.append(bits)
    bits = torch.stack(out).view(s.B, s.Hq, s.nqb, s.words, 64).to(torch.int64)
    return (bits << torch.arange(64, device=DEVICE)).sum(-1)


def _random_tables(case, s, gen):
    counts = s.listed_cached(case)
    rows = []
    for b in range(s.B):
        for g in range(s.G):
            order = torch.rand(s.nc[b], generator=gen, device=DEVICE).argsort()
            keep = order[:counts[b * s.G + g]].sort().values
            own = torch.arange(s.nc[b], s.nkb[b], device=DEVICE)
            rows.append(torch.cat([keep, own]).to(torch.int32))
    indptr = torch.zeros(len(rows) + 1, dtype=torch.int32)
    indptr[1:] = torch.tensor([len(r) for r in rows]).cumsum(0)
    indices = torch.zeros(len(rows) * s.max_kv, dtype=torch.int32, device=DEVICE)
    flat = torch.cat(rows)
    indices[:flat.numel()] = flat
    return indptr.to(DEVICE), indices


def prepare(case, seed):
    s = _Sizes(case)
    kind = case["kind"]
    st = _inputs(case, seed)
    p = ca.Problem(s.B, s.Hq, s.Hkv, s.D, s.qb, s.C, s.max_kv, s.lens, device=DEVICE,
                   v_layout=ca.V_TRANSPOSED if s.transposed else ca.V_TOKEN_MAJOR)
    st.update(case=dict(case), s=s, p=p, scale=s.D ** -0.5)
    zeros = lambda *shape, dtype=torch.float32: torch.zeros(*shape, dtype=dtype, device=DEVICE)  # noqa: E731
    if kind in ("step", "fused", "estimate", "threshold"):
        st["bufs"] = {"q_mean": zeros(s.B, s.Hq, s.nqb, s.D),
                      "k_mean": zeros(s.B, s.Hkv, s.max_kv, s.D),
                      "scores": zeros(s.B, s.Hq, s.nqb, s.max_kv)}
        if kind != "fused":
            st["bufs"]["masks"] = zeros(s.B, s.Hq, s.nqb, s.words, dtype=torch.int64)
        st["first_block"] = 0
        if kind in ("fused", "threshold"):   # what the earlier chunks left behind
            st["first_block"] = _first_block(s)
            ca.pool_k_blocks(p, st["k_pool"], st["page_table"], st["bufs"]["k_mean"])
    if kind in ("step", "fused", "tables"):
        rows = s.B * s.G
        st["tables"] = (zeros(rows + 1, dtype=torch.int32),
                        zeros(rows * s.max_kv, dtype=torch.int32))
        st["tables_ws"] = zeros(max(8, ca.tables_workspace_bytes(p, s.gs)), dtype=torch.uint8)
    if kind in ("step", "fused", "attention", "dense"):
        gs = s.ratio if kind == "dense" else s.gs
        st["out"] = torch.empty_like(st["q"])
        st["lse"] = zeros(s.B, s.Hq, s.C)
        n = ca.attention_workspace_bytes(p, gs, 0)
        st["ws"] = zeros(n, dtype=torch.uint8) if n else None
    return st


def run(st):
    kind, p, case = st["case"]["kind"], st["p"], st["case"]
    if kind == "tables":
        indptr, indices = ca.build_block_tables(p, st["masks"], case["group"], out=st["tables"],
                                                ws=st["tables_ws"])
        return {"kv_indptr": indptr, "kv_indices": indices}
    q, page_table = st["q"], st["page_table"]
    if kind == "threshold":
        masks, b = ca.estimate_masks_threshold(
            p, q, st["k_pool"], page_table, ALPHA, TEMPERATURE, st["scale"], SINK, LOCAL,
            k_mean_first_block=st["first_block"], bufs=st["bufs"])
        return {"masks": masks, "q_mean": b["q_mean"], "k_mean": b["k_mean"],
                "scores": b["scores"]}
    if kind in ("step", "estimate"):
        masks, b = ca.estimate_masks(p, q, st["k_pool"], page_table, case["top"], SINK, LOCAL,
                                     bufs=st["bufs"])
        if kind == "estimate":
            return {"masks": masks, "q_mean": b["q_mean"], "k_mean": b["k_mean"],
                    "scores": b["scores"]}
    kv = (st["k_pool"], st["v_pool"])
    if kind == "dense":
        out, lse = ca.dense_paged_chunk_attention(p, q, kv, page_table, st["scale"],
                                                  out=st["out"], lse=st["lse"], ws=st["ws"])
        return {"out": out, "lse": lse}
    got = {}
    if kind == "step":
        tables = ca.build_block_tables(p, masks, case["group"], out=st["tables"],
                                       ws=st["tables_ws"])
        got["masks"] = masks
    elif kind == "fused":
        tables, b = ca.estimate_tables(p, q, st["k_pool"], page_table, case["top"], case["group"],
                                       SINK, LOCAL, k_mean_first_block=st["first_block"],
                                       bufs=st["bufs"], out=st["tables"], ws=st["tables_ws"])
        got["k_mean"] = b["k_mean"]
    else:
        tables = st["tables"]
    got["out"], got["lse"] = ca.chunk_attention(p, q, kv, page_table, tables, case["group"],
                                                st["scale"], out=st["out"], lse=st["lse"],
                                                ws=st["ws"])
    return got


# ---------------------------------------------------------------------------
# the same in 64 bits, in plain torch
# ---------------------------------------------------------------------------
def exact(case, seed):
    s = _Sizes(case)
    kind = case["kind"]
    if kind == "tables":
        return None
    d = _inputs(case, seed)
    res = {}
    if kind in ("step", "fused", "estimate", "threshold"):
        q_mean, k_mean, scores = _pooled(s, d)
        if kind in ("estimate", "threshold"):
            return {"masks": None, "q_mean": q_mean, "k_mean": k_mean, "scores": scores}
        if kind == "step":
            res["masks"] = None
        else:
            res["k_mean"] = k_mean
        listed_blocks = _selected(case, s, scores)
    elif kind == "attention":
        ip, ix = d["tables"][0].cpu().tolist(), d["tables"][1]
        listed_blocks = [ix[ip[r]:ip[r + 1]].long() for r in range(s.B * s.G)]
    else:
        listed_blocks = [torch.arange(s.nkb[b], device=DEVICE) for b in range(s.B)
                         for _ in range(s.G)]
    res["out"], res["lse"] = _attend(s, d, listed_blocks)
    return res


def _pooled(s, d):
    q_mean = torch.zeros(s.B, s.Hq, s.nqb, s.D, dtype=torch.float64, device=DEVICE)
    k_mean = torch.zeros(s.B, s.Hkv, s.max_kv, s.D, dtype=torch.float64, device=DEVICE)
    scores = torch.zeros(s.B, s.Hq, s.nqb, s.max_kv, dtype=torch.float64, device=DEVICE)
    for b in range(s.B):
        for i in range(s.nqb):
            q_mean[b, :, i] = d["q"][b, i * s.qb:(i + 1) * s.qb].double().mean(0)
        for h in range(s.Hkv):
            k = d["k_pool"][d["page_table"][b, h, :s.nkb[b]].long()].double()
            k_mean[b, h, :s.nkb[b]] = k.mean(1)
            rows = s.lens[b] + s.C - PAGE * (s.nkb[b] - 1)
            k_mean[b, h, s.nkb[b] - 1] = k[-1, :rows].mean(0)
            heads = slice(h * s.ratio, (h + 1) * s.ratio)
            at = q_mean[b, heads].reshape(-1, s.D) @ k_mean[b, h, :s.nc[b]].T
            scores[b, heads, :, :s.nc[b]] = at.view(s.ratio, s.nqb, s.nc[b])
    return q_mean, k_mean, scores


def _selected(case, s, scores):
    rows = []
    for b in range(s.B):
        nc = s.nc[b]
        keep = torch.zeros(s.Hq, s.nqb, s.nkb[b], dtype=torch.bool, device=DEVICE)
        if nc:
            k = int(torch.ceil(torch.tensor(case["top"], dtype=torch.float32) * nc))
            keep.scatter_(2, scores[b, :, :, :nc].topk(min(k, nc), dim=2).indices, True)
            keep[..., :SINK] = True
            keep[..., max(0, nc - LOCAL):nc] = True
        keep[..., nc:] = True      # the last Q-block sees the whole chunk
        union = keep.view(s.G, s.gs, s.nqb, -1).any(1).any(1)
        rows += [union[g].nonzero().flatten() for g in range(s.G)]
    return rows


def _attend(s, d, listed_blocks):
    out = torch.empty(s.B, s.C, s.Hq, s.D, dtype=torch.float64, device=DEVICE)
    lse = torch.empty(s.B, s.Hq, s.C, dtype=torch.float64, device=DEVICE)
    ramp = torch.arange(PAGE, device=DEVICE)
    for b in range(s.B):
        pos = s.lens[b] + torch.arange(s.C, device=DEVICE)
        for g in range(s.G):
            blocks = listed_blocks[b * s.G + g]
            kv_head = g * s.gs // s.ratio
            ids = d["page_table"][b, kv_head][blocks].long()
            k = d["k_pool"][ids].reshape(-1, s.D).double()
            v = d["v_pool"][ids]
            v = (v.transpose(1, 2) if s.transposed else v).reshape(-1, s.D).double()
            at = (blocks[:, None] * PAGE + ramp).flatten()
            for h in range(g * s.gs, (g + 1) * s.gs):
                w = (d["q"][b, :, h].double() @ k.T).mul_(s.D ** -0.5)
                w.masked_fill_(at[None, :] > pos[:, None], -math.inf)
                lse[b, h] = torch.logsumexp(w, 1)
                out[b, :, h] = w.sub_(lse[b, h][:, None]).exp_() @ v
                del w
    return out, lse
