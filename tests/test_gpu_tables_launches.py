"""Block tables around the line between one launch and two (48 rows, 4 MiB of mask
reads, four rounds of loads per wave) and at the edges of the word layout (one word,
32, 64 and 256 words)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_16839_amd as ca
from _helpers import u64_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("blocks", [1, 63, 64, 65, 2015, 2049, 4097, 16384])
@pytest.mark.parametrize("batch,heads,gs,chunk", [
    (1, 4, 4, 64),      # 1 row
    (2, 12, 2, 200),    # 12 rows of two heads x 4 Q-blocks
    (8, 8, 1, 64),      # 64 rows
    (5, 13, 1, 64),     # 65 rows
    (6, 8, 1, 64),      # 48 rows
    (7, 7, 1, 64),      # 49 rows: two launches
    (1, 8, 8, 1024),    # 128 mask rows: one launch up to 32 words
    (2, 4, 4, 1024),    # 64 mask rows: one launch up to 64 words
    (4, 32, 4, 1100),   # up to 4.7 MB of masks
])
def test_tables_match_oracle(blocks, batch, heads, gs, chunk):
    rng = np.random.default_rng(blocks)
    qb = 64
    cap = blocks * 64 - chunk
    if cap < 0:
        pytest.skip("the chunk alone needs more blocks")
    cached = [cap] + [int(rng.integers(0, cap + 1)) for _ in range(batch - 1)]
    p = ca.Problem(batch, heads, 1, 64, qb, chunk, blocks, cached)
    nkb = [(c + chunk + 63) // 64 for c in cached]
    shape = (batch, heads, p.n_qblocks, p.words)
    masks = rng.integers(0, 2**64, shape, dtype=np.uint64)
    for _ in range(4):          # sparse, with bits past each sequence's end too
        masks &= rng.integers(0, 2**64, shape, dtype=np.uint64)
    masks[0, :, :, 0] = 0
    ip, ix = oracle.tables_to_csr(oracle.block_tables(masks, gs, nkb))
    out = (torch.full((batch * (heads // gs) + 1,), -7, dtype=torch.int32, device="cuda"),
           torch.full((batch * (heads // gs) * blocks,), -7, dtype=torch.int32, device="cuda"))
    ca.build_block_tables(p, u64_dev(masks), gs, out=out)
    assert np.array_equal(out[0].cpu().numpy(), ip)
    got = out[1].cpu().numpy()
    assert np.array_equal(got[:ip[-1]], ix) and (got[ip[-1]:] == -7).all()
