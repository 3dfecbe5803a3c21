"""Block scores and top-k selection at the edges of their kernels: tile remainders,
register-held key counts, and score distributions that take each search path."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_16839_amd as ca
from _helpers import u64_host

pytestmark = pytest.mark.gpu

# keys per thread change after 256, 1024, 2048, 4096 and 8192 blocks
SIZES = [1, 2, 255, 256, 257, 1024, 1025, 2048, 2049, 4097, 8192, 9000]


def _scores(kind, rng, shape):
    n = shape[-1]
    s = rng.standard_normal(shape).astype(np.float32)
    if kind == "equal":            # one bucket, every key tied
        s[...] = 1.25
    elif kind == "outlier":        # one far score: the rest in one bucket
        s[..., rng.integers(n)] = 1e20
    elif kind == "outliers":       # and one far from the next: bucket after bucket
        s[..., :8] = np.float32(10.0) ** np.arange(4, 36, 4)[:min(n, 8)]
    elif kind == "scales":         # every scale of float32, both signs
        s = (np.sign(s) * 2.0 ** rng.integers(-140, 127, s.shape)).astype(np.float32)
    elif kind == "few":            # a few values: more ties than a bucket ranks
        s = np.round(2 * s).astype(np.float32)
    elif kind == "clusters":       # buckets of many nearly equal keys
        s = (np.round(s) + 1e-4 * s).astype(np.float32)
    elif kind == "huge":           # the range overflows float32
        s = np.where(s > 0, 3e38, -3e38).astype(np.float32)
        s[..., ::7] = 0.0
    elif kind == "tiny":           # denormal range
        s = (s * np.float32(1e-41)).astype(np.float32)
    elif kind == "infinite":       # a few infinities of both signs
        s[..., ::11] = np.inf
        s[..., 3::13] = -np.inf
    return s


@pytest.mark.parametrize("kind", ["normal", "equal", "outlier", "outliers", "scales", "few",
                                  "clusters", "huge", "tiny", "infinite"])
@pytest.mark.parametrize("nc", SIZES)
def test_select_is_exact(kind, nc):
    rng = np.random.default_rng(nc)
    Hq, C, qb = 2, 192, 128
    maxkb = nc + C // 64
    p = ca.Problem(1, Hq, 1, 64, qb, C, maxkb, [64 * nc])
    scores = np.full((1, Hq, 2, maxkb), np.nan, dtype=np.float32)
    s = _scores(kind, rng, (Hq, 2, nc))
    scores[0, :, :, :nc] = s
    for top in sorted({0.0, 0.4 / nc, 1.0 / nc, 0.05, 0.37, 1.0 - 1.0 / nc, 1.0}):
        ref = oracle.masks_from_scores([s], [64 * nc], C, 64, qb, p.words,
                                       oracle.EstimatorParams(top, 1, 4))
        got = ca.select_blocks(p, torch.from_numpy(scores).cuda(), top)
        assert np.array_equal(u64_host(got), ref), top


@pytest.mark.parametrize("heads,chunk,qb,dim", [
    ((1, 1), 64, 64, 64), ((4, 1), 128, 128, 128), ((31, 1), 64, 64, 128), ((8, 2), 500, 64, 64),
    ((33, 1), 64, 64, 128), ((16, 2), 1024, 128, 128), ((13, 1), 320, 64, 64)])
@pytest.mark.parametrize("cached", [(64 * 31, 100), (64 * 64, 64 * 65), (64 * 129, 0)])
def test_scores_at_tile_edges(heads, chunk, qb, dim, cached):
    """Row tiles of 32 (one or two per workgroup) and block tiles of 32, each with
    one row or block too few or too many; fp32 sums of dim products of values of
    about 1: an error of 1e-5 is 80 units in the last place of such a sum."""
    rng = np.random.default_rng(heads[0])
    maxkb = max((c + chunk + 63) // 64 for c in cached)
    p = ca.Problem(len(cached), *heads, dim, qb, chunk, maxkb, list(cached))
    q = rng.standard_normal((len(cached), heads[0], p.n_qblocks, dim)).astype(np.float32)
    k = rng.standard_normal((len(cached), heads[1], maxkb, dim)).astype(np.float32)
    got = ca.block_scores(p, torch.from_numpy(q).cuda(), torch.from_numpy(k).cuda()).cpu().numpy()
    ratio = heads[0] // heads[1]
    for b, c in enumerate(cached):
        nc = c // 64
        ref = np.einsum("hid,hjd->hij", q[b].astype(np.float64),
                        np.repeat(k[b], ratio, axis=0)[:, :nc].astype(np.float64))
        assert np.abs(got[b, :, :, :nc] - ref).max(initial=0.0) <= 1e-5 * np.sqrt(dim)
        assert np.isnan(got[b, :, :, nc:]).all()      # nothing else is written
