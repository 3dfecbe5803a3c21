"""Which launch an attention call takes, asked of the debug library on the host: the
sizes that the GPU tests run for a launch take that launch, a workspace too small
falls back, and sizes whose times the rule was once wrong about."""
import ctypes
import os

import pytest

import paper_2605_16839_amd as ca
import test_gpu_not_finite
import test_gpu_pieces as pieces

HALF, SHARES, XCD, UNIFORM = 1, 2, 3, 16   # UNIFORM + the number of splits


@pytest.fixture(scope="module")
def launch():
    if not os.path.exists(ca.DEBUG_LIB_PATH):
        pytest.fail("libcompactattn_debug.so is not built (run __graft_entry__.build())")
    fn = ca.load(ca.DEBUG_LIB_PATH).ca_debug_attention_launch
    fn.restype, fn.argtypes = ctypes.c_int, [ctypes.c_void_p, ctypes.c_int32, ctypes.c_int32,
                                             ctypes.c_size_t]

    def ask(cached, chunk, heads, dim, group, dense, short=0, ws=None):
        p = _problem(cached, chunk, heads, dim)
        n = ca.attention_workspace_bytes(p, group, 0) - short if ws is None else ws
        return fn(ctypes.addressof(p.c), group, int(dense), n)
    return ask


def _problem(cached, chunk, heads, dim):
    nkb = max(-(-(c + chunk) // 64) for c in cached)
    return ca.Problem(len(cached), *heads, dim, 64, chunk, nkb, list(cached), device=None)


@pytest.mark.parametrize("sizes,want", [(pieces.SHARES, SHARES), (pieces.HALF, HALF)])
def test_listed_sizes(launch, sizes, want):
    for cached, chunk, heads, dim, group, _, density in sizes:
        assert launch(cached, chunk, heads, dim, group, density is None) == want, (cached, chunk)


def test_uniform_sizes(launch):
    got = [launch(c, n, h, d, g, density is None) for c, n, h, d, g, _, density in pieces.UNIFORM]
    assert got == [UNIFORM + 8, UNIFORM + 4, UNIFORM + 4, UNIFORM + 16]


def test_sparse_rows(launch):
    for chunk in (100, 1300):
        assert launch((30000, 8000), chunk, (32, 8), 64, 4, False) == SHARES
    for cached, chunk in pieces.SPARSE_HALF:
        assert launch(cached, chunk, (32, 8), 64, 4, False, ws=0) == HALF


def test_not_finite_launches(launch):
    auto = [x for x in test_gpu_not_finite.LAUNCHES if x[-1] == 0]
    assert [launch(*x[:5], False) for x in auto] == [SHARES, SHARES, XCD]


def test_workspace_too_small(launch):
    cached, chunk, heads, dim, group, _, _ = pieces.SHARES[2]
    assert launch(cached, chunk, heads, dim, group, False, short=1) == UNIFORM + 7
    assert launch(cached, chunk, heads, dim, group, False, ws=0) == HALF
    # tiles that fill the GPU: whole ones
    assert launch((129024,), 2048, (32, 8), 128, 4, False, ws=0) == UNIFORM + 1


# Sizes at which the launch chosen by the sizes alone took longer than another (us,
# chosen : other, one GPU).
@pytest.mark.parametrize("cached,chunk,heads,dim,group,dense,want", [
    # rows of different lengths that the XCDs do not hold alike: half tiles 173 : 122, 188 : 163
    ((154, 2789, 389), 1113, (32, 4), 128, 8, True, UNIFORM + 1),
    ((28864, 33024, 320, 30272, 320, 4544, 896, 128), 2048, (4, 1), 64, 4, False, XCD),
    # uniform splits give every CU one piece: equal shares 38 : 34, 80 : 72
    ((5888, 4544, 1024, 512), 64, (16, 16), 128, 1, False, UNIFORM + 4),
    ((84672, 74240), 64, (32, 8), 128, 2, False, UNIFORM + 8),
    # rows short enough that no cut pays: equal shares 66, uniform splits 54, half tiles 50
    ((8381, 8939, 7720, 1361), 194, (32, 8), 128, 4, False, HALF),
    # 64-dimensional heads walk a page faster and start sooner: half tiles 19 : 16, 17 : 15
    ((1087,), 62, (4, 1), 64, 4, False, UNIFORM + 4),
    ((976,), 17, (4, 1), 64, 2, False, UNIFORM + 4),
    # tiles that fill the GPU once, rows much alike: equal shares 104 : 93
    ((4427, 1022, 5604, 3403), 512, (32, 8), 128, 4, False, XCD),
    # long selections differ from row to row; dense rows do not
    ((129024,), 512, (32, 8), 128, 4, False, SHARES),
    ((129024,), 512, (32, 8), 128, 4, True, UNIFORM + 4),
    ((129024,), 2048, (32, 8), 128, 4, False, XCD),
])
def test_choice(launch, cached, chunk, heads, dim, group, dense, want):
    assert launch(cached, chunk, heads, dim, group, dense) == want


def test_no_shares_workspace_for_half_tiles():
    """Where half tiles run (no workspace), the query does not ask for equal shares:
    only for the splits that an explicit or block-sparse launch may use."""
    p = _problem((0, 0), 700, (32, 8), 64)
    rows = 2 * 32 * 700
    assert ca.attention_workspace_bytes(p, 4, 0) == 2 * rows * 65 * 4   # 176 tiles: 2 splits


@pytest.mark.parametrize("chunk,rows", [(1, 16), (4, 16), (5, 32), (37, 160), (64, 256)])
def test_slots_hold_the_rows_of_the_chunk(launch, chunk, rows):
    """One query tile: a partial result has the 16-row fragments with a query, not
    the 256 rows of the workgroup (a 34.9 MB workspace for one token over 64K)."""
    assert launch((65536,), chunk, (32, 8), 128, 4, False) == SHARES
    slots = 256 + 8     # a piece that goes on from another per CU, a first one per row
    partial = (slots * rows * 129 * 4 + 15) & ~15
    assert ca.attention_workspace_bytes(_problem((65536,), chunk, (32, 8), 128), 4, 0) == \
        partial + 8 * 16
