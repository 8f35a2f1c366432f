"""Which kernels a GEMM call runs on (host logic, no GPU): the launches that each rule of the dispatch gives, around its lines."""
import os

import pytest

import paper_2604_26666_amd as fact

P = 0x10000          # a 128-byte aligned address; never dereferenced


@pytest.fixture(scope="module", autouse=True)
def _built():
    if not os.path.exists(fact.lib_path()):
        from paper_2604_26666_amd import build
        build.build()


def route(M, N, K, nk, act=fact.ACT_NONE, batch=1, ws=False, a=P, lda=None, ldb=None, cfg=-1, split=None, **ep):
    """[(kernel, configuration, columns)]; ws: as fact_gemm_splitk with split_k = 0 and a large workspace, else as fact_gemm(_batched)."""
    nout, ldb = (N // 2 if act == fact.ACT_SILU_GATE else N), (K if nk else N) if ldb is None else ldb
    return fact.fact_test_route(batch, M, N, K, a, K if lda is None else lda, M * K, P, ldb, K * N, nk, P, nout, M * nout,
                                fact.Epilogue(act=act, **ep), cfg, (0 if ws else 1) if split is None else split, 0, P if ws else None, 1 << 40 if ws else 0)


def kernels(*a, **k):
    r = route(*a, **k)
    return r if isinstance(r, int) else [x[0] for x in r]


# a nearly empty last round of tiles: two launches over the columns, of whole tiles in the first
@pytest.mark.parametrize("M,N,K,nk,act", [(1024, 50257, 768, 1, 0), (5018, 6648, 800, 0, 0), (7268, 2536, 2552, 1, 0), (2048, 28672, 4096, 1, 2)])
def test_column_split(M, N, K, nk, act):
    (k1, c1, n1), (k2, c2, n2) = route(M, N, K, nk, act)
    assert k1 == k2 == "tiles" and n1 + n2 == N and c1 == fact.fact_select_config(1, M, N, K, nk, act)[1]
    bm, bn = fact.fact_config_info(c1)[:2]
    rows, full = -(-M // bm), (-(-M // bm) * -(-N // bn) - 1) // 256 * 256
    assert n1 % bn == 0 and rows * (n1 // bn) <= full < rows * (n1 // bn + 1)        # as many whole columns of tiles as the full rounds hold
    # one launch: the columns of the full rounds alone, a launch that the caller chose, and a batch
    assert [x[0] for x in route(M, n1, K, nk, act)] == ["tiles"]
    assert [x[0] for x in route(M, N, K, nk, act, cfg=c1)] == ["tiles"]
    assert [x[0] for x in route(M, N, K, nk, act, batch=2)] == ["tiles"]


def test_a_call_that_is_refused_has_no_route():
    assert route(0, 8, 8, 1) == -2 and route(8, 8, 8, 1, cfg=99) == -7 and route(8, 8, 8, 1, a=None) == -1


# 32-bit indexes: a step loaded ahead, or a tile's edge, must not pass 2^31 (the guarded kernel counts K one by one)
@pytest.mark.parametrize("nk", [0, 1])
def test_ragged_kernel_keeps_its_indexes_in_range(nk):
    top, last = 2 ** 31 - 1, 2 ** 31 - 1 - 4096
    for K in (top, top - 63, top - 960, last + 1):
        assert kernels(1, 8, K, nk) == ["guarded"], K
    # groups x steps ahead x depth, all below the margin, and a tile's edge
    assert 3 * 4 * 64 + 4 * 64 + 64 < 4096 and kernels(1, 8, last, nk) == ["ragged"]
    for K in (9, 999, 2 ** 21 + 8):               # short rows, odd ones, and aligned ones past the tile kernel's leading dimensions
        assert kernels(3, 9, K, nk) == ["ragged"], K
    assert kernels(last + 1, 9, 9, nk) == ["guarded"] and kernels(1, last + 2, 9, nk) == ["guarded"] and kernels(1, last, 9, nk) == ["ragged"]


def test_tile_kernel_keeps_its_edges_in_range():
    # a last tile of up to 256 rows or columns must not reach past 2^31
    edge = 2 ** 31 - 1 - 256
    assert kernels(edge, 8, 8, 0) == ["tiles"] and kernels(72, edge, 8, 1) == ["tiles"]
    for over in (edge + 1, 2 ** 31 - 1):
        assert kernels(over, 8, 8, 0) == ["guarded"] and kernels(72, over, 8, 1) == ["guarded"]
        assert route(over, 8, 8, 0, cfg=0) == -7
