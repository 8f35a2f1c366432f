"""Which kernels a GEMM call runs on (host logic, no GPU): the launches that each rule of the dispatch gives, around its lines."""
import math
import os
import random

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


# A and C above 56 MB: C passes the memory-side cache, in both parts of a call or in neither
def test_both_parts_of_a_column_split_store_alike():
    rng, seen = random.Random(3), [0, 0]
    size = lambda lo, hi: int(math.exp(rng.uniform(math.log(lo), math.log(hi))))
    shapes = [(6521, 3008, 1904, 0, 0), (3300, 5592, 4968, 1, 0), (4907, 7800, 1088, 1, 0), (1024, 50257, 768, 1, 0), (2048, 28672, 4096, 1, 2), (1, 64, 64, 1, 0)]
    shapes += [(size(1024, 8192), size(128, 1024) * 8, size(32, 1024) * 8, 1, 0) for _ in range(4000)]
    for M, N, K, nk, act in shapes:
        r = route(M, N, K, nk, act)
        if len(r) == 2:
            past = M * ((N // 2 if act else N) + K) * 2 > 56 << 20
            assert fact.fact_test_route_streams() == [past, past], (M, N, K, nk, act)
            seen[past] += 1
    assert seen[0] > 5 and seen[1] > 50


def test_a_call_that_is_refused_has_no_route():
    assert route(0, 8, 8, 1) == -2 and route(8, 8, 8, 1, cfg=99) == -7 and route(8, 8, 8, 1, a=None) == -1


# 32-bit indexes: a block of K loaded past the last one, or a tile's edge, must not pass 2^31 (the guarded kernel counts K one by one)
@pytest.mark.parametrize("nk", [0, 1])
def test_ragged_kernel_keeps_its_indexes_in_range(nk):
    top, last = 2 ** 31 - 1, 2 ** 31 - 1 - 4096
    for K in (top, top - 63, top - 960, last + 1):
        assert kernels(1, 8, K, nk) == ["guarded"], K
    # (12 blocks of 64 past the last, with the waves that split K, are well below the margin, and so is a tile's edge)
    assert kernels(1, 8, last, nk) == ["ragged"]
    for K in (25, 999, 2 ** 21 + 8):              # odd rows, and aligned ones past the tile kernel's leading dimensions
        assert kernels(3, 9, K, nk) == ["ragged"], K
    assert kernels(last + 1, 9, 25, nk) == ["guarded"] and kernels(1, last + 2, 25, nk) == ["guarded"] and kernels(1, last, 25, nk) == ["ragged"]


def test_tile_kernel_keeps_its_edges_in_range():
    # a last tile of up to 256 rows or columns must not reach past 2^31
    edge = 2 ** 31 - 1 - 256
    assert kernels(edge, 8, 8, 0) == ["tiles"] and kernels(72, edge, 8, 1) == ["tiles"]
    for over in (edge + 1, 2 ** 31 - 1):
        assert kernels(over, 8, 8, 0) == ["guarded"] and kernels(72, over, 8, 1) == ["guarded"]
        assert route(over, 8, 8, 0, cfg=0) == -7


# Few rows against [N][K] weights.  (M, N, K, batch, with a workspace): the skinny kernel where it measured faster than the plan,
# the plan (here one that splits K over the whole chip, or tiles) where the skinny kernel has a handful of work-groups for
# a long K, or more of them than weights to share A
@pytest.mark.parametrize("M,N,K,batch,ws,want", [
    (16, 4096, 14336, 1, False, "skinny"), (16, 4096, 14336, 1, True, "skinny"), (1, 3072, 768, 1, True, "skinny"), (64, 3072, 768, 1, False, "skinny"),
    (16, 768, 3072, 1, True, "skinny"), (16, 64, 8192, 1, True, "skinny"), (16, 16384, 8192, 1, True, "skinny"), (16, 256, 1024, 8, False, "skinny"),
    (16, 64, 32768, 1, False, "skinny"), (64, 64, 131072, 1, False, "skinny"),
    (64, 64, 131072, 1, True, "tiles"), (16, 64, 65536, 1, True, "tiles"), (16, 128, 131072, 1, True, "tiles"), (1, 16, 32768, 1, True, "tiles"),
    (32, 256, 32768, 1, True, "tiles"), (48, 512, 8192, 1, True, "tiles"), (64, 256, 8192, 1, True, "tiles"),
    (16, 16384, 256, 1, False, "tiles"), (32, 16384, 1024, 1, False, "tiles"), (64, 8192, 1024, 1, False, "tiles"),
    (64, 512, 1024, 128, False, "tiles"), (32, 64, 4096, 128, False, "tiles"), (48, 4096, 1024, 8, False, "tiles")])
def test_few_rows(M, N, K, batch, ws, want):
    got = kernels(M, N, K, 1, batch=batch, ws=ws)
    plan = fact.fact_select_config(batch, M, N, K, 1, 0)
    assert got == (["skinny"] if want == "skinny" else ["tiles", "reduce"] if ws and plan[2] > 1 else ["tiles"])


# small outputs with a workspace, where the plan splits K: the kernel whose waves split it for the shorter ones
@pytest.mark.parametrize("M,N,K,nk,want", [(280, 120, 7232, 1, ["skinny"]), (80, 304, 15168, 1, ["tiles", "reduce"]), (352, 328, 6848, 1, ["tiles", "reduce"]),
                                           (72, 64, 5888, 0, ["skinny"]), (160, 64, 7680, 0, ["tiles", "reduce"]), (256, 64, 8192, 0, ["tiles", "reduce"])])
def test_small_outputs_whose_plan_splits_k(M, N, K, nk, want):
    assert kernels(M, N, K, nk, ws=True) == want and kernels(M, N, K, nk) == ["skinny"]


def test_few_rows_only_where_nothing_else_was_asked_for():
    assert kernels(16, 4096, 4096, 1) == ["skinny"]
    assert kernels(16, 4096, 4096, 0) == ["tiles"] and kernels(65, 4096, 4096, 1) == ["tiles"]
    assert kernels(16, 4096, 4096, 1, cfg=6) == ["tiles"] and kernels(16, 4096, 4096, 1, ws=True, split=4) == ["tiles", "reduce"]
    assert kernels(16, 4096, 4096, 1, a=P + 2) == ["ragged"]


# at most 32 rows: tiles of 32 columns only where tiles of 16 are more than compute units (203, 211 and 256 work-groups; 257 and 304)
@pytest.mark.parametrize("M,N,K,form", [(27, 3248, 1864, "2x1/3"), (30, 3376, 880, "2x1/3"), (32, 4096, 624, "2x1/3"), (25, 4112, 624, "2x2/2"), (26, 4856, 2336, "2x2/3")])
def test_half_the_chip_does_not_fetch_the_weights_of_few_rows(M, N, K, form):
    assert [(k, fact.SKINNY_FORMS[c]) for k, c, _ in route(M, N, K, 1)] == [("skinny", form)]


def test_few_rows_of_more_columns_than_a_grid_counts():
    # (such weights would be 500 GB and more: the pricing alone does not rule them out)
    assert kernels(1, 2 ** 27 - 16, 2048, 1) == ["skinny"]
    assert kernels(1, 2 ** 28, 2048, 1) == ["tiles"] and kernels(16, 2 ** 28, 1024, 1, fact.ACT_SILU_GATE) == ["tiles"]


def test_a_grid_never_has_more_threads_than_it_counts():
    # 2^32 threads and more along x would be cut to 32 bits without an error
    for M, N in ((2 ** 30 - 8, 64), (2 ** 30, 8), (2 ** 30 + 64, 64), (2 ** 31 - 300, 8)):
        for nk in (0, 1):
            (kind, cfg, _), = route(M, N, 8, nk)
            bm, bn, wm, wn, _ = fact.fact_config_info(cfg)
            assert kind == "tiles" and -(-M // bm) * -(-N // bn) * wm * wn * 64 < 2 ** 32, (M, N, nk, cfg)
            for c in range(fact.fact_num_configs()):
                bm, bn, wm, wn, _ = fact.fact_config_info(c)
                if nk or bn != 192:
                    fits = -(-M // bm) * -(-N // bn) * wm * wn * 64 < 2 ** 32
                    assert kernels(M, N, 8, nk, cfg=c) == (["tiles"] if fits else -2), (M, N, c)


# rows of any alignment with a short K: the guarded kernel where it has little to do or the ragged kernel's tiles are mostly edge
@pytest.mark.parametrize("M,N,K,nk,batch,want", [
    (8, 8, 9, 0, 1, "guarded"), (1, 1000, 9, 1, 1, "guarded"), (300, 300, 9, 0, 1, "guarded"), (150, 50, 13, 1, 1, "guarded"), (100000, 9, 9, 1, 1, "guarded"),
    (100000, 9, 17, 0, 1, "guarded"), (9, 100000, 9, 0, 1, "guarded"),
    (8, 8, 17, 0, 1, "ragged"), (300, 300, 17, 1, 1, "ragged"), (1000, 1000, 9, 0, 1, "ragged"), (4000, 300, 9, 1, 1, "ragged"), (100000, 33, 9, 0, 1, "ragged"),
    (100000, 9, 17, 1, 1, "ragged"), (9, 100000, 13, 0, 1, "ragged"), (100, 100, 9, 0, 64, "ragged"), (8, 8, 25, 0, 1, "ragged"), (8, 8, 7, 1, 1, "guarded")])
def test_short_k_of_any_alignment(M, N, K, nk, batch, want):
    assert kernels(M, N, K, nk, batch=batch) == [want]


def test_persistent_launches_are_taken_as_they_stand():
    M, N, K = 16, 131072, 4096
    grid = fact.fact_persistent_grid(1, M, N, K, 1)
    assert grid == 0 and kernels(M, N, K, 1) == ["skinny"]
    was = fact.fact_tune_persistent(1)
    try:
        assert fact.fact_persistent_grid(1, M, N, K, 1) > 0 and kernels(M, N, K, 1) == ["persistent"]
        assert kernels(M, 4096, K, 1) == ["skinny"]                         # every tile is resident: no persistent launch to take
        assert kernels(1024, 50257, 768, 1) == ["persistent"]              # and none is split into two
    finally:
        fact.fact_tune_persistent(was)


def test_launches_of_a_block():
    from paper_2604_26666_amd import workbench
    gpt = {"d_model": 768, "q_heads": 12, "kv_heads": 12, "head_dim": 64, "d_ff": 3072, "act_gated": False, "rope": False}
    llama = {"d_model": 4096, "q_heads": 32, "kv_heads": 8, "head_dim": 128, "d_ff": 14336, "act_gated": True, "rope": True}
    assert workbench.block_launches(8, 1024, gpt) == 2 + 1 + 4                  # norms, attention, one launch per GEMM
    assert workbench.block_launches(1, 2048, llama) == 2 + 1 + 1 + 5            # rotary as well, and the gate / up GEMM over columns in two
