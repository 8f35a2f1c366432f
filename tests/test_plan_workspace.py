"""What a call with a workspace takes and refuses (host logic, no GPU): a plan that wants more K ranges than the caller's workspace holds gives way to the one
that fits, and the least that is accepted is what it was before such plans (sizes that callers may have kept)."""
import math
import os
import random

import pytest

import paper_2604_26666_amd as fact

P = 0x10000          # a 128-byte aligned address; never dereferenced
WORKSPACE, UNSUPPORTED = -6, -7


@pytest.fixture(scope="module", autouse=True)
def _built():
    if not os.path.exists(fact.lib_path()):
        from paper_2604_26666_amd import build
        build.build()


def route(M, N, K, nk, ws, ws_bytes, split=0, cfg=-1):
    return fact.fact_test_route(1, M, N, K, P, K, M * K, P, K if nk else N, K * N, nk, P, N, M * N, fact.Epilogue(), cfg, split, 0, P if ws else None, ws_bytes)


# (M, N, K, least bytes): the second kind needs none
@pytest.mark.parametrize("nk", [0, 1])
@pytest.mark.parametrize("M,N,K,least", [(162, 888, 3056, 1150848), (398, 2056, 35648, 26185216), (213, 96, 9264, 654336), (851, 144, 32656, 7842816), (73, 168, 3672, 98112),
                                         (600, 2048, 5632, 9830400), (1032, 1024, 4096, 8454144)])
def test_least_workspace(M, N, K, least, nk):
    full = fact.fact_gemm_splitk_workspace_bytes(M, N, K, 0)
    assert full >= least
    # (the query is the largest over layouts: a call of one of them may take less, but never less than its own plan's planes)
    split = next(s for s in (2, 4, 8, 16, 32, 64) if s * M * N * 4 >= least)
    assert split * M * N * 4 == least
    for have in (least, (least + full) // 32 * 16, full, 1 << 40):
        r = route(M, N, K, nk, True, have)
        assert isinstance(r, list) and r, (have, r)
    assert route(M, N, K, nk, True, least - 16) == WORKSPACE


@pytest.mark.parametrize("M,N,K", [(610, 5040, 13784), (1249, 2352, 13952), (2054, 976, 5792)])
def test_no_workspace_where_none_was_needed(M, N, K):
    # the plan has ranges where there is room for them, and none otherwise: nothing is refused
    full = fact.fact_gemm_splitk_workspace_bytes(M, N, K, 0)
    assert full > 0
    assert [x[0] for x in route(M, N, K, 1, True, full)] == ["tiles", "reduce"]
    for have in (0, 16, full - 16):
        without = route(M, N, K, 1, True, have)
        assert isinstance(without, list) and "reduce" not in [x[0] for x in without], (have, without)


# (T, d_model, d_ff, activation, bytes before there was a plan for launches of one round, bytes now)
@pytest.mark.parametrize("T,d,dff,act,least,full", [(384, 1024, 4096, 1, 6291456, 6291456), (105, 4096, 14336, 2, 13762560, 13762560), (600, 2048, 5632, 2, 9830400, 9830400),
                                                    (610, 5040, 13784, 1, 0, 24595200), (96, 768, 3072, 1, 589824, 1769472)])
def test_mlp_query_is_never_below_what_it_was(T, d, dff, act, least, full):
    assert fact.fact_block_mlp_workspace_bytes(T, d, dff, act) == full >= least


def test_ranges_that_the_caller_asks_for_stay():
    for split in (1, 2, 3, 5):
        r = route(600, 2048, 5632, 1, True, 1 << 40, split=split)
        assert [x[0] for x in r] == (["tiles"] if split == 1 else ["tiles", "reduce"])
    assert route(600, 2048, 5632, 1, True, 3 * 600 * 2048 * 4 - 16, split=3) == WORKSPACE


@pytest.mark.parametrize("M,N,K", [(456, 5960, 5464), (3266, 704, 7072), (374, 5416, 6304), (610, 5040, 13784)])
def test_too_small_a_workspace_is_planned_as_none(M, N, K):
    full, none = fact.fact_gemm_splitk_workspace_bytes(M, N, K, 0), route(M, N, K, 1, False, 0)
    assert len(route(M, N, K, 1, True, full)) == 2 and len(none) == 1
    for have in (0, 16, full // 32 * 16, full - 16):
        assert route(M, N, K, 1, True, have) == none, have


def test_no_ranges_beyond_the_static_array():
    # (three ranges of 15 MB would be the quicker plan, and two are no clear gain)
    assert fact.fact_gemm_splitk_workspace_bytes(2074, 1824, 44312, 0) == 0
    assert [x[0] for x in route(2074, 1824, 44312, 1, True, 1 << 40)] == ["tiles"]


def test_the_static_array_has_the_room_of_any_workspace():
    # fact_gemm_splitk_static promises fact_gemm_splitk's bits: one plan for the array's size and for all beyond, wherever the array serves the call
    rng = random.Random(7)
    size = lambda lo, hi: int(math.exp(rng.uniform(math.log(lo), math.log(hi))))
    cap = fact.fact_gemm_splitk_static_capacity()
    shapes = [(1067, 6704, 64504), (370, 464, 89168), (1100, 4096, 14336)] + [(size(65, 8192), size(8, 1024) * 8, size(32, 16384) * 8) for _ in range(3000)]
    split = 0
    for M, N, K in shapes:
        for nk in (0, 1):
            here, beyond = route(M, N, K, nk, True, cap), route(M, N, K, nk, True, 1 << 40)
            assert here == WORKSPACE or here == beyond, (M, N, K, nk, here, beyond)
            split += len(beyond) > 1
    assert split > 500


# more K ranges than a grid counts, on shapes with a plan for one round, with a long K, and on few rows
@pytest.mark.parametrize("M,N,K", [(600, 2048, 5632), (4096, 512, 4096), (65, 8, 2 ** 21), (64, 4096, 4096)])
@pytest.mark.parametrize("cfg", [-1, -2, 6])
@pytest.mark.parametrize("split", [65536, 2 ** 31 - 88, 2 ** 31 - 1])
def test_more_ranges_than_there_can_be_are_refused(M, N, K, cfg, split):
    for nk in (0, 1):
        assert route(M, N, K, nk, True, 1 << 62, split=split, cfg=cfg) == UNSUPPORTED


@pytest.mark.parametrize("M,N", [(65, 8), (4096, 4096)])
def test_as_many_ranges_as_there_can_be(M, N):
    assert [x[0] for x in route(M, N, 2 ** 21, 1, True, 1 << 62, split=65535)] == ["tiles", "reduce"]


# outputs of half a chip of 128 x 128 tiles, and what lies beside them
@pytest.mark.parametrize("M,N,K,nk,tile", [(512, 4096, 14336, 1, (128, 64)), (4096, 512, 4096, 0, (64, 128)), (3136, 488, 3200, 0, (64, 128)), (419, 4096, 1024, 1, (64, 128)),
                                           (256, 4096, 14336, 1, (64, 64)), (2904, 768, 3072, 1, (128, 128)), (4096, 4096, 2048, 1, (256, 256))])
def test_tiles(M, N, K, nk, tile):
    (kind, cfg, _), = route(M, N, K, nk, False, 0, split=1)
    assert kind == "tiles" and tuple(sorted(fact.fact_config_info(cfg)[:2])) == tuple(sorted(tile))


# K whole in the place of the ranges that model_time splits it in: by a clear gain, a clearer one where few compute units read much, and never from 64 MB on
@pytest.mark.parametrize("M,N,K,kinds", [(320, 768, 3072, ["skinny"]), (320, 2048, 5632, ["tiles"]), (1237, 1024, 4096, ["tiles"]), (229, 1224, 3072, ["tiles"]),
                                         (320, 1024, 4096, ["tiles", "reduce"]), (256, 2048, 5632, ["tiles", "reduce"]), (8118, 96, 31360, ["tiles", "reduce"])])
def test_whole_k_in_the_place_of_ranges(M, N, K, kinds):
    assert [x[0] for x in route(M, N, K, 1, True, 1 << 40)] == kinds


# ranges of another tile from 64 MB on: by the same gain as below but for small outputs of B as [K][N]
@pytest.mark.parametrize("M,N,K,nk,tile", [(424, 112, 71104, 1, (64, 64)), (128, 432, 103104, 0, (128, 128))])
def test_ranges_of_large_operands(M, N, K, nk, tile):
    r = route(M, N, K, nk, True, 1 << 40)
    assert [x[0] for x in r] == ["tiles", "reduce"] and tuple(fact.fact_config_info(r[0][1])[:2]) == tile


# calls with a workspace at which model_time's plan is the quicker one, each for a reason of its own (at clear_gain and skinny_choice): where the estimate for one
# round says otherwise it stays.  (M, N, K, B as [N][K], kinds of launch, tile)
@pytest.mark.parametrize("M,N,K,nk,kinds,tile", [
    (94, 11264, 16728, 0, ["tiles", "reduce"], (128, 256)), (8118, 96, 31360, 0, ["tiles", "reduce"], (256, 128)), (7002, 128, 20864, 1, ["tiles", "reduce"], (128, 128)),
    (128, 432, 103104, 0, ["tiles", "reduce"], (128, 128)), (130, 72, 16488, 1, ["tiles", "reduce"], (64, 64)), (168, 1704, 30800, 1, ["tiles", "reduce"], (128, 128)),
    (797, 592, 29520, 1, ["tiles", "reduce"], (128, 192)), (621, 3776, 5568, 1, ["tiles"], (128, 128)), (464, 224, 5912, 1, ["tiles", "reduce"], (64, 64)),
    (208, 80, 6784, 0, ["skinny"], None), (128, 96, 11008, 1, ["skinny"], None)])
def test_model_times_plan_stays(M, N, K, nk, kinds, tile):
    r = route(M, N, K, nk, True, 1 << 40)
    assert [x[0] for x in r] == kinds
    assert tile is None or tuple(fact.fact_config_info(r[0][1])[:2]) == tile
