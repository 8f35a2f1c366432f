"""fact_attention in every shape of work-group that its rule can choose (query groups x key groups x keys of a block), at lengths
where a query group, a key block or a key group's share ends, some of them with key groups that see no key: against 64-bit
attention, with the tolerance of test_gpu_attention.py."""
import math

import pytest
import torch

import paper_2604_26666_amd as fact
from test_gpu_attention_order import check, run, tensors

# (B, T, Hq, Hkv, D) by the shape that they take: groups of 32 queries x key groups x keys of a block
FULL = [(8, 97, 12, 12, 64), (3, 200, 32, 8, 64), (2, 127, 96, 96, 64)]                                      # 4 x 1 x 64
SHORT = [(3, 65, 32, 8, 64), (8, 129, 12, 12, 64), (8, 160, 16, 4, 64), (3, 96, 32, 32, 64)]                 # 4 x 1 x 32
PAIRS = [(2, 65, 32, 8, 64), (3, 97, 16, 16, 64), (5, 129, 12, 12, 64), (3, 200, 16, 4, 64), (2, 300, 24, 6, 64)]       # 2 x 2 x 64
SINGLE = [(1, 65, 2, 1, 64), (1, 96, 4, 4, 64), (1, 97, 2, 2, 64), (2, 127, 4, 2, 64), (3, 129, 2, 2, 64), (1, 417, 2, 1, 64), (1, 900, 2, 2, 64)]       # 1 x 4 x 32
WIDE = [(3, 97, 12, 4, 128), (8, 70, 16, 4, 128), (3, 127, 32, 8, 128)]                                      # head_dim 128: 4 x 1 x 64
WIDE_PAIRS = [(1, 129, 2, 2, 128), (2, 160, 2, 1, 128), (3, 200, 12, 4, 128), (1, 257, 32, 8, 128)]          # 2 x 2 x 32
WIDE_SINGLE = [(1, 65, 2, 1, 128), (1, 96, 2, 2, 128), (1, 97, 2, 2, 128), (3, 127, 2, 2, 128), (2, 65, 4, 4, 128)]     # 1 x 4 x 32
SHAPES = [((4, 1, 64), FULL + WIDE), ((4, 1, 32), SHORT), ((2, 2, 64), PAIRS), ((1, 4, 32), SINGLE + WIDE_SINGLE), ((2, 2, 32), WIDE_PAIRS)]


@pytest.mark.parametrize("causal", [0, 1])
@pytest.mark.parametrize("shape,calls", SHAPES, ids=lambda x: "x".join(map(str, x)) if isinstance(x, tuple) else "")
def test_the_rule(shape, calls, causal):
    for B, T, Hq, _, D in calls:
        assert fact.fact_test_attention_shape(B, T, Hq, D, causal) == shape, (B, T, Hq, D)


@pytest.mark.gpu
@pytest.mark.parametrize("causal", [0, 1])
@pytest.mark.parametrize("B,T,Hq,Hkv,D", FULL + SHORT + PAIRS + SINGLE + WIDE + WIDE_PAIRS + WIDE_SINGLE + [(2, 129, 32, 32, 64), (2, 300, 32, 8, 64)])
def test_lengths(B, T, Hq, Hkv, D, causal):
    q, k, v = tensors(B, T, Hq, Hkv, D, 21)
    check(run(q, k, v, causal), q, k, v, causal, [(0, 0), (0, Hq - 1), (B - 1, Hq // 2)])


@pytest.mark.gpu
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("H,T", [(2, 96), (2, 337), (32, 289)])
@pytest.mark.parametrize("last", [False, True])
def test_one_group_holds_all_the_weight(D, H, T, last):
    # one key outweighs all others by far: the groups' reference exponents differ by hundreds, and all but one sum vanish
    q, k, v = tensors(1, T, H, H, D, 23)
    q.mul_(0.25)
    k.mul_(0.25)
    q[..., 0] = 1.0
    k[..., 0] = 0.0
    k[:, T - 1 if last else T // 2, :, 0] = 400.0
    check(run(q, k, v, 0, 1.0), q, k, v, 0, [(0, 0), (0, H - 1)], 1.0)


@pytest.mark.gpu
def test_the_same_bits_again():
    for B, T, H, D in ((1, 900, 2, 64), (2, 300, 32, 64), (1, 257, 32, 128), (3, 127, 2, 128)):
        q, k, v = tensors(B, T, H, H, D, 25)
        assert torch.equal(run(q, k, v, 1).view(torch.int16), run(q, k, v, 1).view(torch.int16))


# Keys that a caller masks through a spare element of the heads: their scores are the lowest there is, or as good as that.
# (B, T, Hq, Hkv, D, first and last + 1 of the keys left): in every shape, blocks of masked keys before and behind the others, among
# them a wave's first ones
MASKED = [(1, 96, 4, 4, 64, 0, 40), (1, 200, 2, 2, 64, 33, 200), (1, 417, 2, 1, 64, 100, 300), (2, 300, 32, 8, 64, 70, 129), (3, 97, 16, 16, 64, 0, 60),
          (2, 300, 24, 6, 64, 70, 129), (8, 160, 16, 4, 64, 32, 160), (8, 129, 12, 12, 64, 0, 50), (8, 97, 12, 12, 64, 0, 64), (3, 200, 32, 8, 64, 31, 130),
          (1, 97, 2, 2, 128, 0, 32), (2, 127, 4, 4, 128, 64, 127), (2, 160, 2, 1, 128, 0, 30), (1, 257, 32, 8, 128, 33, 257), (3, 127, 32, 8, 128, 40, 127)]


def test_masked_keys_come_in_every_shape():
    assert {(fact.fact_test_attention_shape(B, T, Hq, D, c), c) for B, T, Hq, _, D, _, _ in MASKED for c in (0, 1)} == {(s, c) for s, _ in SHAPES for c in (0, 1)}


@pytest.mark.gpu
@pytest.mark.parametrize("value", [-math.inf, torch.finfo(torch.bfloat16).min, -1e20, -1e9])
@pytest.mark.parametrize("causal", [0, 1])
@pytest.mark.parametrize("B,T,Hq,Hkv,D,first,last", MASKED)
def test_masked_keys(B, T, Hq, Hkv, D, first, last, causal, value):
    q, k, v = tensors(B, T, Hq, Hkv, D, 27)
    q[..., 0] = 1.0
    k[..., 0] = value
    k[:, first:last, :, 0] = 0.0
    O = run(q, k, v, causal)
    seen = first if causal else 0                            # (a query before the first key left sees masked ones alone)
    # the same without the masked keys: against 64-bit attention over the others, each query with the keys that it may see
    assert not torch.isnan(O[:, seen:]).any()
    for b, h in ((0, 0), (0, Hq - 1), (B - 1, Hq // 2)):
        kk, vv = k[b, first:last, h // (Hq // Hkv)].double(), v[b, first:last, h // (Hq // Hkv)].double()
        s = (q[b, seen:, h].double() @ kk.t().contiguous()) / math.sqrt(D)
        if causal:
            s.masked_fill_(torch.arange(first, last, device="cuda")[None] > torch.arange(seen, T, device="cuda")[:, None], -math.inf)
        p = torch.softmax(s, -1)
        want, bound = p @ vv, p @ vv.abs()
        err = (O[b, seen:, h].double() - want).abs()
        assert (err <= 1e-2 * bound + 1e-3).all(), (b, h, float((err - 1e-2 * bound).max()))
