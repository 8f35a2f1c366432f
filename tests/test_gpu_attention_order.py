"""fact_attention where its work-group order folds back (causal launches whose work-groups are all resident at
once, with and without a multiple of 8 (batch, head) pairs, edges of a layer) and where the reference exponent
of the running sums has to be raised: against 64-bit attention, with the tolerance of test_gpu_attention.py."""
import math

import pytest
import torch

import paper_2604_26666_amd as fact

pytestmark = pytest.mark.gpu


def run(q, k, v, causal, scale=0.0):
    B, T, Hq, D = q.shape
    Hkv = k.shape[2]
    O = torch.full((B, T, Hq, D), float("nan"), dtype=torch.bfloat16, device="cuda")
    st = lambda x: tuple(x.stride()[:3])
    fact.binding.check(fact.fact_attention(B, T, Hq, Hkv, D, q, st(q), k, st(k), v, st(v), O, st(O), causal, scale))
    torch.cuda.synchronize()
    return O


def check(O, q, k, v, causal, heads, scale=0.0):
    assert not torch.isnan(O).any(), "rows left unwritten, or no numbers"
    T, D, G = q.shape[1], q.shape[3], q.shape[2] // k.shape[2]
    for b, h in heads:
        s = (q[b, :, h].double() @ k[b, :, h // G].double().t().contiguous()) * (scale or 1.0 / math.sqrt(D))
        if causal:
            s.masked_fill_(torch.ones(T, T, dtype=torch.bool, device="cuda").triu_(1), -math.inf)
        p = torch.softmax(s, -1)
        want, bound = p @ v[b, :, h // G].double(), p @ v[b, :, h // G].double().abs()
        err = (O[b, :, h].double() - want).abs()
        assert (err <= 1e-2 * bound + 1e-3).all(), (b, h, float((err - 1e-2 * bound).max()))
        assert float(err.norm() / want.norm()) < 3e-3


def tensors(B, T, Hq, Hkv, D, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    new = lambda H: torch.randn((B, T, H, D), generator=g, device="cuda").bfloat16()
    return new(Hq), new(Hkv), new(Hkv)


# (B, T, Hq, Hkv, D): two layers of 32 work-groups per XCD just reached and just full, three layers (head_dim 64), one
# work-group past the residency, 12 pairs in one sequence over two layers of 256
@pytest.mark.parametrize("B,T,Hq,Hkv,D", [(1, 1025, 32, 8, 128), (1, 2048, 32, 8, 128), (1, 2049, 32, 8, 128), (8, 1024, 12, 12, 64),
                                          (1, 2800, 12, 4, 128), (1, 5600, 12, 12, 64), (1, 129, 8, 8, 64)])
def test_every_row_of_a_folded_order(B, T, Hq, Hkv, D):
    q, k, v = tensors(B, T, Hq, Hkv, D, 5)
    check(run(q, k, v, 1), q, k, v, 1, [(0, 0), (0, Hq - 1), (B - 1, Hq // 2)])


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("causal", [1, 0])
@pytest.mark.parametrize("jump", [3.0, 9.0, 200.0, 3000.0])
def test_reference_exponent_is_raised(D, causal, jump):
    # every query's score of a key of block j is about j * jump (natural logarithm's domain): sums pass the limit
    # slowly, at every block, or overflow to infinity before they are rescaled
    T = 64 * 5 + 17
    q, k, v = tensors(1, T, 2, 1, D, 7)
    q.mul_(0.25)
    k.mul_(0.25)
    q[..., 0] = 1.0
    k[..., 0] = (torch.arange(T, device="cuda") // 64 * jump).bfloat16()[None, :, None]
    check(run(q, k, v, causal, 1.0), q, k, v, causal, [(0, 0), (0, 1)], 1.0)


@pytest.mark.parametrize("D", [64, 128])
def test_falling_scores_keep_the_first_reference(D):
    T = 300
    q, k, v = tensors(1, T, 2, 2, D, 9)
    q.mul_(0.25)
    k.mul_(0.25)
    q[..., 0] = 1.0
    k[..., 0] = (-(torch.arange(T, device="cuda") // 64) * 40.0).bfloat16()[None, :, None]
    check(run(q, k, v, 0, 1.0), q, k, v, 0, [(0, 0), (0, 1)], 1.0)


def test_more_work_groups_than_one_grid_row_counts():
    # 2^24 + 8 work-groups of 256 threads pass the 32-bit thread count of a grid's row: single tokens, whose result is V itself.
    # The batch stride of Q, K and V is 0, so only the output is large (2 GB)
    B, H, D = 2 ** 21 + 1, 8, 64
    q, k, v = tensors(1, 1, H, H, D, 11)
    O = torch.full((B, H, D), float("nan"), dtype=torch.bfloat16, device="cuda")
    fact.binding.check(fact.fact_attention(B, 1, H, H, D, q, (0, H * D, D), k, (0, H * D, D), v, (0, H * D, D), O, (H * D, H * D, D), 0, 0.0))
    torch.cuda.synchronize()
    for part in O.split(1 << 19):
        assert torch.equal(part, v[0].expand_as(part))
