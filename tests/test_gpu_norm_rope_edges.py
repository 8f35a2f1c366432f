"""fact_norm and fact_rope at the sizes where their work splits change: rows of one wave and of four, the last piece of a
row, few and many tokens per work-group, heads with more than 256 angles - against the block oracle, usual tolerance."""
import pytest
import torch

import paper_2604_26666_amd as fact
import workloads as wl
from oracle import block as blk
from oracle import check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rms", [0, 1])
@pytest.mark.parametrize("T,d", [(1, 512), (3, 520), (5, 1024), (5, 1032), (2, 2048), (2, 2056), (7, 4104),
                                 (2047, 1032), (2049, 1032), (2048, 1536), (2050, 1544), (2051, 2040), (2048, 2048)])
def test_norm_rows_of_one_and_four_waves(T, d, rms):
    X = wl.normal((T, d), 2.0, f"ne.X.{T}.{d}") + wl.normal((T, 1), 3.0, f"ne.s.{T}.{d}")
    g, b = wl.normal((d,), 1.0, f"ne.g.{d}"), wl.normal((d,), 0.5, f"ne.b.{d}")
    Y = torch.full((T + 1, d), 77.0, dtype=torch.bfloat16, device="cuda")
    fact.binding.check(fact.fact_norm(T, d, X.cuda(), d, g.cuda(), None if rms else b.cuda(), 1e-5, rms, Y, d))
    torch.cuda.synchronize()
    assert (Y[T] == 77.0).all()
    r = blk.rmsnorm(wl.bits(X), wl.bits(g)) if rms else blk.layernorm(wl.bits(X), wl.bits(g), wl.bits(b))
    check.assert_close(wl.bits(Y[:T].cpu().contiguous()), r, what=f"T={T} d={d} rms={rms}")


@pytest.mark.parametrize("B,T,H,D", [(1, 1, 1, 16), (3, 171, 2, 64), (2, 1031, 3, 128), (1, 9, 2, 512), (1, 5, 2, 544), (40, 40, 1, 32),
                                     # few heads: a thread per 8 angles and token; work-groups of an intermediate number of tokens
                                     (1, 12501, 1, 64), (3, 7001, 3, 128), (2, 1031, 1, 16), (1, 2100, 1, 544), (40, 60, 1, 32), (1, 16387, 2, 16),
                                     # heads shared by several work-groups, the last group short
                                     (1, 1, 300, 128), (3, 5, 257, 64), (1, 2, 70, 1024), (16, 1, 129, 96)])
def test_rope_token_groups_and_wide_heads(B, T, H, D):
    base = 10000.0
    X = wl.normal((B, T, H, D), 1.0, f"re.{B}.{T}.{H}.{D}")
    Xd = X.cuda()
    fact.binding.check(fact.fact_rope(B, T, H, D, Xd, (T * H * D, H * D, D), base))
    torch.cuda.synchronize()
    ang = torch.arange(T, dtype=torch.float64)[:, None] * base ** (-2.0 * torch.arange(D // 2, dtype=torch.float64) / D)
    c, s, x = ang.cos()[None, :, None], ang.sin()[None, :, None], X.double()
    lo, hi = x[..., : D // 2], x[..., D // 2:]
    want = torch.cat([lo * c - hi * s, hi * c + lo * s], dim=-1)
    # one rounding to bf16 (2^-8 of the value) and the angle's fp32 error, t * 2^-23 of a turned pair of size up to |x|
    err = (Xd.cpu().double() - want).abs()
    assert (err <= 2.0 ** -8 * want.abs() + T * 2.0 ** -22 * x.abs().max() + 1e-6).all(), err.max()


@pytest.mark.parametrize("T,d", [(2 ** 26 + 8, 8), (2 ** 22 + 5, 64), (2 ** 20 + 3, 1032)])
def test_more_rows_than_one_grid_row_holds(T, d):
    # every work-group's row is written, also past the first row of the grid (2^26 rows of one wave each are 2^32 threads).
    # A row of +-c is normed to +-c / sqrt(c^2 + eps): c = 1, 2, 3, 4 in turn
    c = (torch.arange(T, device="cuda") % 4 + 1).bfloat16()
    X = torch.ones((1, d), dtype=torch.bfloat16, device="cuda")
    X[0, ::2] = -1
    X = c[:, None] * X
    g = torch.full((d,), 2.0, dtype=torch.bfloat16, device="cuda")
    Y = torch.full((T, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    fact.binding.check(fact.fact_norm(T, d, X, d, g, None, 0.0, 1, Y, d))
    torch.cuda.synchronize()
    for x, y in zip(X.split(1 << 23), Y.split(1 << 23)):
        assert torch.equal(y, x.sign() * 2)
