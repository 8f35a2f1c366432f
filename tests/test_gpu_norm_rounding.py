"""The norm kernel's last rounding, bit for bit, over all of bfloat16: rows of +1 and -1 with eps = 0 normalise to themselves
exactly, so an output is +-gamma + beta rounded once to fp32 and once to bfloat16, which the host computes as well - halves
between two values, sums that overflow, subnormal results, infinities and NaN."""
import pytest
import torch

import paper_2604_26666_amd as F

pytestmark = pytest.mark.gpu


def _bits(values):
    return torch.tensor(values, dtype=torch.int32).to(torch.int16).view(torch.bfloat16)


@pytest.mark.parametrize("T,d", [(4, 768), (9, 2048), (5, 4096), (2048, 1536)])
def test_rounding_of_every_kind_of_sum(T, d):
    gen = torch.Generator().manual_seed(d)
    gamma = torch.randint(0, 1 << 16, (d,), generator=gen, dtype=torch.int32)
    # beta: half of gamma's last place or thereabouts (ties and their neighbours), or anything
    near = (gamma & 0x8000) | ((gamma & 0x7FFF) - (8 << 7)).clamp(min=0)
    beta = torch.where(torch.arange(d) % 2 == 0, near & 0xFF80, torch.randint(0, 1 << 16, (d,), generator=gen, dtype=torch.int32))
    special = [(0x7F7F, 0x7B80), (0x7F7F, 0x7B00), (0x3F80, 0x3B80), (0x3F81, 0x3B80), (0x0001, 0x0001), (0x0080, 0x8001), (0x7F80, 0x3F80),
               (0x7F80, 0xFF80), (0x7FC0, 0x0000), (0x0000, 0xFFC0), (0x8000, 0x8000), (0x0000, 0x0000)]
    for i, (g, b) in enumerate(special):
        gamma[i], beta[i] = g, b
    gamma, beta = _bits(gamma.tolist()), _bits(beta.tolist())
    x = torch.ones(T, d)
    x[:, 1::2] = -1
    x[1::2] *= -1
    # (a sum of two bfloat16 values needs more than float64's 53 bits only where one is below 2^-45 of the other: no rounding here sees it then)
    want = (x.double() * gamma.double() + beta.double()).float().bfloat16()
    xd, gd, bd = x.bfloat16().cuda(), gamma.cuda(), beta.cuda()
    y = torch.empty_like(xd)
    assert F.fact_norm(T, d, xd, d, gd, bd, 0.0, 0, y, d) == 0
    torch.cuda.synchronize()
    got, nan = y.cpu(), want.isnan()
    assert torch.equal(got.isnan(), nan)
    assert torch.equal(got.view(torch.int16)[~nan], want.view(torch.int16)[~nan])
