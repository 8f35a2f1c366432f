"""The last rounding of norms and GEMMs, bit for bit, over all of bfloat16.  Norms: rows of +1 and -1 with eps = 0 normalise to themselves
exactly, so an output is +-gamma + beta rounded once to fp32 and once to bfloat16, which the host computes as well - halves
between two values, sums that overflow, subnormal results, infinities and NaN.  GEMMs: rows of A that
pick one row of B, so an output is B's value plus the bias."""
import pytest
import torch

import paper_2604_26666_amd as F

pytestmark = pytest.mark.gpu


def _bits(values):
    return torch.tensor(values, dtype=torch.int32).to(torch.int16).view(torch.bfloat16)


@pytest.mark.parametrize("T,d", [(4, 768), (9, 2048), (5, 4096), (2048, 1536)])
def test_norm_rounds_every_kind_of_sum(T, d):
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


# the kernel whose waves split K, the one for rows at any address, the main kernel's interior and edge tiles, split K's reduction pass
@pytest.mark.parametrize("M,N,K,split", [(3, 51, 32, 1), (48, 96, 64, 1), (1201, 1203, 77, 1), (256, 512, 64, 1), (1208, 1208, 64, 1), (300, 264, 1024, 4), (300, 264, 1024, 64)])
def test_gemm_rounds_every_kind_of_sum(M, N, K, split):
    gen = torch.Generator().manual_seed(M + N)
    some = lambda n: torch.randint(0, 1 << 16, n, generator=gen, dtype=torch.int32)
    B = some((N, K))
    e = B & 0x7F80
    B = torch.where((e == 0x7F80) | (e == 0), 0x3F80, B)                        # finite and not subnormal: zeros times them are zeros
    bias = torch.where(torch.arange(N) % 2 == 0, (B[:, 0] & 0x8000) | ((B[:, 0] & 0x7F80) - (8 << 7)).clamp(min=0), some((N,)))
    special = [(0x7F7F, 0x7B80), (0x7F7F, 0x7B00), (0x3F80, 0x3B80), (0x3F81, 0x3B80), (0x0100, 0x80FF), (0x0080, 0x8081), (0x3F80, 0x7F80),
               (0x3F80, 0xFF80), (0x3F80, 0x7FC0), (0x3F80, 0xFFC0), (0x4000, 0xC000)]
    for i, (b, c) in enumerate(special):
        B[i, 0], bias[i] = b, c
    B, bias = _bits(B.tolist()), _bits(bias.tolist())
    A = torch.zeros(M, K, dtype=torch.bfloat16)
    pick = torch.arange(M) % K
    A[torch.arange(M), pick] = 1
    want = (B.double()[:, pick].T + bias.double()).float().bfloat16()
    Ad, Bd, C = A.cuda(), B.cuda(), torch.empty(M, N, dtype=torch.bfloat16, device="cuda")
    ws = torch.empty(max(16, F.fact_gemm_splitk_workspace_bytes(M, N, K, split)), dtype=torch.uint8, device="cuda")
    F.binding.check(F.fact_gemm_splitk(M, N, K, Ad, K, Bd, K, 1, C, N, F.Epilogue(bias=bias.cuda()), split, ws, ws.numel()))
    torch.cuda.synchronize()
    got, nan = C.cpu(), want.isnan()
    assert torch.equal(got.isnan(), nan)
    assert torch.equal(got.view(torch.int16)[~nan], want.view(torch.int16)[~nan])
