"""Outputs on either side of the 56 MB (with A) from which on C's stores pass the memory-side cache: the same bits, through every form of the register
epilogue and the edge tiles' one, and read back by the launch that follows."""
import pytest
import torch

import paper_2604_26666_amd as fact

pytestmark = pytest.mark.gpu
LINE = (56 << 20) // 2           # elements of A and C


def gemm(A, B, C, **ep):
    M, K = A.shape
    N = B.shape[0]
    fact.binding.check(fact.fact_gemm(M, N, K, A, K, B, K, 1, C, C.shape[1], fact.Epilogue(**ep)))


@pytest.mark.parametrize("form", ["plain", "bias", "gelu", "residual", "gated"])
@pytest.mark.parametrize("nout", [8192, 8200])                      # whole and ragged columns (of rows that end in an edge tile)
def test_both_sides_of_the_line(form, nout):
    g = torch.Generator(device="cuda").manual_seed(5)
    K, N = 64, 2 * nout if form == "gated" else nout
    few = LINE // (nout + K)                                              # the last row count without the policy; one more has it
    A = torch.randn(few + 1, K, generator=g, device="cuda").bfloat16()
    B = torch.randn(N, K, generator=g, device="cuda").mul_(K ** -0.5).bfloat16()
    R = torch.randn(few + 1, nout, generator=g, device="cuda").bfloat16()
    bias = torch.randn(nout, generator=g, device="cuda").bfloat16()
    ep = {"plain": {}, "bias": dict(bias=bias), "gelu": dict(bias=bias, act=fact.ACT_GELU_TANH), "residual": dict(bias=bias, residual=R, ldr=nout),
          "gated": dict(act=fact.ACT_SILU_GATE)}[form]
    outs = []
    for M in (few, few + 1):
        C = torch.full((M + 1, nout), 77.0, dtype=torch.bfloat16, device="cuda")
        gemm(A[:M], B, C, **ep)
        # the next launch reads C: a product with the identity gives its bits back
        D = torch.empty(M, 64, dtype=torch.bfloat16, device="cuda")
        eye = torch.zeros(64, nout, dtype=torch.bfloat16, device="cuda")
        eye[:, -64:] = torch.eye(64, device="cuda").bfloat16()
        gemm(C[:M], eye, D)
        torch.cuda.synchronize()
        assert (C[M] == 77.0).all(), "wrote past C"
        assert torch.equal(D, C[:M, -64:])
        outs.append(C[:M])
    assert torch.equal(outs[0], outs[1][:few])
    z = A.float() @ B.float().t()
    if form == "gated":
        z = torch.nn.functional.silu(z[:, :nout]) * z[:, nout:]
    if "bias" in ep:
        z = z + bias.float()
    if form == "gelu":
        z = torch.nn.functional.gelu(z, approximate="tanh")
    if form == "residual":
        z = z + R.float()
    err = (outs[1].float() - z).abs()
    # one rounding to bf16 (2^-9 of the value), and fp32 sums of 64 products of the operands' size
    assert bool((err <= z.abs() * 2.0 ** -8 + 2e-5 * (1 + z.abs())).all()), float(err.max())


@pytest.mark.parametrize("config", [13, 14, 15])                    # the 192-wide tiles, with a kernel for either policy
@pytest.mark.parametrize("f16", [0, 1])
def test_both_sides_of_the_line_192_wide(config, f16):
    dtype = torch.float16 if f16 else torch.bfloat16
    g = torch.Generator(device="cuda").manual_seed(6)
    K, N = 64, 7688
    few = LINE // (N + K)
    A = torch.randn(few + 1, K, generator=g, device="cuda").to(dtype)
    B = torch.randn(N, K, generator=g, device="cuda").mul_(K ** -0.5).to(dtype)
    bias = torch.randn(N, generator=g, device="cuda").to(dtype)
    outs = []
    for M in (few, few + 1):
        C = torch.full((M + 1, N), 77.0, dtype=dtype, device="cuda")
        fact.binding.check(fact.fact_gemm_ex(1, M, N, K, A, K, 0, B, K, 0, 1, C, N, 0, fact.Epilogue(bias=bias, act=fact.ACT_GELU_TANH, f16=f16), config, 1, 4, None, 0))
        torch.cuda.synchronize()
        assert (C[M] == 77.0).all(), "wrote past C"
        outs.append(C[:M])
    assert torch.equal(outs[0], outs[1][:few])
    ref = torch.nn.functional.gelu(A.float() @ B.float().t() + bias.float(), approximate="tanh")
    # one rounding to bfloat16 (2^-9) or binary16 (2^-12, subnormal below 2^-14) of sums and a tanh that differ in the last places of fp32
    assert ((outs[1].float() - ref).abs() <= ref.abs() * 2.0 ** -8 + 2.0 ** -16).all()


# every tile width whose policy is chosen in its code, interior and edge tiles (the last rows and columns of all of these)
@pytest.mark.parametrize("config", [0, 2, 5, 6, 7, 16, 17])
@pytest.mark.parametrize("gated", [False, True])
def test_both_sides_of_the_line_by_tile(config, gated):
    g = torch.Generator(device="cuda").manual_seed(7)
    K, nout = 64, 7744                                                  # rows of whole and of half lines, written through for either form
    few = LINE // (nout + K)
    A = torch.randn(few + 1, K, generator=g, device="cuda").bfloat16()
    B = torch.randn(2 * nout if gated else nout, K, generator=g, device="cuda").mul_(K ** -0.5).bfloat16()
    outs = []
    for M in (few, few + 1):
        C = torch.full((M + 1, nout), 77.0, dtype=torch.bfloat16, device="cuda")
        ep = fact.Epilogue(act=fact.ACT_SILU_GATE if gated else fact.ACT_NONE)
        fact.binding.check(fact.fact_gemm_ex(1, M, len(B), K, A, K, 0, B, K, 0, 1, C, nout, 0, ep, config, 1, 4, None, 0))
        torch.cuda.synchronize()
        assert (C[M] == 77.0).all(), "wrote past C"
        outs.append(C[:M])
    assert torch.equal(outs[0], outs[1][:few])
    ref = A.float() @ B.float().t()
    if gated:
        ref = torch.nn.functional.silu(ref[:, :nout]) * ref[:, nout:]
    # one rounding to bfloat16 (2^-9) of sums of 64 products of the operands' size, whose order differs
    assert ((outs[1].float() - ref).abs() <= ref.abs() * 2.0 ** -8 + 2e-5 * (1 + ref.abs())).all()
