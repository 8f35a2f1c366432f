"""GEMMs whose last round of work-groups is nearly empty run as two launches over the columns: every output column is
written once, with the bits that one launch on a forced configuration gives (K is whole in both, so the order of the
sums is the same), for each operand that the second launch reaches at an offset."""
import pytest
import torch

import paper_2604_26666_amd as fact
import workloads as wl
from oracle import check, ref

pytestmark = pytest.mark.gpu

# (M, N, K, B as [N][K]): 3.08 rounds and odd rows of C; 2.03 rounds, B as [K][N]; 1.59 rounds of 256 x 192 tiles
SHAPES = [(1024, 50257, 768, 1), (5018, 6648, 800, 0), (7268, 2536, 2552, 1)]


def assert_two_launches(M, N, K, nk, act=fact.ACT_NONE):
    p, nout = 1 << 16, N // 2 if act == fact.ACT_SILU_GATE else N
    r = fact.fact_test_route(1, M, N, K, p, K, 0, p, K if nk else N, 0, nk, p, nout, 0, fact.Epilogue(act=act))
    assert [x[0] for x in r] == ["tiles", "tiles"], r


def tensor(shape, dt, seed, std=1.0):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return (torch.randn(shape, generator=g, device="cuda") * std).to(dt)


@pytest.mark.parametrize("f16,f32", [(0, 0), (1, 0), (0, 1)])
@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_same_bits_as_one_launch(shape, f16, f32):
    M, N, K, nk = shape
    assert_two_launches(M, N, K, nk)
    dt, odt = (torch.float16 if f16 else torch.bfloat16), (torch.float32 if f32 else torch.float16 if f16 else torch.bfloat16)
    A, B = tensor((M, K), dt, 1), tensor((N, K) if nk else (K, N), dt, 2, K ** -0.5)
    bias, res = tensor((N,), dt, 3), tensor((M, N), dt, 4)
    ep = fact.Epilogue(bias=bias, residual=res, ldr=N, f16=f16, out_f32=f32)
    ldc = N + 8
    C, D = (torch.full((M + 1, ldc), float("nan"), dtype=odt, device="cuda") for _ in range(2))
    rc, cfg, _ = fact.fact_select_config(1, M, N, K, nk, fact.ACT_NONE)
    fact.binding.check(rc)
    ldb = K if nk else N
    fact.binding.check(fact.fact_gemm(M, N, K, A, K, B, ldb, nk, C, ldc, ep))
    fact.binding.check(fact.fact_gemm_ex(1, M, N, K, A, K, 0, B, ldb, 0, nk, D, ldc, 0, ep, cfg, 1, 4, None, 0))
    torch.cuda.synchronize()
    assert torch.isnan(C[M]).all() and torch.isnan(C[:, N:]).all(), "wrote outside C"
    assert not torch.isnan(C[:M, :N]).any(), "columns left unwritten"
    assert torch.equal(C[:M, :N], D[:M, :N])


@pytest.mark.parametrize("halves", [False, True])
def test_gated_rest_takes_both_weight_matrices_at_an_offset(halves):
    T, d, dff = 2048, 4096, 14336
    assert_two_launches(T, 2 * dff, d, 1, fact.ACT_SILU_GATE)
    X, W = tensor((T, d), torch.bfloat16, 5), tensor((2 * dff, d), torch.bfloat16, 6, 0.02)
    ep = fact.Epilogue(act=fact.ACT_SILU_GATE)
    H, D = (torch.full((T, dff), float("nan"), dtype=torch.bfloat16, device="cuda") for _ in range(2))
    if halves:
        W2 = tensor((d, dff), torch.bfloat16, 7, 0.02)
        need = fact.fact_block_mlp_workspace_bytes(T, d, dff, fact.ACT_SILU_GATE)
        ws, Y = torch.empty(max(need, 16), dtype=torch.uint8, device="cuda"), torch.empty((T, d), dtype=torch.bfloat16, device="cuda")
        up = W[dff:].clone()
        fact.binding.check(fact.fact_block_mlp(T, d, dff, X, W[:dff], up, None, fact.ACT_SILU_GATE, W2, None, None, H, Y, ws, need))
    else:
        fact.binding.check(fact.fact_gemm(T, 2 * dff, d, X, d, W, d, 1, H, dff, ep))
    fact.binding.check(fact.fact_gemm_ex(1, T, 2 * dff, d, X, d, 0, W, d, 0, 1, D, dff, 0, ep, 0, 1, 4, None, 0))
    torch.cuda.synchronize()
    assert torch.equal(H, D)


def test_against_the_oracle_around_the_seam():
    M, N, K = 1024, 50257, 768
    assert_two_launches(M, N, K, 1)
    A, B = wl.small_int((M, K), -4, 4, "cs.A"), wl.small_int((N, K), -4, 4, "cs.B")
    Ad, Bd = A.cuda(), B.cuda()
    C = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    fact.binding.check(fact.fact_gemm(M, N, K, Ad, K, Bd, K, 1, C, N, None))
    cols = slice(49152 - 64, 49152 + 64)
    got = wl.bits(C[:, cols].cpu().contiguous())
    rows = wl.choice_rows(M, 16, "cs.rows", edges=(0, 255, 256, M - 1))
    check.assert_bits_equal(got, ref.gemm_epilogue(A, B[cols].contiguous(), 1, rows=rows), rows="full", what="columns around the seam")
