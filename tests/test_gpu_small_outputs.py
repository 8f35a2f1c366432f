"""Small outputs of either layout of B on the kernel whose waves split K: every tile that the rule can choose, at the edges of
its rows and columns, of the 64-deep blocks and of the waves' turns, against the CPU oracle.  Small integers keep every sum
exact, so equal bits are demanded whatever the order of additions."""
import pytest
import torch

import paper_2604_26666_amd as fact
import workloads as wl
from oracle import check, ref

P = 1 << 16


def route(M, N, K, nk, batch=1, **ep):
    return [x[0] for x in routes(M, N, K, nk, batch, **ep)]


def routes(M, N, K, nk, batch=1, **ep):
    return fact.fact_test_route(batch, M, N, K, P, K, M * K, P, K if nk else N, K * N, nk, P, N, M * N, fact.Epilogue(**ep))


# (M, N, K, B as [N][K], form): the tile in 16 x 16 and the LDS stages of a wave that the rule takes for these sizes
CASES = [(1, 8, 8, 0, "1x1/4"), (5, 216, 264, 0, "1x1/4"), (22, 168, 424, 0, "1x1/4"), (33, 40, 1480, 0, "1x1/4"),
         (7, 480, 72, 0, "2x2/2"), (65, 1000, 136, 0, "2x2/2"), (26, 2184, 64, 0, "2x2/2"), (33, 40, 8, 0, "1x4/3"),
         (42, 152, 96, 0, "1x2/4"), (24, 752, 168, 0, "1x2/4"), (24, 1728, 328, 0, "1x2/4"),
         (9, 104, 16, 0, "1x4/3"), (5, 344, 48, 0, "1x4/3"), (198, 312, 8, 0, "1x4/3"),
         (103, 8, 16, 1, "1x1/4"), (131, 33, 24, 1, "1x1/4"), (56, 137, 1160, 1, "1x1/4"),
         (273, 23, 24, 1, "2x1/3"), (26, 345, 112, 1, "2x1/3"), (54, 961, 352, 1, "4x1/2"), (126, 525, 1896, 1, "2x1/3"),
         (138, 1121, 8, 1, "2x2/2"), (26, 2705, 104, 1, "2x1/3"), (58, 2547, 1840, 1, "2x2/2"), (300, 481, 584, 1, "2x2/2"), (512, 512, 512, 0, "2x2/2"),
         (96, 1535, 2056, 1, "2x2/3"), (62, 2043, 2048, 1, "2x2/3")]         # (two blocks ahead)


@pytest.mark.parametrize("M,N,K,nk,form", CASES, ids=str)
def test_route(M, N, K, nk, form):
    assert [(k, fact.SKINNY_FORMS[n]) for k, n, _ in routes(M, N, K, nk)] == [("skinny", form)]


def test_where_the_tile_kernel_stays():
    # many columns, a B that only memory delivers, an output that fills the chip, a gated call, more work-groups than fit at once
    assert route(159, 5840, 928, 0) == ["tiles"] and route(3, 7856, 4152, 0) == ["tiles"] and route(572, 1552, 2128, 1) == ["tiles"]
    assert route(16, 16384, 256, 0) == ["tiles"] and route(300, 480, 584, 1, act=fact.ACT_SILU_GATE) == ["tiles"]
    assert route(128, 128, 64, 0, batch=64) == ["tiles"] and route(128, 128, 64, 0, batch=4) == ["skinny"]


@pytest.mark.gpu
@pytest.mark.parametrize("f16", [0, 1])
@pytest.mark.parametrize("M,N,K,nk,form", CASES, ids=str)
def test_exact_sums(M, N, K, nk, form, f16):
    dt, ints = (torch.float16, wl.small_int_f16) if f16 else (torch.bfloat16, wl.small_int)
    A, B = ints((M, K), -4, 4, f"so.A.{M}.{K}"), ints((N, K) if nk else (K, N), -4, 4, f"so.B.{N}.{K}")
    bias, res = ints((N,), -9, 9, "so.b"), ints((M, N), -9, 9, "so.r")
    want = ref.gemm_epilogue(A, B, bool(nk), bias=bias, residual=res, fmt="f16" if f16 else "bf16")
    for pad in (0, 8):                               # rows followed by NaN: nothing outside the matrices may reach a sum

        def padded(t):
            buf = torch.full((t.shape[0] + 1, t.shape[1] + pad), float("nan"), dtype=dt, device="cuda")
            buf[:-1, : t.shape[1]] = t.cuda()
            return buf

        Ab, Bb, R = padded(A), padded(B), padded(res)
        C = torch.full((M + 1, N + pad + 1), 77.0, dtype=dt, device="cuda")
        bd = bias.cuda()
        ep = fact.Epilogue(bias=bd, residual=R, ldr=N + pad, f16=f16)
        fact.binding.check(fact.fact_gemm(M, N, K, Ab, K + pad, Bb, (K if nk else N) + pad, nk, C, N + pad + 1, ep))
        torch.cuda.synchronize()
        out = C.cpu()
        assert (out[M] == 77.0).all() and (out[:, N:] == 77.0).all(), "wrote outside C"
        check.assert_bits_equal(wl.bits(out[:M, :N].contiguous()), want, what=f"{(M, N, K, nk, pad)}")


@pytest.mark.gpu
@pytest.mark.parametrize("nk", [0, 1])
def test_batches_and_activation(nk):
    b, M, N, K = 5, 70, 72, 200
    assert route(M, N, K, nk, batch=b, act=fact.ACT_GELU_TANH) == ["skinny"]
    A, B = wl.normal((b, M, K), 1.0, "so.bA"), wl.normal((b, N, K) if nk else (b, K, N), K ** -0.5, f"so.bB{nk}")
    Ad, Bd, C = A.cuda(), B.cuda(), torch.zeros(b, M, N, dtype=torch.bfloat16, device="cuda")
    ep = fact.Epilogue(act=fact.ACT_GELU_TANH)
    fact.binding.check(fact.fact_gemm_batched(b, M, N, K, Ad, K, M * K, Bd, K if nk else N, K * N, nk, C, N, M * N, ep))
    torch.cuda.synchronize()
    for i in range(b):
        check.assert_close(wl.bits(C[i].cpu()), ref.gemm_epilogue(A[i], B[i], bool(nk), act=fact.ACT_GELU_TANH), what=f"batch {i}")


@pytest.mark.gpu
def test_weights_past_the_line_of_streaming_loads():
    # 64 MB of [N][K] weights and less, and more: the same kernel with either cache policy
    for N in (4096, 4097):
        A, W = wl.small_int((3, 8192), -2, 2, "so.sA"), wl.small_int((N, 8192), -2, 2, f"so.sW{N}")
        C = torch.zeros(3, N, dtype=torch.bfloat16, device="cuda")
        fact.binding.check(fact.fact_gemm(3, N, 8192, A.cuda(), 8192, W.cuda(), 8192, 1, C, N, None))
        torch.cuda.synchronize()
        check.assert_bits_equal(wl.bits(C.cpu()), ref.gemm_epilogue(A, W, True), what=str(N))
