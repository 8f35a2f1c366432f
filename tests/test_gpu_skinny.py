"""GEMMs of at most 64 rows against [N][K] weights (the kernel whose waves split K), at the edges of its row and column
tiles, of a 64-deep block and of the waves' turns, against the CPU oracle.  Small integers keep every sum exact, so equal
bits are demanded whatever the order of additions; activations are held to the usual tolerance."""
import pytest
import torch

import paper_2604_26666_amd as fact
import workloads as wl
from oracle import check, ref

pytestmark = pytest.mark.gpu


def run(A, W, bias=None, res=None, act=fact.ACT_NONE, f16=0, pad=0, out_f32=0, entry="gemm"):
    """Rows padded with NaN by `pad` elements on A and W and by `pad` + 1 on C; C's surroundings are checked."""
    dt = torch.float16 if f16 else torch.bfloat16
    (M, K), N = A.shape, W.shape[0]
    nout = N // 2 if act == fact.ACT_SILU_GATE else N

    def padded(t):
        buf = torch.full((t.shape[0], t.shape[1] + pad), float("nan"), dtype=dt, device="cuda")
        buf[:, : t.shape[1]] = t.cuda()
        return buf

    Ab, Wb, ldc = padded(A), padded(W), nout + (pad + 1 if pad else 0)
    Cb = torch.full((M + 1, ldc), 77.0, dtype=torch.float32 if out_f32 else dt, device="cuda")
    keep = [None if t is None else t.cuda() for t in (bias, res)]
    ep = fact.Epilogue(bias=keep[0], residual=keep[1], ldr=nout, act=act, f16=f16, out_f32=out_f32)
    if entry == "gemm":
        rc = fact.fact_gemm(M, N, K, Ab, K + pad, Wb, K + pad, 1, Cb, ldc, ep)
    else:
        need = max(fact.fact_gemm_splitk_workspace_bytes(M, N, K, 0), fact.fact_gemm_f32out_workspace_bytes(M, N, K, 0))
        ws = torch.full((need + 16,), 0xA5, dtype=torch.uint8, device="cuda")
        rc = fact.fact_gemm_splitk(M, N, K, Ab, K + pad, Wb, K + pad, 1, Cb, ldc, ep, 0, ws, need)
    fact.binding.check(rc, f"{(M, N, K)}")
    torch.cuda.synchronize()
    out = Cb.cpu()
    assert (out[M] == 77.0).all() and (out[:, nout:] == 77.0).all(), "wrote outside C"
    return out[:M, :nout].contiguous()


@pytest.mark.parametrize("f16", [0, 1])
@pytest.mark.parametrize("M", [1, 16, 17, 32, 33, 64])
@pytest.mark.parametrize("N,K,pad", [(1, 8, 0), (15, 64, 0), (17, 72, 8), (3080, 264, 0), (250, 1096, 8), (6160, 512, 0)])
def test_exact_sums(M, N, K, pad, f16):
    ints = wl.small_int_f16 if f16 else wl.small_int
    A, W = ints((M, K), -4, 4, f"sk.A.{M}.{K}"), ints((N, K), -4, 4, f"sk.W.{N}.{K}")
    bias, res = ints((N,), -9, 9, "sk.b"), ints((M, N), -9, 9, "sk.r")
    r = ref.gemm_epilogue(A, W, True, bias=bias, residual=res, fmt="f16" if f16 else "bf16")
    check.assert_bits_equal(wl.bits(run(A, W, bias, res, f16=f16, pad=pad)), r, what=f"{(M, N, K)}")


@pytest.mark.parametrize("act", [fact.ACT_GELU_TANH, fact.ACT_SILU_GATE])
@pytest.mark.parametrize("M", [3, 16, 31])
@pytest.mark.parametrize("N,K,pad", [(36, 200, 8), (3072, 768, 0), (34, 2056, 0)])
def test_activations(M, N, K, pad, act):
    A, W = wl.normal((M, K), 1.0, f"sk.a.{M}.{K}"), wl.normal((N, K), K ** -0.5, f"sk.w.{N}.{K}")
    check.assert_close(wl.bits(run(A, W, act=act, pad=pad)), ref.gemm_epilogue(A, W, True, act=act), what=f"{(M, N, K, act)}")


@pytest.mark.parametrize("N,K", [(17, 136), (128, 8192)])
def test_fp32_output_and_a_plan_that_splits_k(N, K):
    # integers: the fp32 result is the exact sum, with K whole and where the plan behind the call would split it
    A, W = wl.small_int((20, K), -3, 3, f"sk.fA.{K}"), wl.small_int((N, K), -3, 3, f"sk.fW.{N}.{K}")
    want = A.double() @ W.double().t()
    for entry in ("gemm", "splitk"):
        assert torch.equal(run(A, W, out_f32=1, entry=entry).double(), want), entry
    check.assert_bits_equal(wl.bits(run(A, W, entry="splitk")), ref.gemm_epilogue(A, W, True), what="splitk")


def test_workspace_is_asked_for_as_before():
    # a plan that splits K needs its workspace whatever kernel serves the call in the end
    M, N, K = 16, 128, 8192
    need = fact.fact_gemm_splitk_workspace_bytes(M, N, K, 0)
    assert need > 0
    A, W, C = (torch.zeros(s, dtype=torch.bfloat16, device="cuda") for s in ((M, K), (N, K), (M, N)))
    assert fact.fact_gemm_splitk(M, N, K, A, K, W, K, 1, C, N, None, 0, None, 0) == -6


def test_batches():
    A, W = wl.small_int((5, 9, 72), -4, 4, "sk.bA"), wl.small_int((5, 40, 72), -4, 4, "sk.bW")
    C = torch.zeros(5, 9, 40, dtype=torch.bfloat16, device="cuda")
    fact.binding.check(fact.fact_gemm_batched(5, 9, 40, 72, A.cuda(), 72, 9 * 72, W.cuda(), 72, 40 * 72, 1, C, 40, 360, None))
    torch.cuda.synchronize()
    for b in range(5):
        check.assert_bits_equal(wl.bits(C[b].cpu()), ref.gemm_epilogue(A[b], W[b], True), what=f"batch {b}")


@pytest.mark.parametrize("M,N,K,pad", [(1, 16, 16384 + 72, 8), (16, 64, 32768, 0), (33, 64, 16384 + 8, 0), (64, 100, 65536, 8)])
def test_long_k_and_few_columns(M, N, K, pad):
    # without a workspace the skinny kernel walks all of K; with one the plan splits K over the chip.  Both exact on integers
    A, W = wl.small_int((M, K), -2, 2, f"sk.lA.{M}.{K}"), wl.small_int((N, K), -2, 2, f"sk.lW.{N}.{K}")
    r = ref.gemm_epilogue(A, W, True)
    p = 1 << 16
    route = lambda ws, split: [x[0] for x in fact.fact_test_route(1, M, N, K, p, K + pad, 0, p, K + pad, 0, 1, p, N, 0, None, -1, split, 0, ws, 1 << 40)]
    assert route(None, 1) == ["skinny"] and route(p, 0) == ["tiles", "reduce"]
    for entry in ("gemm", "splitk"):
        check.assert_bits_equal(wl.bits(run(A, W, pad=pad, entry=entry)), r, what=f"{(M, N, K, entry)}")
