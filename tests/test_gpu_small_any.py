"""Small outputs of operands of any alignment, on the kernel whose waves split K with one and two 16-wide tiles a side, and around
the line to the kernel of larger tiles, held to the CPU oracle where a tile, a 64-wide step, a wave's share of K or a piece of 8 ends.
Integers of at most 4 keep every sum exact in 32 bits, so equal bits are demanded; padding is NaN and must not be read."""
import pytest
import torch

import paper_2604_26666_amd as fact
import workloads as wl
from oracle import check, ref

pytestmark = pytest.mark.gpu

ONE_TILE = [(1, 14, 14), (16, 16, 63), (17, 15, 64), (15, 17, 65), (31, 9, 71), (33, 33, 127), (1, 34, 1917), (9, 83, 255), (5, 40, 257), (130, 48, 513), (273, 53, 777), (129, 513, 201), (129, 513, 511)]
TWO_TILES = [(116, 1179, 1441), (63, 2163, 1015), (700, 187, 705), (68, 1845, 493), (958, 2437, 73)]        # (the last two: waves of two blocks and of one at most)
# [K][N], [N][K]
AROUND = {(85, 469, 14): ("32x64/1", "1x1"), (311, 709, 783): ("32x64/4", "2x2"), (350, 1167, 1081): ("32x64/4",) * 2, (578, 2517, 21): ("64x64/1",) * 2,
          (1209, 2190, 589): ("128x128/2",) * 2}
FORMS = {**{s: ("1x1",) * 2 for s in ONE_TILE}, **{s: ("2x2",) * 2 for s in TWO_TILES}, **AROUND}


def odd(t, dt):
    """Rows of an odd length and entries of an odd stride from an odd element, everything between them NaN."""
    b, r, c = t.shape
    ld = c + 1 + c % 2
    stride = r * ld + 1 + (r * ld) % 2
    buf = torch.full((b * stride + 1,), float("nan"), dtype=dt, device="cuda")
    torch.as_strided(buf, (b, r, c), (stride, ld, 1), 1).copy_(t.cuda())
    return buf, buf.data_ptr() + 2, ld, stride


def run(A, B, nk, bias, res, f16, form, act=fact.ACT_NONE):
    dt = torch.float16 if f16 else torch.bfloat16
    (b, M, K), N = A.shape, B.shape[1] if nk else B.shape[2]
    nout = N // 2 if act == fact.ACT_SILU_GATE else N
    (Ab, ap, lda, sa), (Bb, bp, ldb, sb) = odd(A, dt), odd(B, dt)
    ldc = nout + 3
    sc = M * ldc + 1
    Cb = torch.full((b * sc + 1,), 77.0, dtype=dt, device="cuda")
    ep = fact.Epilogue(act=act, f16=f16)
    if bias is not None:
        bd, (Rb, rp, ldr, sr) = bias.cuda(), odd(res, dt)
        ep = fact.Epilogue(bias=bd, residual=rp, ldr=ldr, stride_r=sr, act=act, f16=f16)
    assert [(k, fact.RAGGED_FORMS[n]) for k, n, _ in fact.fact_test_route(b, M, N, K, ap, lda, sa, bp, ldb, sb, nk, Cb.data_ptr() + 2, ldc, sc, ep)] == [("ragged", form)]
    fact.binding.check(fact.fact_gemm_batched(b, M, N, K, ap, lda, sa, bp, ldb, sb, nk, Cb.data_ptr() + 2, ldc, sc, ep), f"{(b, M, N, K, nk)}")
    torch.cuda.synchronize()
    out = Cb.cpu()
    view = torch.as_strided(out, (b, M, nout), (sc, ldc, 1), 1)
    got = [wl.bits(view[z].clone()) for z in range(b)]
    view.fill_(77.0)
    assert (out == 77.0).all(), "wrote outside C"
    return got


@pytest.mark.parametrize("f16", [0, 1])
@pytest.mark.parametrize("nk", [0, 1])
@pytest.mark.parametrize("batch,shape", [(1, s) for s in FORMS] + [(3, (19, 35, 99))], ids=str)
def test_exact_sums_bias_and_residual(batch, shape, nk, f16):
    M, N, K = shape
    ints, fmt = (wl.small_int_f16, "f16") if f16 else (wl.small_int, "bf16")
    A, B = ints((batch, M, K), -4, 4, f"sa.A.{shape}"), ints((batch, N, K) if nk else (batch, K, N), -4, 4, f"sa.B.{shape}.{nk}")
    bias, res = ints((N,), -9, 9, "sa.bias"), ints((batch, M, N), -9, 9, f"sa.res.{shape}")
    rows = wl.choice_rows(M, 40, f"sa.rows.{shape}", edges=(0, min(15, M - 1), min(16, M - 1), min(31, M - 1), min(32, M - 1), M - 1))
    for z, got in enumerate(run(A, B, nk, bias, res, f16, FORMS.get(shape, ("1x1",) * 2)[nk])):
        want = ref.gemm_epilogue(A[z], B[z], bool(nk), bias=bias, residual=res[z], rows=rows, fmt=fmt)
        check.assert_bits_equal(got, want, rows="full", what=f"{shape} nk={nk} entry {z}")


@pytest.mark.parametrize("act,nk,f16", [(fact.ACT_SILU_GATE, 1, 0), (fact.ACT_SILU_GATE, 1, 1), (fact.ACT_GELU_TANH, 1, 1), (fact.ACT_GELU_TANH, 0, 0)])
@pytest.mark.parametrize("shape,form,gated", [((9, 82, 1443), "1x1", "32x64/4"), ((33, 66, 71), "1x1", "32x64/1"), ((116, 1178, 1441), "2x2", "32x64/4")], ids=str)
def test_activations(shape, form, gated, act, nk, f16):
    M, N, K = shape
    normal, fmt = (wl.normal_f16, "f16") if f16 else (wl.normal, "bf16")
    A, B = normal((1, M, K), 1.0, f"sa.a.{shape}"), normal((1, N, K) if nk else (1, K, N), K ** -0.5, f"sa.b.{shape}.{nk}")
    rows = wl.choice_rows(M, 32, f"sa.r.{shape}", edges=(0, M - 1))
    got = run(A, B, nk, None, None, f16, gated if act == fact.ACT_SILU_GATE else form, act)[0]
    check.assert_close(got, ref.gemm_epilogue(A[0], B[0], bool(nk), act=act, rows=rows, fmt=fmt), rows="full", what=f"{shape} act={act}")
