"""GEMMs on operands of any alignment (odd rows, widths that are no multiple of 8) on the matrix cores, held to the CPU
oracle at the sizes where a tile, a K step or a K group ends: small integers keep every sum exact, so equal bits are
demanded; the activations are held to the usual tolerance.  Padding is poisoned and must not be read."""
import numpy as np
import pytest
import torch

import paper_2604_26666_amd as fact
import workloads as wl
from oracle import check, ref

pytestmark = pytest.mark.gpu

# shape: what serves it with B as [K][N] and as [N][K].  Every tile and K-group count of the dispatch rule in both layouts; steps of K
# (64 wide, per group) that leave each remainder of the loop, which runs from 4 steps on: 1, 2, 3 steps without it, and with it an
# even count (2 left) and an odd one (3); 512 tiles of 128 x 128 and more, which keep one K group whatever K is
FORMS = {(601, 1003, 8): ("64x64/1",) * 2, (1003, 601, 9): ("64x64/1",) * 2, (700, 999, 100): ("64x64/1",) * 2, (700, 999, 150): ("64x64/1",) * 2,
         (700, 999, 201): ("64x64/1",) * 2, (700, 999, 300): ("64x64/2",) * 2, (700, 999, 777): ("64x64/2",) * 2, (900, 901, 600): ("64x64/2",) * 2,
         (1801, 1499, 77): ("128x128/1", "2x2"), (1801, 1499, 201): ("128x128/1",) * 2, (2000, 1999, 300): ("128x128/1",) * 2,
         (2900, 2901, 777): ("128x128/1",) * 2, (1801, 1499, 521): ("128x128/2",) * 2, (1801, 1499, 1000): ("128x128/2",) * 2,
         (500, 1200, 201): ("32x64/1",) * 2, (500, 1201, 300): ("32x64/1",) * 2, (400, 1001, 600): ("32x64/1",) * 2, (150, 2201, 77): ("32x64/1",) * 2,
         (350, 1167, 1081): ("32x64/4",) * 2, (401, 1001, 777): ("32x64/4",) * 2,
         (37, 131, 777): ("1x1",) * 2, (33, 65, 71): ("1x1",) * 2, (65, 64, 1025): ("1x1",) * 2, (1, 9, 8): ("guarded",) * 2, (31, 8, 9): ("guarded",) * 2}


def run(A, B, nk, bias=None, res=None, act=fact.ACT_NONE, f16=0, form=None):
    """Rows padded to odd lengths with NaN, pointers 2-byte aligned only; returns the bits of C after checking its surroundings."""
    dt = torch.float16 if f16 else torch.bfloat16

    def odd(t):
        r, c = t.shape
        ld = c + 1 if c % 2 == 0 else c + 2
        buf = torch.full((r * ld + 1,), float("nan"), dtype=dt, device="cuda")
        torch.as_strided(buf, (r, c), (ld, 1), 1).copy_(t.cuda())
        return buf, buf.data_ptr() + 2, ld

    (M, K), N = A.shape, B.shape[0] if nk else B.shape[1]
    nout = N // 2 if act == fact.ACT_SILU_GATE else N
    Ab, ap, lda = odd(A)
    Bb, bp, ldb = odd(B)
    ldc = nout + 3
    Cb = torch.full((M + 1, ldc), 77.0, dtype=dt, device="cuda")
    keep = [None if t is None else t.cuda() for t in (bias, res)]
    ep = fact.Epilogue(bias=keep[0], residual=keep[1], ldr=nout, act=act, f16=f16)
    (kind, n, _), = fact.fact_test_route(1, M, N, K, ap, lda, 0, bp, ldb, 0, nk, Cb, ldc, 0, ep)
    assert form is None or (fact.RAGGED_FORMS[n] if kind == "ragged" else kind) == form, (M, N, K, nk)
    fact.binding.check(fact.fact_gemm(M, N, K, ap, lda, bp, ldb, nk, Cb, ldc, ep), f"{(M, N, K, nk)}")
    torch.cuda.synchronize()
    out = Cb.cpu()
    assert (out[M] == 77.0).all() and (out[:, nout:] == 77.0).all(), "wrote outside C"
    return wl.bits(out[:M, :nout].contiguous())


@pytest.mark.parametrize("f16", [0, 1])
@pytest.mark.parametrize("nk", [0, 1])
@pytest.mark.parametrize("shape", FORMS, ids=str)
def test_exact_sums_bias_and_residual(shape, nk, f16):
    M, N, K = shape
    ints = wl.small_int_f16 if f16 else wl.small_int
    fmt = "f16" if f16 else "bf16"
    A, B = ints((M, K), -4, 4, f"rg.A.{shape}"), ints((N, K) if nk else (K, N), -4, 4, f"rg.B.{shape}.{nk}")
    bias, res = ints((N,), -9, 9, "rg.bias"), ints((M, N), -9, 9, "rg.res")
    rows = wl.choice_rows(M, 48, f"rg.rows.{shape}", edges=(0, 31, 32, 63, 64, 127, 128, M - 1))
    got = run(A, B, nk, bias, res, f16=f16, form=FORMS[shape][nk])
    check.assert_bits_equal(got, ref.gemm_epilogue(A, B, nk, bias=bias, residual=res, rows=rows, fmt=fmt), rows="full", what=f"{shape} nk={nk}")


@pytest.mark.parametrize("act", [fact.ACT_GELU_TANH, fact.ACT_SILU_GATE])
@pytest.mark.parametrize("shape,forms", [((1801, 1498, 521), ("128x128/2",) * 2), ((1801, 1498, 201), ("128x128/1",) * 2), ((700, 998, 300), ("64x64/2",) * 2),
                                         ((700, 998, 201), ("64x64/1",) * 2), ((400, 1000, 300), ("32x64/1",) * 2), ((401, 1002, 777), ("32x64/4",) * 2),
                                         ((37, 130, 777), ("1x1", "32x64/4")), ((33, 66, 71), ("1x1", "32x64/1"))], ids=str)
def test_activations(shape, forms, act):
    M, N, K = shape
    A, B = wl.normal((M, K), 1.0, f"rg.a.{shape}"), wl.normal((N, K), K ** -0.5, f"rg.b.{shape}")
    rows = wl.choice_rows(M, 32, f"rg.r.{shape}", edges=(0, M - 1))
    got = run(A, B, 1, act=act, form=forms[act == fact.ACT_SILU_GATE])
    check.assert_close(got, ref.gemm_epilogue(A, B, True, act=act, rows=rows), rows="full", what=f"{shape} act={act}")


@pytest.mark.parametrize("act,nk,f16", [(fact.ACT_SILU_GATE, 1, 1), (fact.ACT_GELU_TANH, 0, 0), (fact.ACT_GELU_TANH, 0, 1)])
@pytest.mark.parametrize("shape", [(700, 998, 300), (37, 130, 777)], ids=str)
def test_activations_in_fp16_and_with_row_major_weights(shape, act, nk, f16):
    M, N, K = shape
    normal, fmt = (wl.normal_f16, "f16") if f16 else (wl.normal, "bf16")
    A, B = normal((M, K), 1.0, f"rg.fa.{shape}"), normal((N, K) if nk else (K, N), K ** -0.5, f"rg.fb.{shape}.{nk}")
    rows = wl.choice_rows(M, 32, f"rg.fr.{shape}", edges=(0, M - 1))
    got = run(A, B, nk, act=act, f16=f16)
    check.assert_close(got, ref.gemm_epilogue(A, B, bool(nk), act=act, rows=rows, fmt=fmt), rows="full", what=f"{shape} act={act}")


@pytest.mark.parametrize("nk", [0, 1])
def test_batches_of_odd_strides(nk):
    # every operand of a batch entry begins at an odd element, rows and entries padded with NaN
    b, M, N, K = 3, 45, 71, 99
    A, B = wl.small_int((b, M, K), -4, 4, "rg.bA"), wl.small_int((b, N, K) if nk else (b, K, N), -4, 4, f"rg.bB.{nk}")
    bias, res = wl.small_int((N,), -9, 9, "rg.bb"), wl.small_int((b, M, N), -9, 9, "rg.br")

    def odd(t):
        r, c = t.shape[1:]
        ld = c + 1 + c % 2                                       # odd
        stride = r * ld + 1 + (r * ld) % 2                       # odd as well
        buf = torch.full((b * stride + 1,), float("nan"), dtype=torch.bfloat16, device="cuda")
        torch.as_strided(buf, (b, r, c), (stride, ld, 1), 1).copy_(t.cuda())
        return buf, buf.data_ptr() + 2, ld, stride

    (Ab, ap, lda, sa), (Bb, bp, ldb, sb), (Rb, rp, ldr, sr) = odd(A), odd(B), odd(res)
    ldc = N + 2
    sc = M * ldc + 1
    Cb = torch.full((b * sc + 1,), 77.0, dtype=torch.bfloat16, device="cuda")
    bd = bias.cuda()
    ep = fact.Epilogue(bias=bd, residual=rp, ldr=ldr, stride_r=sr)
    assert fact.fact_test_route(b, M, N, K, ap, lda, sa, bp, ldb, sb, nk, Cb.data_ptr() + 2, ldc, sc, ep)[0][0] == "ragged"
    fact.binding.check(fact.fact_gemm_batched(b, M, N, K, ap, lda, sa, bp, ldb, sb, nk, Cb.data_ptr() + 2, ldc, sc, ep))
    torch.cuda.synchronize()
    out = torch.as_strided(Cb, (b, M, N), (sc, ldc, 1), 1).cpu()
    for z in range(b):
        r = ref.gemm_epilogue(A[z], B[z], bool(nk), bias=bias, residual=res[z])
        check.assert_bits_equal(wl.bits(out[z].contiguous()), r, what=f"batch entry {z}")
    written = torch.zeros(Cb.numel(), dtype=torch.bool)
    torch.as_strided(written, (b, M, N), (sc, ldc, 1), 1).fill_(True)
    assert (Cb.cpu()[~written] == 77.0).all(), "wrote outside C"


def test_a_row_of_infinities_stays_in_its_row():
    # rows and columns past an edge repeat the last one and K past the end is zero on both sides: 0 x inf must not leak
    A, B = wl.small_int((65, 73), -4, 4, "rg.inf.A").clone(), wl.small_int((73, 67), 1, 4, "rg.inf.B")
    A[64] = float("inf")
    got = run(A, B, 0)
    check.assert_bits_equal(got, ref.gemm_epilogue(A, B, False, rows=np.arange(64)), rows="full", what="finite rows")
    assert (wl.from_bits(got[64:]).float() == float("inf")).all()      # B is positive: no inf - inf, and no 0 x inf from past K


@pytest.mark.parametrize("f16", [0, 1])
@pytest.mark.parametrize("cfg", range(16))
def test_odd_rows_of_c_in_every_configuration(cfg, f16):
    # aligned operands, C, bias and residual at odd addresses: interior tiles (unaligned register path), ragged edges
    tm, tn = fact.fact_config_info(cfg)[:2]
    M, N, K = 2 * tm + 9, 2 * tn + 13, 72
    ints, dt = (wl.small_int_f16, torch.float16) if f16 else (wl.small_int, torch.bfloat16)
    A, B = ints((M, K), -4, 4, f"rg.oA.{M}"), ints((N, K), -4, 4, f"rg.oB.{N}")
    bias, res = ints((N + 1,), -9, 9, "rg.ob"), ints((M, N), -9, 9, "rg.or")
    Cb = torch.full((M + 1, N + 2), 77.0, dtype=dt, device="cuda")
    bd, rd = bias.cuda(), res.cuda()
    ep = fact.Epilogue(bias=bd.data_ptr() + 2, residual=rd, ldr=N, f16=f16)
    fact.binding.check(fact.fact_gemm_ex(1, M, N, K, A.cuda(), K, 0, B.cuda(), K, 0, 1, Cb, N + 2, 0, ep, cfg, 1, 0, None, 0))
    torch.cuda.synchronize()
    out = Cb.cpu()
    assert (out[M] == 77.0).all() and (out[:, N:] == 77.0).all(), "wrote outside C"
    r = ref.gemm_epilogue(A, B, True, bias=bias[1:], residual=res, fmt="f16" if f16 else "bf16")
    check.assert_bits_equal(wl.bits(out[:M, :N].contiguous()), r, what=f"cfg {cfg}")


@pytest.mark.parametrize("act", [fact.ACT_GELU_TANH, fact.ACT_SILU_GATE])
@pytest.mark.parametrize("cfg", range(16))
def test_activations_on_odd_rows_of_c_in_every_configuration(cfg, act):
    # the same tiles with the activations, a residual at odd addresses, and edges of one row and of one column
    tm, tn = fact.fact_config_info(cfg)[:2]
    gated = act == fact.ACT_SILU_GATE
    for M, nout in ((tm + 1, (tn // 2 if gated else tn) + 1), (tm - 3, 2 * tn - 5)):
        N, K = 2 * nout if gated else nout, 72
        A, B = wl.normal((M, K), 1.0, f"rg.eA.{M}"), wl.normal((N, K), K ** -0.5, f"rg.eB.{N}")
        res, bias = wl.normal((M, nout + 1), 1.0, f"rg.er.{M}.{nout}"), None if gated else wl.normal((nout,), 1.0, f"rg.eb.{nout}")
        Cb = torch.full((M + 1, nout + 2), 77.0, dtype=torch.bfloat16, device="cuda")
        rd, bd = res.cuda(), None if bias is None else bias.cuda()
        ep = fact.Epilogue(bias=bd, residual=rd.data_ptr() + 2, ldr=nout + 1, act=act)
        fact.binding.check(fact.fact_gemm_ex(1, M, N, K, A.cuda(), K, 0, B.cuda(), K, 0, 1, Cb, nout + 2, 0, ep, cfg, 1, 0, None, 0))
        torch.cuda.synchronize()
        out = Cb.cpu()
        assert (out[M] == 77.0).all() and (out[:, nout:] == 77.0).all(), "wrote outside C"
        r = ref.gemm_epilogue(A, B, True, bias=bias, act=act, residual=res[:, 1:].contiguous())
        check.assert_close(wl.bits(out[:M, :nout].contiguous()), r, what=f"cfg {cfg} {M} x {nout}")


@pytest.mark.parametrize("nk", [0, 1])
def test_guarded_kernel_on_more_elements_than_a_grid_row_counts(nk):
    # one thread per element: 2^32 elements and more go into further rows of the grid.  Small integers, exact in bf16
    M, N, K = 65536 + 24, 65536 + 8, 3
    A, B = (torch.randint(-4, 5, s, device="cuda").bfloat16() for s in ((M, K), (N, K) if nk else (K, N)))
    C = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    p = fact.fact_test_route(1, M, N, K, A, K, 0, B, K if nk else N, 0, nk, C, N, 0, None)
    assert [x[0] for x in p] == ["guarded"]
    fact.binding.check(fact.fact_gemm(M, N, K, A, K, B, K if nk else N, nk, C, N, None))
    torch.cuda.synchronize()
    Bk = (B.t() if nk else B).float()
    for a, c in zip(A.split(8192), C.split(8192)):
        want = sum(a[:, k:k + 1].float() * Bk[k:k + 1] for k in range(K))
        assert torch.equal(c.float(), want)
