"""Outputs whose rows begin at any 2-byte address, through each tile of the main kernel: the store of a row at half a word passes
one element from lane to lane, so every place where that chain begins, is handed on or ends is held to the oracle, in interior and
edge tiles.  Integers of at most 4 keep every sum exact, so equal bits are demanded, and nothing beside C is written."""
import pytest
import torch

import paper_2604_26666_amd as fact
import workloads as wl
from oracle import check, ref

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pad,off", [(1, 0), (1, 1), (2, 1), (3, 0), (4, 1)])
@pytest.mark.parametrize("cfg", range(16))
def test_exact_sums(cfg, pad, off):
    bm, bn = fact.fact_config_info(cfg)[:2]
    # an interior tile, an edge tile whose last columns end `pad` short of and past a chunk of 8, rows past the last 16
    M, K = bm + 17 + pad, 128
    for nk in (0, 1) if 64 % (bn // 8) == 0 else (1,):
        N = 2 * bn - 32 + 8 * (pad & 1) + (pad if nk else 0)     # (as [K][N] it has to be a multiple of 8)
        ldc = N + 2 if nk else N + pad                           # odd for odd pads, even for even ones
        A = wl.small_int((M, K), -4, 4, f"or.A.{M}")
        B = wl.small_int((N, K) if nk else (K, N), -4, 4, f"or.B.{N}.{nk}")
        bias, res = wl.small_int((N,), -9, 9, "or.b"), wl.small_int((M, N), -9, 9, "or.r")
        Ad, Bd, bd, rd = A.cuda(), B.cuda(), bias.cuda(), res.cuda()
        for ep in (fact.Epilogue(), fact.Epilogue(bias=bd, residual=rd, ldr=N)):
            buf = torch.full(((M + 1) * ldc + off,), 77.0, dtype=torch.bfloat16, device="cuda")
            fact.binding.check(fact.fact_gemm_ex(1, M, N, K, Ad, K, 0, Bd, K if nk else N, 0, nk, buf.data_ptr() + 2 * off, ldc, 0, ep, cfg, 1, 0, None, 0), f"{(M, N, K, nk, cfg)}")
            torch.cuda.synchronize()
            out = buf.cpu()
            view = torch.as_strided(out, (M, N), (ldc, 1), off)
            got = wl.bits(view.clone())
            view.fill_(77.0)
            assert (out == 77.0).all(), "wrote outside C"
            rows = wl.choice_rows(M, 48, f"or.rows.{M}", edges=(0, 1, 15, 16, bm - 1, bm, M - 1))
            want = ref.gemm_epilogue(A, B, bool(nk), bias=bias if ep.bias is not None else None, residual=res if ep.residual is not None else None, rows=rows)
            check.assert_bits_equal(got, want, rows="full", what=f"{(M, N, K, ldc, nk, cfg)}")


@pytest.mark.parametrize("pad,odd,off", [(2, 1, 0), (2, 0, 1), (1, 0, 0)])          # entries at half a word in turn, all of them, rows in turn
@pytest.mark.parametrize("cfg", [0, 2, 6, 13, 15])
def test_batches(cfg, pad, odd, off):
    bm, bn = fact.fact_config_info(cfg)[:2]
    b, M, N, K = 3, bm + 17, bn + 24, 72
    A, B, res = wl.small_int((b, M, K), -4, 4, f"orb.A.{M}"), wl.small_int((b, N, K), -4, 4, f"orb.B.{N}"), wl.small_int((b, M, N), -9, 9, "orb.r")
    ldc = N + pad
    sc = M * ldc + (M * ldc + odd) % 2
    Ad, Bd, rd = A.cuda(), B.cuda(), res.cuda()
    buf = torch.full((b * sc + off,), 77.0, dtype=torch.bfloat16, device="cuda")
    ep = fact.Epilogue(residual=rd, ldr=N, stride_r=M * N)
    fact.binding.check(fact.fact_gemm_ex(b, M, N, K, Ad, K, M * K, Bd, K, N * K, 1, buf.data_ptr() + 2 * off, ldc, sc, ep, cfg, 1, 0, None, 0))
    torch.cuda.synchronize()
    out = buf.cpu()
    view = torch.as_strided(out, (b, M, N), (sc, ldc, 1), off)
    got = [wl.bits(view[z].clone()) for z in range(b)]
    view.fill_(77.0)
    assert (out == 77.0).all(), "wrote outside C"
    rows = wl.choice_rows(M, 48, f"orb.rows.{M}", edges=(0, 1, 15, 16, bm - 1, bm, M - 1))
    for z in range(b):
        check.assert_bits_equal(got[z], ref.gemm_epilogue(A[z], B[z], True, residual=res[z], rows=rows), rows="full", what=f"{(cfg, pad, odd, off, z)}")


def test_tail_split_after_full_rounds():
    # whole tiles on the lane chain, the shared tiles of the last round through the hand-over
    n, K, ldc = 64 * 24, 512, 64 * 24 + 1
    A, B = wl.small_int((n, K), -4, 4, "ort.A"), wl.small_int((n, K), -4, 4, "ort.B")
    need = fact.fact_gemm_splitk_workspace_bytes(n, n, K, -2)
    ws, buf = torch.empty(need, dtype=torch.uint8, device="cuda"), torch.full((n, ldc), 77.0, dtype=torch.bfloat16, device="cuda")
    assert fact.fact_test_route(1, n, n, K, A, K, 0, B, K, 0, 1, buf, ldc, 0, None, 6, -2, 0, ws, need) == [("tail", 6, n)]
    fact.binding.check(fact.fact_gemm_ex(1, n, n, K, A.cuda(), K, 0, B.cuda(), K, 0, 1, buf, ldc, 0, None, 6, -2, 0, ws, need))
    torch.cuda.synchronize()
    out = buf.cpu()
    assert (out[:, n] == 77.0).all(), "wrote outside C"
    rows = wl.choice_rows(n, 96, "ort.rows", edges=(0, 63, 64, n - 1))
    check.assert_bits_equal(wl.bits(out[:, :n].contiguous()), ref.gemm_epilogue(A, B, True, rows=rows), rows="full", what="tail split")
