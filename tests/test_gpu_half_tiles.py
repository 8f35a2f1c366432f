"""The tiles of 64 x 128 and 128 x 64: whole and partial K steps around their four ring slots, edges of both sides, both layouts, K ranges,
and rows of C at any address, on small integers whose sums are exact."""
import pytest
import torch

import paper_2604_26666_amd as fact
import workloads as wl
from oracle import check, ref
import test_gpu_odd_rows_of_c as odd_rows
import test_gpu_ragged as ragged

pytestmark = pytest.mark.gpu
HALF = [16, 17]


@pytest.mark.parametrize("cfg", HALF)
def test_shape(cfg):
    assert sorted(fact.fact_config_info(cfg)[:2]) == [64, 128]


@pytest.mark.parametrize("split", [1, 3])
@pytest.mark.parametrize("K", [8, 64, 192, 256, 320, 840])
@pytest.mark.parametrize("cfg", HALF)
def test_exact_sums(cfg, K, split):
    bm, bn = fact.fact_config_info(cfg)[:2]
    if split > 1 and K < 192:
        pytest.skip("fewer K steps than ranges")
    ws = torch.empty(8 << 20, dtype=torch.uint8, device="cuda")
    for M, N in ((bm, bn), (2 * bm + 1, bn + 8), (bm - 1, 2 * bn - 8)):
        A = wl.small_int((M, K), -4, 4, f"ht.A.{M}.{K}")
        bias, res = wl.small_int((N,), -9, 9, f"ht.b.{N}"), wl.small_int((M, N), -9, 9, f"ht.r.{M}.{N}")
        for nk in (0, 1):
            B = wl.small_int((N, K) if nk else (K, N), -4, 4, f"ht.B.{N}.{K}.{nk}")
            C = torch.full((M + 1, N), 77.0, dtype=torch.bfloat16, device="cuda")
            bd, rd = bias.cuda(), res.cuda()
            fact.binding.check(fact.fact_gemm_ex(1, M, N, K, A.cuda(), K, 0, B.cuda(), K if nk else N, 0, nk, C, N, 0,
                                                 fact.Epilogue(bias=bd, residual=rd, ldr=N), cfg, split, 0, ws, 8 << 20))
            torch.cuda.synchronize()
            out = C.cpu()
            assert (out[M] == 77.0).all(), "wrote past C"
            check.assert_bits_equal(wl.bits(out[:M].contiguous()), ref.gemm_epilogue(A, B, bool(nk), bias=bias, residual=res), what=f"{(M, N, K, nk, cfg, split)}")


@pytest.mark.parametrize("pad,off", [(1, 0), (2, 1), (3, 0)])
@pytest.mark.parametrize("cfg", HALF)
def test_rows_of_c_at_any_address(cfg, pad, off):
    odd_rows.test_exact_sums(cfg, pad, off)


@pytest.mark.parametrize("act", [fact.ACT_GELU_TANH, fact.ACT_SILU_GATE])
@pytest.mark.parametrize("cfg", HALF)
def test_activations_on_odd_rows_of_c(cfg, act):
    ragged.test_activations_on_odd_rows_of_c_in_every_configuration(cfg, act)


@pytest.mark.parametrize("cfg", HALF)
def test_odd_rows_of_c_f16(cfg):
    ragged.test_odd_rows_of_c_in_every_configuration(cfg, 1)
