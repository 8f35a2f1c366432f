"""Split-K reductions whose count of K ranges leaves every remainder of the batches in which they are loaded, with bias and
residual that can and cannot be loaded four at a time.  Small integers: equal bits whatever the order of additions."""
import pytest
import torch

import workloads as wl
from gpu_util import gemm
from oracle import check, ref

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,trans_b", [(3, 64, 0), (65, 36, 1), (33, 1000, 1)])
@pytest.mark.parametrize("split", [2, 3, 5, 6, 7, 8, 11, 15, 33])
def test_every_remainder(M, N, trans_b, split):
    K = 64 * split
    A, B = wl.small_int((M, K), -3, 3, f"rd.A.{M}.{K}"), wl.small_int((N, K) if trans_b else (K, N), -3, 3, f"rd.B.{N}.{K}")
    bias, res = wl.small_int((N,), -9, 9, "rd.b"), wl.small_int((M, N), -9, 9, "rd.r")
    want = ref.gemm_epilogue(A, B, bool(trans_b), bias=bias, residual=res)
    for pad in (0, 8):
        got = gemm(A, B, trans_b, bias=bias, residual=res, split=split, pad=pad)
        check.assert_bits_equal(got, want, what=f"{(M, N, K, split, pad)}")
