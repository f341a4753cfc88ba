"""vabft_encode_gemm_weighted against the four calls that it stands for, bit by bit.  Thresholds of nearly nothing flag what
rounding leaves of every row, so that rows are localised, corrected and counted without the injector (which takes the four
calls)."""
import ctypes

import pytest
import torch

from paper_2602_08043_amd import binding as vb
from paper_2602_08043_amd.session import VerifiedGemm
from test_routes_cpu import DIRECT_16, DIRECT_32, DIRECT_32W, DIRECT_64, route

pytestmark = pytest.mark.gpu
TORCH = {"f64": torch.float64, "f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16,
         "f8": torch.float8_e4m3fn, "f8e5m2": torch.float8_e5m2}
NAMES = ("Be", "Be2", "bstat", "astat", "expected", "expected2", "T", "rowsum", "rowsum2", "E", "flags", "nflag", "loc",
         "delta", "ncorrected", "C")


@pytest.mark.parametrize("dtype,M,N,K,transB", [
    ("bf16", 1024, 1024, 1024, 0), ("bf16", 7, 100, 300, 1), ("f32", 256, 100, 300, 1), ("f32", 250, 64, 96, 0),
    ("f64", 40, 63, 100, 0), ("f64", 300, 130, 64, 1), ("f8", 33, 96, 80, 0), ("f8e5m2", 16, 64, 256, 1),
    ("f16", 5000, 64, 64, 0), ("f16", 5000, 320, 64, 1),   # counters shared by tile-rows, and one each
    ("bf16", 100, 101, 64, 1), ("f16", 64, 66, 64, 0),     # rows of C that are not at whole 8 bytes: localised by a launch
    ("f32", 2000, 3000, 64, 0), ("bf16", 2048, 2048, 1024, 0), ("bf16", 8192, 64, 1024, 0),  # so these, of many tiles
    ("f32", 93, 345, 5527, 0), ("bf16", 78, 192, 6871, 0)])  # K shared by workgroups
def test_same_bits_as_four_calls(dtype, M, N, K, transB):
    td = TORCH[dtype]
    g = torch.Generator().manual_seed(7)
    A = torch.randn(M, K, generator=g).to(td).cuda()
    B = torch.randn((N, K) if transB else (K, N), generator=g).to(td).cuda()
    one, four = VerifiedGemm(M, N, K, dtype, transB), VerifiedGemm(M, N, K, dtype, transB)
    seen = 0
    for e_max, correct in ((None, 1), (1e-30, 1), (1e-30, 0), (None, 1)):
        one.run_weighted(A, B, e_max, correct=correct)
        four.encode_weighted(B)
        torch.cuda.synchronize()
        # K sums of terms of one sign, which fold in another grouping where K has many rows; T as it follows from the same
        assert bool(((one.S - four.S).abs() <= K * 2.0 ** -53 * four.S).all()), (e_max, correct)
        four.S.copy_(one.S)
        four.threshold_weighted(A, e_max)
        four.gemm_weighted(A, B)
        four.locate_correct(correct)
        torch.cuda.synchronize()
        for n in NAMES:
            x, y = getattr(one, n), getattr(four, n)
            assert torch.equal(x, y), (n, e_max, correct)
        if e_max is None:
            assert int(one.nflag.item()) == 0 and int(one.ncorrected.item()) == 0
        else:
            seen += int(one.ncorrected.item())
            assert int(one.nflag.item()) > 0
    assert seen > 0 or M < 64


# (tiles of 16 rows, of 32 by eight and by four wavefronts, of 64; K shared; columns that end inside a tile)
CORRECTED = [("bf16", 16, 200, 512, 0, DIRECT_16), ("f16", 16, 128, 512, 1, DIRECT_16), ("f8", 16, 136, 512, 0, DIRECT_16),
             ("f8e5m2", 16, 128, 512, 1, DIRECT_16), ("bf16", 17, 36, 2112, 1, DIRECT_32), ("bf16", 300, 192, 512, 1, DIRECT_32W), ("f16", 300, 204, 512, 0, DIRECT_32W),
             ("f8", 300, 204, 512, 1, DIRECT_32W), ("f8e5m2", 300, 128, 512, 0, DIRECT_32W), ("bf16", 1700, 516, 1024, 0, DIRECT_64),
             ("f16", 1024, 1024, 2048, 1, DIRECT_64), ("f8", 1700, 516, 2048, 0, DIRECT_64), ("f8e5m2", 1700, 512, 2048, 1, DIRECT_64)]
SHARED = [("bf16", 78, 192, 6912, 0, None), ("f16", 40, 200, 6144, 1, None), ("f8", 48, 128, 8192, 1, None),
          ("f8e5m2", 40, 132, 8192, 0, None)]


@pytest.mark.parametrize("dtype,M,N,K,transB,kernel", CORRECTED + SHARED)
def test_correction_of_stored_elements(dtype, M, N, K, transB, kernel):
    """Large terms that cancel along K leave the row sums and the expected ones apart by more than the last place of C's elements:
    what the launch corrects changes in memory, and nothing else does."""
    r = route(dtype, M, N, K, transB, more_sums=1)
    assert r[2] == kernel if kernel is not None else r[3] > 1, r
    h = (K - 64) // 2
    big = {"bf16": (2.0 ** 14, 1.0), "f16": (2.0 ** 12, 4.0), "f8": (128.0, 64.0), "f8e5m2": (2.0 ** 10, 16.0)}[dtype]
    g = torch.Generator().manual_seed(11)
    P = torch.randn(M, h, generator=g) * big[0] * 0.25
    Q = torch.randn(h, N, generator=g) * big[1]
    A = torch.cat([P, -P, torch.randn(M, K - 2 * h, generator=g)], 1).to(TORCH[dtype]).cuda()
    B = torch.cat([Q, Q, torch.randn(K - 2 * h, N, generator=g)], 0).to(TORCH[dtype])
    B = (B.t().contiguous() if transB else B).cuda()
    one, four = VerifiedGemm(M, N, K, dtype, transB), VerifiedGemm(M, N, K, dtype, transB)
    f = vb.load().vabft_internal_locates
    f.restype, f.argtypes = ctypes.c_int32, [ctypes.POINTER(vb.Problem)] + [ctypes.c_void_p] * 3 + [ctypes.c_size_t]
    assert f(one.problem, A.data_ptr(), B.data_ptr(), one.C.data_ptr(), one.ws_bytes) == 1
    one.run_weighted(A, B, 1e-30, correct=0)
    stored = one.C.clone()
    assert int(one.ncorrected.item()) == 0
    one.run_weighted(A, B, 1e-30, correct=1)
    four.encode_weighted(B)
    four.S.copy_(one.S)
    four.threshold_weighted(A, 1e-30)
    four.gemm_weighted(A, B)
    assert torch.equal(four.C, stored)
    four.locate_correct(1)
    torch.cuda.synchronize()
    for n in NAMES:
        assert torch.equal(getattr(one, n), getattr(four, n)), n
    rows = torch.nonzero(one.loc >= 0).flatten()
    assert rows.numel() == int(one.ncorrected.item()) and rows.numel() > 0
    at = torch.zeros_like(stored, dtype=torch.bool)
    at[rows, one.loc[rows].long()] = True
    changed = one.C != stored
    assert not bool((changed & ~at).any())
    # of the located elements all whose correction is more than their last place
    x, by = stored[rows, one.loc[rows].long()].double(), one.delta[rows].double()
    must = by.abs() > x.abs() * 2.0 ** (-7 if dtype == "bf16" else -10) + 2.0 ** -24
    assert bool(must.any()) and bool(changed[rows, one.loc[rows].long()][must].all()), (int(must.sum()), rows.numel())


def test_inf_and_nan_rows():
    M, N, K = 70, 128, 96
    g = torch.Generator().manual_seed(9)
    A, B = torch.randn(M, K, generator=g).cuda(), torch.randn(K, N, generator=g).cuda()
    A[3, 5], A[40, 0] = float("nan"), float("inf")
    v = VerifiedGemm(M, N, K, "f32", 0)
    v.run_weighted(A, B)
    torch.cuda.synchronize()
    assert torch.nonzero(v.flags).flatten().tolist() == [3, 40]
    assert v.loc[[3, 40]].tolist() == [-2, -2] and int(v.ncorrected.item()) == 0 and int(v.nflag.item()) == 2
