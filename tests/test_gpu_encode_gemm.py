"""vabft_encode_gemm_fused against vabft_encode and vabft_gemm_verified_fused: the same bits, and S1..S3, whichever
launch folds them: the direct kernels', the tiled kernels', the one that copies operands, the fold of its own."""
import pytest
import torch

from paper_2602_08043_amd.session import VerifiedGemm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,M,N,K,transB", [
    ("f32", 256, 256, 256, 0), ("bf16", 90, 840, 840, 1), ("f64", 33, 200, 130, 0),  # A-side pass in the direct launch
    ("f32", 8192, 64, 256, 0),                       # more rows than that takes: fold and pass of their own
    ("bf16", 2048, 2048, 1024, 0), ("f16", 1000, 3072, 1024, 1), ("f8", 2048, 2048, 2048, 1),  # tiled kernels
    ("bf16", 2048, 2048, 1000, 0),                   # tiled kernel, pass of its own
    ("bf16", 3001, 1873, 5001, 0)])                  # copies
def test_same_bits_as_two_calls(dtype, M, N, K, transB):
    td = {"f32": torch.float32, "f64": torch.float64, "bf16": torch.bfloat16, "f16": torch.float16,
          "f8": torch.float8_e4m3fn}[dtype]
    g = torch.Generator().manual_seed(3)
    A = torch.randn(M, K, generator=g).to(td).cuda()
    B = torch.randn((N, K) if transB else (K, N), generator=g).to(td).cuda()
    one, two = VerifiedGemm(M, N, K, dtype, transB), VerifiedGemm(M, N, K, dtype, transB)
    for defer in (False, True):
        two.encode(B)  # for S
        S = two.S.clone()
        two.encode(B, defer_S=True)
        two.gemm_fused(A, B, deferred_S=True)
        one.S.fill_(-1.0)
        one.run_fused(A, B, defer_S=defer)
        torch.cuda.synchronize()
        assert int(one.nflag.item()) == 0
        if defer:
            assert bool((one.S == -1.0).all())  # left alone
        else:  # K sums of terms of one sign, in groups that differ with the encode's workgroups
            assert bool(((one.S - S).abs() <= K * 2.0 ** -53 * S).all())
        for n in ("Be", "bstat", "astat", "expected", "T", "rowsum", "E", "flags", "nflag", "C"):
            assert torch.equal(getattr(one, n), getattr(two, n)), (n, defer)


@pytest.mark.parametrize("dtype,M,N,K,transB", [
    ("f16", 1000, 3072, 1024, 1), ("bf16", 2048, 2048, 1024, 0), ("bf16", 1499, 2496, 1504, 1), ("f16", 2305, 2048, 1096, 0),
    ("bf16", 2304, 3840, 512, 0), ("bf16", 1793, 4352, 1032, 0)])
def test_pass_on_units_without_a_tile(dtype, M, N, K, transB):
    """The A-side pass behind the tiles of the 16-bit kernels (whole and ragged tiles, any K): the bits of vabft_threshold, and
    its checks see what the three calls see."""
    td = {"bf16": torch.bfloat16, "f16": torch.float16}[dtype]
    g = torch.Generator().manual_seed(4)
    A = torch.randn(M, K, generator=g).to(td).cuda()
    B = torch.randn((N, K) if transB else (K, N), generator=g).to(td).cuda()
    one, three = VerifiedGemm(M, N, K, dtype, transB), VerifiedGemm(M, N, K, dtype, transB)
    for e_max in (None, 1e-30, None):  # (1e-30: what rounding leaves of a row flags it)
        three.encode(B)
        three.threshold(A, e_max)
        three.gemm(A, B)
        one.encode(B)
        one.gemm_fused(A, B, e_max)
        torch.cuda.synchronize()
        for n in ("astat", "expected", "T", "rowsum", "E", "flags", "nflag", "C"):
            assert torch.equal(getattr(one, n), getattr(three, n)), (n, e_max)
        assert (int(one.nflag.item()) > 0) == (e_max is not None)
