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
