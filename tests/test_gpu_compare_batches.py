"""The compare at the end of a direct kernel's launch reads a row's partials in batches whose size goes with their number:
row sums, weighted row sums and flags on both sides of every change of batch."""
import numpy as np
import pytest
import torch

from paper_2602_08043_amd.session import VerifiedGemm

pytestmark = pytest.mark.gpu

# tile-columns at 64 columns each (16 rows of a K x N B: 32 groups of threads; 32 rows: 8), for 2, 8 and 24 loads to a batch
COLS = {16: [63, 64, 65, 128], 32: [15, 16, 17, 63, 64, 65, 172], 64: [7, 8, 9, 33]}


@pytest.mark.parametrize("dtype,M,transB", [("f32", 32, 1), ("f32", 70, 0), ("bf16", 16, 0), ("bf16", 33, 1), ("f64", 40, 0),
                                            ("f64", 9, 0), ("f8", 16, 0), ("f32", 3, 0)])
def test_rowsums_at_every_batch(dtype, M, transB):
    td = {"f32": torch.float32, "f64": torch.float64, "bf16": torch.bfloat16, "f8": torch.float8_e4m3fn}[dtype]
    K, u = 40, 2.0 ** -53 if dtype == "f64" else 2.0 ** -24
    g = torch.Generator().manual_seed(5)
    for cols in COLS[16 if M <= 16 else 32 if M <= 32 else 64]:
        for N in (64 * cols, 64 * cols - 5):
            A = torch.randn(M, K, generator=g, dtype=torch.float64).to(td)
            B = torch.randn((N, K) if transB else (K, N), generator=g, dtype=torch.float64).to(td)
            v = VerifiedGemm(M, N, K, dtype, transB)
            Ad, Bd = A.cuda(), B.cuda()
            A64, B64 = A.double(), (B.double().t() if transB else B.double())
            w = torch.arange(1, N + 1, dtype=torch.float64)
            C = A64 @ B64
            # every sum of n terms in floating point is within (n - 1) u (1 + O(u)) of the sum of their magnitudes
            bound = 1.01 * (K + N) * u * (A64.abs() @ B64.abs())
            want = {"rowsum": (C.sum(1), bound.sum(1)), "rowsum2": (C @ w, 2 * (bound @ w))}
            v.run_fused(Ad, Bd)
            torch.cuda.synchronize()
            assert int(v.nflag.item()) == 0
            err = (v.rowsum.cpu().double() - want["rowsum"][0]).abs()
            assert bool((err <= want["rowsum"][1]).all()), (dtype, M, N, float((err / want["rowsum"][1]).max()))
            v.run_weighted(Ad, Bd, correct=0)
            torch.cuda.synchronize()
            for k in ("rowsum", "rowsum2"):
                err = (getattr(v, k).cpu().double() - want[k][0]).abs()
                assert bool((err <= want[k][1]).all()), (dtype, M, N, k, float((err / want[k][1]).max()))
            # one fault in the first, one in the last tile-column: their rows are flagged, no others
            top = 62 if dtype == "f64" else 30
            v.run_fused(Ad, Bd, inj=v.make_inject(mode=1, faults=[(0, 0, top), (M - 1, N - 1, top)]))
            torch.cuda.synchronize()
            assert np.array_equal(np.flatnonzero(v.flags.cpu().numpy()), sorted({0, M - 1}))
            assert int(v.nflag.item()) == len({0, M - 1})
