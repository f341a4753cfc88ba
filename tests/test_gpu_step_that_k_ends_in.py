"""Direct kernels where K is no multiple of a step (128 bytes of a row): the last step ends where K does and reads some k twice,
which must count once, in every tile shape, type and layout."""
import pytest
import torch

from paper_2602_08043_amd.session import VerifiedGemm
from test_routes_cpu import DIRECT_16, DIRECT_32W, DIRECT_64, OWN32, TILED, route

pytestmark = pytest.mark.gpu
TORCH = {"f64": torch.float64, "f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16, "f8": torch.float8_e4m3fn,
         "f8e5m2": torch.float8_e5m2}
STEP = {"f64": 16, "f32": 32, "bf16": 64, "f16": 64, "f8": 128, "f8e5m2": 128}
# (rows, columns, steps), the kernels that these take in some type: one tile of each kind, few and many steps, K shared
SIZES = [(9, 70, 1), (16, 200, 5), (33, 64, 1), (65, 131, 2), (100, 190, 9), (40, 96, 40), (93, 345, 70), (1025, 2049, 1), (2049, 2049, 3),
         (1100, 1700, 14), (2048, 1024, 14), (4097, 2050, 2)]


def _sides(dtype, M, N, K, transB):
    g = torch.Generator(device="cuda").manual_seed(M + 3 * N + 7 * K)
    A = (torch.rand(M, K, generator=g, device="cuda") + 0.25).to(TORCH[dtype])
    B = (torch.rand((N, K) if transB else (K, N), generator=g, device="cuda") + 0.25).to(TORCH[dtype])
    return A, B


@pytest.mark.parametrize("dtype", list(STEP))
@pytest.mark.parametrize("transB", [0, 1])
def test_every_shape_and_remainder(dtype, transB):
    kernels, shared, step = set(), 0, STEP[dtype]
    u = 2.0 ** -53 if dtype == "f64" else 2.0 ** -24
    unit = {"f64": 0.0, "f32": 0.0, "bf16": 2.0 ** -8}.get(dtype, 2.0 ** -11)
    for M, N, steps in SIZES:
        for rest in (1, step // 2 + 1, step - 1):
            K = steps * step + rest
            r = route(dtype, M, N, K, transB)
            if r[2] == TILED:
                continue
            kernels.add(r[2])
            shared += r[3] > 1
            A, B = _sides(dtype, M, N, K, transB)
            # an infinity among the k that the last step reads again, a NaN behind them: in their row and column only, and
            # against positive numbers an infinity stays one
            A[M // 2, K - step] = float("inf") if dtype != "f8" else float("nan")  # (E4M3 has no infinity)
            B[(N // 2, K - 1) if transB else (K - 1, N // 2)] = float("nan")
            v = VerifiedGemm(M, N, K, dtype, transB)
            v.run_fused(A, B)
            C = v.C.double()
            bad = ~torch.isfinite(C)
            assert bool(bad[M // 2].all()) and bool(torch.isnan(C[:, N // 2]).all()), (dtype, M, N, K)
            if dtype != "f8":
                assert int(torch.isnan(C[M // 2]).sum()) == 1, (dtype, M, N, K)
            bad[M // 2], bad[:, N // 2] = False, False
            assert not bool(bad.any()), (dtype, M, N, K)
            # finite operands against FP64: sums of K terms, then one rounding
            A[M // 2, K - step] = 1.0
            B[(N // 2, K - 1) if transB else (K - 1, N // 2)] = 1.0
            v.run_fused(A, B)
            A64, B64 = A.double(), (B.double().t().contiguous() if transB else B.double())
            P = A64 @ B64
            bound = (K + 1) * u * (A64.abs() @ B64.abs()) * (2 if dtype == "f64" else 1)  # (FP64: the reference's rounding too)
            assert bool(((v.C.double() - P).abs() <= unit * P.abs() + bound).all()), (dtype, M, N, K)
            assert int(v.nflag.item()) == 0 and bool(((v.rowsum.double() - P.sum(1)).abs() <= v.T.double()).all()), (dtype, M, N, K)
    # (FP64 has no 64 x 64 tiles)
    assert shared > 0 and {DIRECT_16, DIRECT_32W, OWN32} | ({DIRECT_64} if dtype != "f64" else set()) <= kernels, (kernels, shared)
