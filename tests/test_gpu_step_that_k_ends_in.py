"""Direct kernels where K is no multiple of a step (128 bytes of a row): the last step ends where K does and reads some k twice,
which must count once, in every tile shape, type and layout."""
import pytest
import torch

from paper_2602_08043_amd import binding as vb
from paper_2602_08043_amd.session import VerifiedGemm
from test_routes_cpu import DIRECT_16, DIRECT_32, DIRECT_32W, DIRECT_64, DIRECT_ANY, OWN32, OWN64, TILED, route

pytestmark = pytest.mark.gpu
TORCH = {"f64": torch.float64, "f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16, "f8": torch.float8_e4m3fn,
         "f8e5m2": torch.float8_e5m2}
STEP = {"f64": 16, "f32": 32, "bf16": 64, "f16": 64, "f8": 128, "f8e5m2": 128}
# (rows, columns, steps), the kernels that these take in some type: one tile of each kind, few and many steps, K shared
SIZES = [(9, 70, 1), (16, 200, 5), (33, 64, 1), (65, 131, 2), (100, 190, 9), (40, 96, 40), (93, 345, 70), (1025, 2049, 1), (2049, 2049, 3),
         (1100, 1700, 14), (2048, 1024, 14), (4097, 2050, 2), (2790, 2065, 1), (18, 48, 14), (19, 2393, 15), (2337, 30, 23), (17, 4202, 18),
         (1102, 68, 16), (17, 2649, 29), (1381, 32, 33), (35, 2144, 37), (37, 2783, 34), (33, 2957, 74), (2930, 30, 78)]


def _sides(dtype, M, N, K, transB):
    g = torch.Generator(device="cuda").manual_seed(M + 3 * N + 7 * K)
    A = (torch.rand(M, K, generator=g, device="cuda") + 0.25).to(TORCH[dtype])
    B = (torch.rand((N, K) if transB else (K, N), generator=g, device="cuda") + 0.25).to(TORCH[dtype])
    return A, B


def _check(dtype, M, N, K, transB, A, B, v, product, verified):
    """product(): one pass over A and B, which change in between, to v.C."""
    step, u = STEP[dtype], 2.0 ** -53 if dtype == "f64" else 2.0 ** -24
    unit = {"f64": 0.0, "f32": 0.0, "bf16": 2.0 ** -8}.get(dtype, 2.0 ** -11)
    # an infinity among the k that the last step reads again, a NaN behind them: in their row and column only, and
    # against positive numbers an infinity stays one
    last = (N // 2, K - 1) if transB else (K - 1, N // 2)
    A[M // 2, K - step] = float("inf") if dtype != "f8" else float("nan")  # (E4M3 has no infinity)
    B[last] = float("nan")
    product()
    C = v.C.double()
    bad = ~torch.isfinite(C)
    assert bool(bad[M // 2].all()) and bool(torch.isnan(C[:, N // 2]).all()), (dtype, M, N, K)
    if dtype != "f8":
        assert int(torch.isnan(C[M // 2]).sum()) == 1, (dtype, M, N, K)
    bad[M // 2], bad[:, N // 2] = False, False
    assert not bool(bad.any()), (dtype, M, N, K)
    # finite operands against FP64: sums of K terms, then one rounding
    A[M // 2, K - step] = 1.0
    B[last] = 1.0
    product()
    A64, B64 = A.double(), (B.double().t().contiguous() if transB else B.double())
    P = A64 @ B64
    bound = (K + 1) * u * (A64.abs() @ B64.abs()) * (2 if dtype == "f64" else 1)  # (FP64: the reference's rounding too)
    assert bool(((v.C.double() - P).abs() <= unit * P.abs() + bound).all()), (dtype, M, N, K)
    if verified:
        assert int(v.nflag.item()) == 0 and bool(((v.rowsum.double() - P.sum(1)).abs() <= v.T.double()).all()), (dtype, M, N, K)


@pytest.mark.parametrize("dtype", list(STEP))
@pytest.mark.parametrize("transB", [0, 1])
def test_every_shape_and_remainder(dtype, transB):
    kernels, shared, step = set(), set(), STEP[dtype]
    for M, N, steps in SIZES:
        for rest in (1, step // 2 + 1, step - 1):
            K = steps * step + rest
            kernel, split = route(dtype, M, N, K, transB)[2:4]
            # (without a workspace a call keeps its tiles and no two workgroups share one)
            unshared = route(dtype, M, N, K, transB, room=0)[2]
            if kernel == TILED:
                continue
            A, B = _sides(dtype, M, N, K, transB)
            v = VerifiedGemm(M, N, K, dtype, transB)
            kernels.add(kernel)
            if split > 1:
                shared.add(kernel)
            _check(dtype, M, N, K, transB, A, B, v, lambda: v.run_fused(A, B), True)
            if unshared == DIRECT_32:
                kernels.add(unshared)
                none = [None] * 6
                _check(dtype, M, N, K, transB, A, B, v, lambda: vb.vabft_gemm_verified(
                    v.problem, A.data_ptr(), B.data_ptr(), v.C, None, None, 0, None, *none, None, 0, v._stream()), False)
    # (FP64 has no tiles of 64 rows)
    assert kernels == {DIRECT_16, DIRECT_32, DIRECT_32W, OWN32} | ({DIRECT_64, OWN64} if dtype != "f64" else set()), kernels
    assert {DIRECT_16, DIRECT_32W} <= shared and len(shared) >= 3, shared


@pytest.mark.parametrize("dtype", list(STEP))
@pytest.mark.parametrize("transB", [0, 1])
def test_rows_far_apart(dtype, transB):
    """The kernel with 64-bit offsets: rows of A 64 MiB apart."""
    M, N, step = 18, 70, STEP[dtype]
    lda = (1 << 26) // torch.empty(0, dtype=TORCH[dtype]).element_size()
    memory = torch.empty(M * (1 << 26), dtype=torch.uint8, device="cuda").view(TORCH[dtype])
    for steps in (1, 6):
        for rest in (1, step // 2 + 1, step - 1):
            K = steps * step + rest
            assert route(dtype, M, N, K, transB, lda=lda)[2] == DIRECT_ANY
            near, B = _sides(dtype, M, N, K, transB)
            A = memory.as_strided((M, K), (lda, 1))
            A.copy_(near)
            v = VerifiedGemm(M, N, K, dtype, transB)
            v.problem = vb.make_problem(M, N, K, dtype, transB, lda)
            _check(dtype, M, N, K, transB, A, B, v, lambda: v.run_fused(A, B), True)
