"""Tiles whose K several workgroups share, and operands that are copied in front of the tiled kernels: every form of both, each
test asking the library first (on the host) that its size takes the form it is there for; with padded rows, infinities and
NaN, and inside a HIP graph."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2602_08043_amd import binding as vb  # noqa: E402
from test_gpu_parity import _dev, _session  # noqa: E402
from test_gpu_routes import ALL, _check, _gen  # noqa: E402
from test_routes_cpu import CHAINS, DIRECT_16, DIRECT_32, DIRECT_32W, DIRECT_64, TILED, route  # noqa: E402

# every tile shape in the types and layouts that have it (16-bit and FP8: DIRECT_32 for N x K only)
SHARED = [("f16", 101, 1311, 10873, 0, DIRECT_64), ("f32", 712, 374, 4801, 1, DIRECT_64), ("f8", 472, 1016, 8372, 0, DIRECT_64),
          ("bf16", 198, 305, 2969, 1, DIRECT_32), ("f32", 271, 262, 501, 1, DIRECT_32), ("f32", 1093, 100, 799, 0, DIRECT_32),
          ("f64", 1082, 83, 519, 0, DIRECT_32), ("f64", 71, 813, 565, 1, DIRECT_32), ("f8", 68, 840, 2078, 1, DIRECT_32),
          ("bf16", 686, 74, 2379, 0, DIRECT_32W), ("f32", 196, 712, 570, 0, DIRECT_32W), ("f32", 132, 834, 563, 1, DIRECT_32W),
          ("f64", 406, 315, 509, 1, DIRECT_32W), ("f8", 986, 80, 1879, 0, DIRECT_32W), ("f8", 18, 117, 1862, 1, DIRECT_32W),
          ("f64", 2, 126, 1410, 0, DIRECT_16), ("f8", 3, 391, 5109, 1, DIRECT_16)]


@pytest.mark.parametrize("dtype,M,N,K,transB,shape", SHARED)
def test_shared_tiles_of_every_shape(dtype, M, N, K, transB, shape):
    _, _, kernel, split, _, _ = route(dtype, M, N, K, transB)
    assert kernel == shape and split > 1
    A, B = _gen(dtype, M, N, K, transB, 29)
    vg = _session(M, N, K, dtype, transB)
    _check(vg, A, B, _dev(A, dtype), _dev(B, dtype), dtype, M, N, K, transB, ALL)


# A and B copied: K with padding in both layouts; A alone, B alone (rows at odd addresses; an odd number of columns); rows that 16
# lanes or 32 or a wavefront copy; FP8
COPIED = [("f16", 2312, 2697, 639, 0, 0, 0, (1, 1)), ("bf16", 1738, 2885, 577, 1, 0, 0, (1, 1)),
          ("bf16", 2312, 2672, 784, 0, 3, 0, (1, 0)), ("bf16", 2387, 2136, 560, 1, 3, 0, (1, 0)),
          ("f16", 2890, 2459, 680, 0, 0, 0, (0, 1)), ("f16", 2840, 2528, 560, 1, 0, 5, (0, 1)),
          ("bf16", 4252, 1837, 65, 0, 0, 0, (1, 1)), ("bf16", 1770, 4361, 65, 1, 0, 0, (1, 1)),
          ("f16", 2505, 2819, 139, 0, 0, 0, (1, 1)), ("bf16", 4096, 1739, 137, 1, 0, 0, (1, 1)),
          ("f8", 2038, 3995, 165, 0, 0, 0, (1, 1)), ("f8e5m2", 2774, 2529, 274, 1, 0, 0, (1, 1)),
          ("f8", 2281, 2731, 555, 1, 7, 1, (1, 1)), ("f8e5m2", 2304, 3072, 2048, 0, 0, 0, (1, 1))]


def _padded(t, pad):
    """The same matrix with `pad` elements more from row to row, NaN in them."""
    if not pad:
        return t
    r, c = t.shape
    wide = torch.full((r, c + pad), float("nan"), dtype=torch.float32, device=t.device).to(t.dtype)
    wide.view(torch.uint8).view(r, -1)[:, : c * t.element_size()] = t.contiguous().view(torch.uint8).view(r, -1)
    return wide


def _copied_session(dtype, M, N, K, transB, pad_a=0, pad_b=0, copied=(1, 1)):
    lda, ldb = K + pad_a, (K if transB else N) + pad_b
    a, b, kernel, _, form, _ = route(dtype, M, N, K, transB, lda=lda, ldb=ldb)
    assert ((a, b), kernel, form) == (copied, TILED, CHAINS)
    vg = _session(M, N, K, dtype, transB)
    vg.problem = vb.make_problem(M, N, K, dtype, transB, lda, ldb)
    vg.ws_bytes = vb.vabft_workspace_bytes(vg.problem)
    vg.ws = torch.full((vg.ws_bytes,), 0xff, dtype=torch.uint8, device=vg.ws.device)  # (nothing but counters has to be zero)
    vg.ws[: 1 << 20] = 0
    return vg


@pytest.mark.parametrize("dtype,M,N,K,transB,pad_a,pad_b,copied", COPIED)
def test_copied_operands_of_every_kind(dtype, M, N, K, transB, pad_a, pad_b, copied):
    """Against FP64, and against the kernels that read the rows as they lie: without room for the copies the same call takes them."""
    vg = _copied_session(dtype, M, N, K, transB, pad_a, pad_b, copied)
    A, B = (_dev(x, dtype) for x in _gen(dtype, M, N, K, transB, 33))
    dA, dB = _padded(A, pad_a), _padded(B, pad_b)
    before = dA.clone(), dB.clone()
    vg.encode(dB)
    vg.threshold(dA)
    want = [vg.astat.clone(), vg.expected.clone(), vg.T.clone()]
    vg.astat.fill_(float("nan"))
    vg.gemm_fused(dA, dB)
    # the pass over A on the rows as they are copied has the bits of the pass by itself
    assert all(torch.equal(x, y) for x, y in zip(want, [vg.astat, vg.expected, vg.T]))
    assert int(vg.nflag.item()) == 0 and not vg.flags.any()
    assert all(torch.equal(x.view(torch.uint8), y.view(torch.uint8)) for x, y in zip(before, (dA, dB)))
    C, rowsum = vg.C.clone(), vg.rowsum.clone()
    A64, B64 = A.float().double(), B.float().double()
    B64 = B64.t().contiguous() if transB else B64
    P, size = A64 @ B64, A64.abs() @ B64.abs()
    # FP32 accumulation (32 terms to a sum of the instruction, four chains): within K 2^-24 of the terms' size; then one rounding
    unit = 2.0 ** -8 if dtype == "bf16" else 2.0 ** -11
    assert bool(((C.double() - P).abs() <= unit * P.abs() + K * 2.0 ** -24 * size + 2.0 ** -24).all())
    assert bool(((rowsum.double() - P.sum(1)).abs() <= vg.T.double()).all())
    # separate calls: same bits
    vg.C.zero_()
    vg.gemm(dA, dB)
    assert torch.equal(vg.C, C) and torch.equal(vg.rowsum, rowsum)
    # as the rows lie
    vg.ws_bytes -= 1 << 20
    assert route(dtype, M, N, K, transB, lda=K + pad_a, ldb=(K if transB else N) + pad_b, room=vg.ws_bytes)[:2] == (0, 0)
    vg.C.zero_()
    vg.gemm_fused(dA, dB)
    assert bool(((vg.C.double() - P).abs() <= unit * P.abs() + K * 2.0 ** -24 * size + 2.0 ** -24).all())
    assert bool(((vg.rowsum - rowsum).abs() <= 2 * vg.T).all()) and int(vg.nflag.item()) == 0


@pytest.mark.parametrize("dtype,M,N,K,transB", [("f16", 2312, 2697, 639, 0), ("bf16", 1738, 2885, 577, 1), ("f8e5m2", 2774, 2529, 274, 1)])
def test_infinities_and_nan_stay_in_their_row_and_column(dtype, M, N, K, transB):
    """Zeros behind the copies' rows and columns must not meet them: only the row of an infinity in A and the column of a NaN in
    B hold anything that is not finite."""
    vg = _copied_session(dtype, M, N, K, transB)
    A, B = (_dev(x, dtype).float().abs().clamp(0.125, 2.0) for x in _gen(dtype, M, N, K, transB, 34))
    A[M - 1, K - 1] = float("inf")
    B[(N - 1, 0) if transB else (0, N - 1)] = float("nan")
    dA, dB = A.to(vg_dtype := _dev(_gen(dtype, 1, 8, 8, 1, 1)[0], dtype).dtype), B.to(vg_dtype)
    vg.encode(dB)
    vg.gemm_fused(dA, dB)
    bad = ~torch.isfinite(vg.C)
    assert bool(bad[M - 1].all()) and bool(bad[:, N - 1].all())
    bad[M - 1], bad[:, N - 1] = False, False
    assert not bool(bad.any())
    assert int(vg.nflag.item()) == M  # every row's sum has the NaN


@pytest.mark.parametrize("dtype,M,N,K,transB,pad_a,pad_b", [
    ("f32", 93, 345, 5527, 0, 3, 7), ("bf16", 198, 305, 2969, 1, 5, 1), ("f16", 101, 1311, 10873, 0, 7, 9), ("f64", 48, 192, 1921, 1, 1, 2),
    ("f8", 68, 840, 2078, 1, 3, 5)])
def test_shared_tiles_with_padded_rows(dtype, M, N, K, transB, pad_a, pad_b):
    lda, ldb, ldc = K + pad_a, (K if transB else N) + pad_b, N + 3
    assert route(dtype, M, N, K, transB, lda=lda, ldb=ldb, ldc=ldc)[3] > 1
    A, B = (_dev(x, dtype) for x in _gen(dtype, M, N, K, transB, 35))
    vg = _session(M, N, K, dtype, transB)
    vg.run_fused(A, B)
    want = [x.clone() for x in (vg.C, vg.rowsum, vg.expected, vg.T, vg.E, vg.Be)]
    vg.problem = vb.make_problem(M, N, K, dtype, transB, lda, ldb, ldc)
    vg.C = torch.full((M, ldc), 7.0, dtype=vg.C.dtype, device=vg.C.device)
    vg.run_fused(_padded(A, pad_a), _padded(B, pad_b))
    assert bool((vg.C[:, N:] == 7).all())
    got = [vg.C[:, :N], vg.rowsum, vg.expected, vg.T, vg.E, vg.Be]
    # (whole 16-byte pieces of a row are loaded wherever they start: the same sums)
    assert all(torch.equal(x, y) for x, y in zip(got, want))


# a matrix of 64 columns' panels and of two launches' (rows from row to row padded): infinities, NaN and the type's lowest value
@pytest.mark.parametrize("dtype,cols,rows", [("bf16", 300, 600), ("f16", 41, 1100), ("f32", 100, 700), ("f64", 70, 300), ("f8e5m2", 81, 900),
                                             ("bf16", 300, 2771), ("f32", 100, 2109)])
def test_column_passes_with_padded_rows_infinities_and_nan(dtype, cols, rows):
    g = torch.Generator().manual_seed(cols + rows)
    acc = torch.float64 if dtype == "f64" else torch.float32
    X = torch.randint(-2, 3, (rows, cols), generator=g).to(acc)
    X[rows - 1, 0], X[0, 1], X[rows // 2, cols - 1] = float("inf"), float("-inf"), float("nan")
    vg = _session(3, rows, cols, dtype, 1)
    t = _dev(_gen(dtype, 1, 8, 8, 1, 1)[0], dtype).dtype
    low = torch.finfo(t).min if dtype != "f32" and dtype != "f64" else -1.0e30
    X[:, 2] = low  # a column of nothing else
    dX = _padded(X.to(t).to(vg.Be.device), 5)
    vg.problem = vb.make_problem(3, rows, cols, dtype, 1, None, cols + 5)
    vg.encode_weighted(dX)
    stat = vg.bstat.cpu()
    X = X.to(t).to(acc)  # (as stored)
    fin = torch.ones(cols, dtype=torch.bool)
    fin[[0, 1, 2, cols - 1]] = False
    assert torch.equal(vg.Be.cpu()[fin], X.sum(0)[fin])
    w = torch.arange(1, rows + 1, dtype=acc) @ torch.nan_to_num(X, 0.0, 0.0, 0.0)
    assert torch.equal(vg.Be2.cpu()[fin], w[fin])
    assert torch.equal(stat[fin, 0], X.amax(0)[fin]) and torch.equal(stat[fin, 1], X.amin(0)[fin])
    assert float(vg.Be[0]) == float("inf") and float(stat[0, 0]) == float("inf")
    assert float(vg.Be[1]) == float("-inf") and float(stat[1, 1]) == float("-inf")
    assert float(stat[2, 0]) == float(stat[2, 1]) == float(X[0, 2])
    assert bool(torch.isnan(vg.Be[cols - 1])) and bool(torch.isnan(vg.bstat[cols - 1, 2]))
    # extrema pass a NaN by, as the two-launch form's
    rest = torch.cat([X[: rows // 2, cols - 1], X[rows // 2 + 1:, cols - 1]])
    assert float(stat[cols - 1, 0]) == float(rest.max()) and float(stat[cols - 1, 1]) == float(rest.min())


@pytest.mark.parametrize("dtype,M,N,K,transB", [("f32", 93, 345, 5527, 0), ("f16", 101, 1311, 10873, 0), ("bf16", 1738, 2885, 577, 1),
                                                ("f16", 2890, 2459, 680, 0), ("bf16", 300, 400, 600, 1)])
def test_shared_copied_and_column_passes_inside_a_graph(dtype, M, N, K, transB):
    """Recorded once, replayed with the program's own eager calls and synchronisations in between: the eager bits every time."""
    A, B = (_dev(x, dtype) for x in _gen(dtype, M, N, K, transB, 36))
    A2, B2 = (_dev(x, dtype) for x in _gen(dtype, M, N, K, transB, 37))
    vg = _session(M, N, K, dtype, transB)
    keys = ("C", "Be", "bstat", "S", "astat", "expected", "T", "rowsum", "E", "flags", "eA", "acolstat", "SA", "expected_col", "T_col")

    def calls():
        vg.encode_a(A)
        vg.threshold_cols(B)
        vg.encode(B, defer_S=True)
        vg.gemm_fused(A, B, deferred_S=True)
        vg.encode(B)
        vg.gemm(A, B, 0)
        vg.gemm_fused(A, B)

    calls()
    want = {k: getattr(vg, k).clone() for k in keys}
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        calls()
    torch.cuda.current_stream().wait_stream(s)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        calls()
    for replay in range(3):
        vg.run_fused(A2, B2)
        vg.gemm(A2, B2, 0)
        torch.cuda.synchronize()
        for k in keys:
            getattr(vg, k).fill_(3)
        g.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(getattr(vg, k), want[k]) for k in keys), replay
