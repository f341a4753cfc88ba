"""Both families of GEMM kernels on every route, at the sizes where they can go wrong: the direct kernels (every tile
shape: single rows, remainders in every direction, a K that ends inside a step, rows of under 16 bytes, rows far apart,
unaligned bases and pitches) and the whole-tile kernels with the smallest number of tiles that still takes them."""
import numpy as np
import pytest

import workloads as wl
from oracle import vabft_oracle as orc

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from test_gpu_parity import _acc_np, _dev, _emax, _session, check_C, check_light, check_rows  # noqa: E402
from test_gpu_blocks import check_blocks  # noqa: E402
from test_gpu_columns import check_columns  # noqa: E402
from test_gpu_fp8 import check_C8  # noqa: E402
from test_gpu_weighted import check_weighted  # noqa: E402

FP8 = ("f8", "f8e5m2")
_TDT = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32, "f64": torch.float64,
        "f8": torch.float8_e4m3fn, "f8e5m2": torch.float8_e5m2}


def _gen(dtype, M, N, K, transB, seed):
    g = wl.rng(seed, 23)
    A = wl.to_storage(g.normal(size=(M, K)), dtype)
    B = wl.to_storage(g.normal(size=(N, K) if transB else (K, N)), dtype)
    return A, B


def _check(vg, A, B, dA, dB, dtype, M, N, K, transB, routes):
    from paper_2602_08043_amd import binding as vb
    o = orc.verify(A, B, dtype, transB, e_max=_emax(dtype, K, N))
    C_ok = check_C8 if dtype in FP8 else check_C
    C_args = (A, B, transB, dtype) if dtype in FP8 else (A, B, dtype, transB)
    for route in routes:
        print(f"{route} {dtype} {M}x{N}x{K} transB={transB}", flush=True)
        vg.astat.fill_(float("nan"))
        if route == "fused_deferred":
            vg.run_fused(dA, dB, defer_S=True)
        elif route == "blocks":
            e_blk = vb.vabft_default_emax(dtype, K, min(N, vg.W))
            vg.run_blocks(dA, dB)
            r = vg.results()
            ob = orc.verify_blocks(A, B, dtype, transB, vg.W, e_blk)
            check_blocks(r, ob, dtype)
            C_ok(r, o, *C_args)
            assert r["nflag"] == 0 and r["nblockflag"] == 0 and not r["blockflags"].any()
            continue
        else:
            getattr(vg, route)(dA, dB)
        r = vg.results()
        if route == "fused_deferred":
            r["S"] = o["S"]
        check_light(r, o, dtype, M, N, K)
        check_rows(r, o, dtype)
        C_ok(r, o, *C_args)
        assert r["nflag"] == 0 and not r["flags"].any()
        if route == "run_weighted":
            check_weighted(r, o, dtype)
        if route == "run_rc":
            oc = orc.verify_columns(A, B, dtype, transB, e_max=_emax(dtype, K, max(N, M)))
            check_columns(r, oc, dtype, M, N, K)
            assert r["ncolflag"] == 0
    # one flip in the last row and column, one in the first
    bit = 60 if dtype == "f64" else 29
    faults = sorted({(0, 0, bit), (M - 1, N - 1, bit)})
    inj = vg.make_inject(mode=1, faults=faults)
    vg.run_fused(dA, dB, inj=inj)
    r = vg.results()
    n, recs = vg.inject_records()
    assert n == len(faults) and [q[:3] for q in recs] == faults
    acc = _acc_np(dtype) if dtype not in FP8 else np.float32
    assert all(after == orc.bitflip(before, b, acc) for (_i, _j, b, before, after) in recs)
    rs = orc.replay_faults(o["rowsum"], recs)
    want = orc.fault_flags(orc.verification_difference(o["expected"], rs), o["T"])
    assert np.array_equal(r["flags"], want) and r["nflag"] == int(want.sum()) > 0


ALL = ("run", "run_fused", "fused_deferred", "run_weighted", "run_rc", "blocks")

DIRECT = [
    # at most 16 rows: 16 x 32 / 16 x 64 tiles
    ("bf16", 1, 33, 65, 1), ("f16", 16, 130, 127, 0), ("f32", 15, 31, 200, 1), ("f64", 7, 65, 17, 0), ("f8", 5, 70, 129, 1),
    ("f8e5m2", 3, 66, 300, 0),
    # few tiles, long K: 32 x 32
    ("bf16", 33, 70, 2100, 1), ("f16", 70, 65, 2049, 0), ("f32", 65, 33, 1027, 1), ("f64", 40, 100, 515, 0),
    ("f8", 35, 97, 4100, 1),
    # 32 x 64
    ("bf16", 100, 200, 130, 0), ("f16", 31, 64, 64, 1), ("f32", 65, 129, 33, 0), ("f64", 97, 130, 15, 1),
    ("f8", 100, 130, 50, 0), ("f8e5m2", 64, 64, 128, 1),
    # 64 x 64
    ("bf16", 641, 1001, 2050, 1), ("f16", 640, 1000, 2049, 0), ("bf16", 1473, 1409, 63, 0), ("f32", 1473, 1473, 31, 0),
    ("f32", 1500, 1500, 33, 1), ("f8", 1473, 1409, 130, 1),
    # rows of under 16 bytes
    ("bf16", 40, 70, 7, 1), ("f16", 33, 5, 20, 0), ("f32", 10, 3, 3, 0), ("f64", 5, 1, 1, 1), ("f8", 9, 15, 40, 0),
    ("bf16", 20, 1, 90, 0),
    # ... of A only, with rows of B (K x N) that end inside a group of 16 bytes: the last group is read from N - 16 bytes on
    ("bf16", 20, 70, 7, 0), ("bf16", 17, 20, 1, 0), ("f16", 9, 20, 4, 0), ("f32", 70, 66, 3, 0), ("f32", 10, 13, 3, 0),
    ("f64", 40, 33, 1, 0), ("f64", 5, 5, 1, 0), ("f8", 9, 33, 15, 0), ("f8", 34, 72, 7, 0), ("f8e5m2", 33, 200, 15, 0),
    # 64 x 64, FP32
    ("f32", 1000, 2040, 801, 0), ("f32", 999, 2048, 770, 1),
]


@pytest.mark.parametrize("dtype,M,N,K,transB", DIRECT)
def test_direct_shapes(dtype, M, N, K, transB):
    A, B = _gen(dtype, M, N, K, transB, 5)
    vg = _session(M, N, K, dtype, transB)
    _check(vg, A, B, _dev(A, dtype), _dev(B, dtype), dtype, M, N, K, transB, ALL)


# few tiles and a long K: several workgroups share the K of a tile (K that ends inside a step, and at one; mostly tiles of 16 x 32
# and 16 x 64: test_gpu_shared_and_copied has every shape)
SPLIT = [
    ("f32", 93, 345, 5527, 0), ("f32", 33, 65, 4096, 0), ("f32", 400, 520, 2500, 1), ("f32", 1, 153, 5193, 1),
    ("bf16", 78, 192, 6871, 0), ("bf16", 161, 128, 5120, 0), ("bf16", 300, 450, 6145, 1), ("f16", 3, 70, 9001, 1),
    ("f64", 48, 192, 1921, 1), ("f64", 100, 130, 1500, 0), ("f8", 100, 300, 8001, 0), ("f8e5m2", 9, 211, 6032, 0),
    ("f8", 53, 192, 9000, 1),
]


@pytest.mark.parametrize("dtype,M,N,K,transB", SPLIT)
def test_workgroups_that_share_the_k_of_a_tile(dtype, M, N, K, transB):
    A, B = _gen(dtype, M, N, K, transB, 19)
    vg = _session(M, N, K, dtype, transB)
    dA, dB = _dev(A, dtype), _dev(B, dtype)
    _check(vg, A, B, dA, dB, dtype, M, N, K, transB, ALL)
    vg.gemm(dA, dB)
    C = vg.C.clone()
    vg.gemm(dA, dB, 0)  # plain product
    assert torch.equal(vg.C, C)
    # a workspace without room for the parts of tiles serves as well
    vg.ws_bytes -= 5 << 20
    _check(vg, A, B, dA, dB, dtype, M, N, K, transB, ("run_fused",))


@pytest.mark.parametrize("dtype,M,N,K,transB", [("f32", 93, 345, 5527, 0), ("bf16", 300, 450, 6145, 1), ("f64", 100, 130, 1500, 0)])
def test_plain_product_with_a_workspace_that_was_never_zeroed(dtype, M, N, K, transB):
    """The counters of shared tiles start at anything (here -1): the product is whole all the same, twice in a row."""
    A, B = _gen(dtype, M, N, K, transB, 23)
    vg = _session(M, N, K, dtype, transB)
    dA, dB = _dev(A, dtype), _dev(B, dtype)
    vg.gemm(dA, dB, 0)
    C = vg.C.clone()
    vg.ws.view(torch.uint8).fill_(0xff)
    for _ in range(2):
        vg.C.fill_(float("nan"))
        vg.gemm(dA, dB, 0)
        assert torch.equal(vg.C, C)


@pytest.mark.parametrize("dtype,M,N,K,transB", [("bf16", 70, 131, 200, 1), ("f16", 33, 100, 2065, 0), ("f32", 65, 67, 70, 0),
                                                ("f64", 40, 70, 33, 1), ("f8", 50, 70, 131, 1), ("f8e5m2", 17, 90, 70, 0)])
def test_direct_unaligned_base_and_pitch(dtype, M, N, K, transB):
    """A, B and C start one element behind an aligned address and their rows are one, three and one elements longer
    than needed; what lies between the rows of C is not written, what lies between those of A and B not used."""
    from paper_2602_08043_amd import binding as vb
    A, B = _gen(dtype, M, N, K, transB, 6)
    rb, cb = B.shape

    def shifted(x, ld, fill):
        t = torch.full((x.shape[0] * ld + 1,), fill, dtype=torch.float32, device="cuda").to(x.dtype)
        v = t[1:].view(x.shape[0], ld)
        v[:, :x.shape[1]].view(torch.uint8 if x.element_size() == 1 else v.dtype).copy_(
            x.view(torch.uint8) if x.element_size() == 1 else x)
        return v
    dA, dB = shifted(_dev(A, dtype), K + 1, 400.0), shifted(_dev(B, dtype), cb + 3, -400.0)
    vg = _session(M, N, K, dtype, transB)
    vg.problem = vb.make_problem(M, N, K, dtype, transB, K + 1, cb + 3, N + 1)
    buf = torch.full((M * (N + 1) + 1,), 7.0, dtype=vg.C.dtype, device="cuda")

    class Narrow(type(vg)):
        def results(self):
            r = super().results()
            full = self.C.float().cpu().numpy()
            assert np.all(full[:, N:] == 7.0)
            r["C"] = r["C"][:, :N]
            return r
    vg.__class__ = Narrow
    vg.C = buf[1:].view(M, N + 1)
    _check(vg, A, B, dA, dB, dtype, M, N, K, transB, ALL)


def test_direct_rows_far_apart():
    """Rows of A 68 MB apart: byte offsets inside a tile need more than 32 bits."""
    from paper_2602_08043_amd import binding as vb
    dtype, M, N, K, lda = "bf16", 66, 70, 130, 34_000_000
    A, B = _gen(dtype, M, N, K, 1, 7)
    far = torch.zeros(((M - 1) * lda + K,), dtype=torch.bfloat16, device="cuda").as_strided((M, K), (lda, 1))
    far.copy_(_dev(A, dtype))
    vg = _session(M, N, K, dtype, 1)
    vg.problem = vb.make_problem(M, N, K, dtype, 1, lda, K, N)
    _check(vg, A, B, far, _dev(B, dtype), dtype, M, N, K, 1, ("run", "run_fused", "blocks"))


@pytest.mark.parametrize("dtype,M,N,K,transB", [("bf16", 35, 75, 70, 1), ("bf16", 35, 75, 70, 0), ("f32", 35, 75, 37, 0),
                                                ("f64", 35, 75, 19, 1), ("f16", 100, 130, 2100, 0)])
def test_direct_infinities_stay_in_their_row_and_column(dtype, M, N, K, transB):
    """What a tile reads in place of rows, columns and k past the end must not leak: an infinity in the last row of A
    reaches that row of C only, one in the last column of B that column only (and flags every row through its sum)."""
    g = wl.rng(8, 23)
    A = np.abs(g.normal(size=(M, K))) + 0.1
    Bl = np.abs(g.normal(size=(K, N))) + 0.1
    A[M - 1, K - 1] = np.inf
    for col in (False, True):
        Bc = Bl.copy()
        if col:
            Bc[K - 1, N - 1] = np.inf

        def dev(x):
            return torch.from_numpy(np.ascontiguousarray(x)).to(_TDT[dtype]).cuda()
        dA, dB = dev(A), dev(Bc.T if transB else Bc)
        vg = _session(M, N, K, dtype, transB)
        vg.encode(dB)
        vg.gemm_fused(dA, dB)
        C = vg.C.float().cpu().numpy()
        print(f"infinities {dtype} {M}x{N}x{K} transB={transB} col={col}", flush=True)
        want = np.zeros((M, N), dtype=bool)
        want[M - 1, :] = True
        want[:, N - 1] |= col
        assert np.array_equal(~np.isfinite(C), want)
        flags = vg.flags.cpu().numpy()
        assert flags[M - 1] == 1 and (flags.all() if col else not flags[:M - 1].any())
        assert int(vg.nflag.item()) == int(flags.sum())


@pytest.mark.parametrize("dtype,M,N,K,transB", [("bf16", 9000, 33, 70, 0), ("f64", 1057, 300, 33, 1), ("f8", 4200, 40, 64, 1),
                                                ("f32", 33, 31, 20, 0)])
def test_column_sums_of_many_tile_rows(dtype, M, N, K, transB):
    """More tile-rows than a thread folds at once, shared by groups of threads: from 282 of them down to two, of which most
    groups have none."""
    A, B = _gen(dtype, M, N, K, transB, 15)
    _check(_session(M, N, K, dtype, transB), A, B, _dev(A, dtype), _dev(B, dtype), dtype, M, N, K, transB, ("run_rc",))


def test_more_tiles_than_one_row_of_workgroups():
    """600 million rows in tiles of 32: more threads than a launch holds in one dimension.  C = 2 A for one column, and a
    checked product whose rows are all right but one."""
    from paper_2602_08043_amd import binding as vb
    M = 600_000_001
    if torch.cuda.mem_get_info()[0] < 60 << 30:
        pytest.skip("needs 60 GB of device memory")
    p = vb.make_problem(M, 1, 1, "bf16", 1)
    A = (torch.arange(M, device="cuda", dtype=torch.int32) % 128).to(torch.bfloat16)
    B = torch.full((1,), 2.0, device="cuda", dtype=torch.bfloat16)
    C = torch.zeros(M, device="cuda", dtype=torch.bfloat16)
    expected = A.float() * 2.0
    expected[M - 7] += 1.0
    T = torch.full((M,), 0.5, device="cuda")
    rowsum, E = torch.empty_like(T), torch.empty_like(T)
    flags, nflag = torch.empty(M, dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
    n = vb.vabft_workspace_bytes(p)
    ws = torch.empty(n, dtype=torch.uint8, device="cuda")
    vb.vabft_workspace_init(ws.data_ptr(), n, None)
    print("600 million rows", flush=True)
    vb.vabft_gemm_verified(p, A.data_ptr(), B.data_ptr(), C.data_ptr(), expected.data_ptr(), T.data_ptr(), 1, None,
                           rowsum.data_ptr(), E.data_ptr(), flags.data_ptr(), nflag.data_ptr(), None, None, ws.data_ptr(), n, None)
    torch.cuda.synchronize()
    assert int(nflag.item()) == 1 and int(flags[M - 7].item()) == 1 and int(flags.sum().item()) == 1
    assert bool((C == A * 2.0).all()) and bool((rowsum == C.float()).all()) and float(E[M - 7].item()) == 1.0


def test_more_rows_than_one_launch_of_the_row_passes():
    """70 million rows, a wavefront each: the A-side pass and the offline check of the last row, and of one in the middle."""
    from paper_2602_08043_amd import binding as vb
    M, N, K = 70_000_003, 2, 8
    if torch.cuda.mem_get_info()[0] < 20 << 30:
        pytest.skip("needs 20 GB of device memory")
    p = vb.make_problem(M, N, K, "bf16", 0)
    A = torch.ones((M, K), device="cuda", dtype=torch.bfloat16)
    A[M - 1] = 3.0
    Be = torch.full((K,), 2.0, device="cuda")
    S = torch.zeros(3, device="cuda", dtype=torch.float64)
    S[0] = 8.0
    astat, expected, T = (torch.full((n,), float("nan"), device="cuda") for n in (3 * M, M, M))
    print("70 million rows", flush=True)
    vb.vabft_threshold(p, A.data_ptr(), Be.data_ptr(), S.data_ptr(), 1e-3, 2.5, astat.data_ptr(), expected.data_ptr(),
                       T.data_ptr(), None)
    torch.cuda.synchronize()
    assert bool((expected[:-1] == 16.0).all()) and float(expected[-1].item()) == 48.0
    assert bool((astat.view(M, 3)[:-1] == 1.0).all()) and bool((T > 0).all()) and bool((T < 1).all())
    del A, astat
    C = torch.full((M, N), 8.0, device="cuda", dtype=torch.bfloat16)  # the last row should hold 24
    C[M // 2, 1] = 10.0
    rowsum, E = torch.full_like(T, float("nan")), torch.full_like(T, float("nan"))
    flags, nflag = torch.full((M,), 7, dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
    vb.vabft_check_offline(p, C.data_ptr(), expected.data_ptr(), T.data_ptr(), rowsum.data_ptr(), E.data_ptr(), flags.data_ptr(),
                           nflag.data_ptr(), None)
    torch.cuda.synchronize()
    assert int(nflag.item()) == 2 and int(flags.sum().item()) == 2
    assert int(flags[M // 2].item()) == 1 and int(flags[M - 1].item()) == 1 and float(rowsum[M // 2].item()) == 18.0


@pytest.mark.parametrize("transB", [0, 1])
@pytest.mark.parametrize("dtype,K", [("bf16", 7), ("bf16", 8), ("f16", 9), ("bf16", 511), ("f16", 512), ("bf16", 513), ("bf16", 1030),
                                     ("f8", 15), ("f8e5m2", 16), ("f8", 17), ("f8", 1025), ("f32", 3), ("f32", 255), ("f32", 257),
                                     ("f64", 1), ("f64", 2), ("f64", 127), ("f64", 129)])
def test_column_walk_at_the_end_of_a_row(dtype, K, transB):
    """Column statistics, sums and weighted sums of matrices whose rows end before, at and behind a lane's and a
    workgroup's share of columns (N x K B and A along K, K x N B along N = K + 1)."""
    M, N = 140, K + 1
    A, B = _gen(dtype, M, N, K, transB, 21)
    _check(_session(M, N, K, dtype, transB), A, B, _dev(A, dtype), _dev(B, dtype), dtype, M, N, K, transB, ("run_weighted", "run_rc"))


_PIECE = {"f64": 2, "f32": 4, "bf16": 8, "f16": 8, "f8": 16, "f8e5m2": 16}


@pytest.mark.parametrize("dtype,M,pieces,tail,transB", [
    # four, two and one row per wavefront, at the lengths where that changes, with and without a last piece that is not full
    ("bf16", 67, 16, 0, 1), ("f16", 67, 16, 7, 0), ("f32", 70, 17, 3, 1), ("f64", 33, 32, 1, 0), ("f8", 65, 32, 15, 1),
    ("f8e5m2", 130, 33, 0, 0), ("bf16", 9, 1, 1, 1), ("f32", 15, 16, 3, 1),
    # more rows than the GEMM's launch takes along: a launch of its own, with the rows' sums folded by one more when deferred
    ("bf16", 4200, 33, 1, 1), ("f64", 4101, 40, 0, 0),
    # ... unless they share a wavefront
    ("f32", 40000, 2, 1, 1)])
def test_rows_of_the_fused_pass_have_the_bits_of_the_separate_one(dtype, M, pieces, tail, transB):
    N, K = 70, pieces * _PIECE[dtype] + tail
    A, B = _gen(dtype, M, N, K, transB, 16)
    vg = _session(M, N, K, dtype, transB)
    dA, dB = _dev(A, dtype), _dev(B, dtype)
    o = orc.verify(A, B, dtype, transB, e_max=_emax(dtype, K, N))
    vg.run(dA, dB)
    want = vg.results()
    check_rows(want, o, dtype)
    for defer in (False, True):
        for t in (vg.astat, vg.expected, vg.T):
            t.fill_(float("nan"))
        vg.run_fused(dA, dB, defer_S=defer)
        r = vg.results()
        print(f"fused rows {dtype} {M}x{N}x{K} transB={transB} defer={defer}", flush=True)
        assert np.array_equal(r["astat"], want["astat"]) and np.array_equal(r["expected"], want["expected"])
        assert np.allclose(r["T"], want["T"], rtol=1e-12 if dtype == "f64" else 1e-6, atol=0.0)
        assert r["nflag"] == 0 and not r["flags"].any()


@pytest.mark.parametrize("dtype,M,N,K,transB", [("bf16", 255, 40, 70, 1), ("bf16", 256, 250, 70, 0), ("bf16", 257, 64, 300, 1),
                                                ("f32", 513, 200, 33, 0), ("f64", 1000, 130, 65, 1), ("f8", 777, 256, 40, 0),
                                                ("f16", 300, 300, 130, 1)])
def test_tile_rows_that_share_a_counter(dtype, M, N, K, transB):
    """Up to four tile-columns: 256 rows are compared at once.  Sizes around one and two such groups, and one column more."""
    A, B = _gen(dtype, M, N, K, transB, 17)
    vg = _session(M, N, K, dtype, transB)
    _check(vg, A, B, _dev(A, dtype), _dev(B, dtype), dtype, M, N, K, transB, ("run", "run_fused", "run_weighted"))


OWN = [
    # 32 rows per wavefront
    ("f32", 833, 2070, 33, 0), ("f32", 801, 2300, 200, 1), ("f64", 833, 2070, 17, 0), ("f64", 865, 2049, 65, 1),
    ("bf16", 1501, 1999, 70, 0), ("bf16", 1537, 2047, 129, 1), ("f16", 1500, 2001, 260, 1), ("f8", 1501, 1999, 300, 0),
    ("f8e5m2", 1600, 2100, 16, 1), ("f32", 2047, 2305, 4, 0),
    # 64 rows
    ("f32", 2100, 3100, 33, 0), ("f32", 2049, 3329, 70, 1), ("bf16", 2100, 3101, 33, 1), ("f16", 2111, 3073, 131, 0),
    ("f8", 2100, 3100, 190, 0), ("f8e5m2", 2177, 3120, 65, 1), ("bf16", 2041, 3500, 801, 1),
    ("bf16", 3607, 1665, 407, 1),  # (the size before is one that is copied for the tiled kernels)
]


@pytest.mark.parametrize("dtype,M,N,K,transB", OWN)
def test_a_tile_per_wavefront(dtype, M, N, K, transB):
    """Enough tiles that K is not split: remainders in every direction, a last workgroup of a tile-row in which some
    wavefronts have no columns, a K below, inside and above one step."""
    A, B = _gen(dtype, M, N, K, transB, 18)
    vg = _session(M, N, K, dtype, transB)
    dA, dB = _dev(A, dtype), _dev(B, dtype)
    _check(vg, A, B, dA, dB, dtype, M, N, K, transB, ALL)
    vg.gemm(dA, dB, 0)  # plain product
    o = orc.verify(A, B, dtype, transB, e_max=_emax(dtype, K, N))
    (check_C8 if dtype in FP8 else check_C)(vg.results(), o, *((A, B, transB, dtype) if dtype in FP8 else (A, B, dtype, transB)))


@pytest.mark.parametrize("dtype,M,N,K,transB", [
    ("f64", 2048, 2048, 2048, 0), ("f64", 333, 250, 5000, 1), ("f32", 2048, 2048, 2048, 0), ("f32", 1111, 777, 999, 1),  # K split
    ("f64", 4096, 4096, 600, 1), ("f64", 2100, 4100, 257, 0), ("f32", 8192, 1024, 1024, 1), ("f32", 4100, 4099, 515, 0),  # OWN
])
def test_error_of_the_product_against_more_precision(dtype, M, N, K, transB):
    """FP32 and FP64 products are sums of four chains over a quarter of K each.  With N(0,1) operands the sum after j
    terms has variance j, an addition rounds by at most u |sum| (u^2 / 3 sum^2 in the mean of a uniform error): the squares
    of four chains add up to 4 (K/4)^2 / 6 u^2, of the additions that join them to (1/2 + 3/4 + 1) K / 3 u^2, relative to
    C's own K together u^2 (K / 24 + 3/4).  One chain over K has u^2 K / 6, twice the error.  Rows sampled, the reference in
    extended precision (FP32: in FP64)."""
    A, B = _gen(dtype, M, N, K, transB, 21)
    vg = _session(M, N, K, dtype, transB)
    vg.run_fused(_dev(A, dtype), _dev(B, dtype))
    X = np.longdouble if dtype == "f64" else np.float64
    rows = np.linspace(0, M - 1, 16).astype(int)
    exact = A[rows].astype(X) @ (B.T if transB else B).astype(X)
    off = vg.C.cpu().numpy()[rows].astype(X) - exact
    rel = float(np.sqrt((off * off).sum() / (exact * exact).sum()))
    u = 2.0 ** (-53 if dtype == "f64" else -24)
    print(f"{dtype} {M}x{N}x{K} transB={transB}: {rel:.2e}, bound {u * np.sqrt(K / 24 + 0.75):.2e}", flush=True)
    assert rel <= u * np.sqrt(K / 24 + 0.75)


@pytest.mark.parametrize("scale", [1e-85, 1e79])
@pytest.mark.parametrize("M,N,K,transB", [(70, 65, 50, 0), (5, 130, 600, 1)])
def test_fp64_thresholds_of_very_small_and_large_data(M, N, K, transB, scale):
    """The variance term of T is a product of three roots: what stands under them, multiplied, leaves FP64's range for data
    below about 1e-81 and above about 1e77, although the term itself is well inside it."""
    g = wl.rng(14, 23)
    A, B = scale * g.normal(size=(M, K)), scale * g.normal(size=(N, K) if transB else (K, N))
    for x, axis in ((A, 1), (B, 0 if transB else 1)):  # row means of zero leave this term alone
        x -= x.mean(axis=axis, keepdims=True)
    vg = _session(M, N, K, "f64", transB)
    dA, dB = _dev(A, "f64"), _dev(B, "f64")
    o = orc.verify(A, B, "f64", transB, e_max=_emax("f64", K, N))
    for route in ("run", "run_fused", "run_weighted", "run_rc"):
        vg.T.fill_(float("nan"))
        getattr(vg, route)(dA, dB)
        r = vg.results()
        print(f"{route} {M}x{N}x{K} transB={transB} scale={scale}", flush=True)
        assert np.all(np.isfinite(o["T"]) & (o["T"] > 0)) and np.allclose(r["T"], o["T"], rtol=1e-12, atol=0.0)
        assert r["nflag"] == 0


WHOLE = [("bf16", 3840, 4096, 256, 0), ("f16", 4096, 3840, 192, 1), ("bf16", 2304, 2304, 256, 0), ("bf16", 2304, 2304, 192, 1), ("f16", 2304, 2304, 384, 1), ("f16", 2304, 2304, 64, 0),
         ("f8", 1792, 1792, 512, 1), ("f8e5m2", 1792, 1792, 256, 1)]


@pytest.mark.parametrize("dtype,M,N,K,transB", WHOLE)
def test_whole_tile_kernels(dtype, M, N, K, transB):
    """240 tiles of 256 x 256, which the 16-bit types run as such, and 81 (FP8: 49), just above the line below which the
    direct kernels take over (in tiles of 128 columns where the product is the plain or the checked one)."""
    A, B = _gen(dtype, M, N, K, transB, 9)
    vg = _session(M, N, K, dtype, transB)
    _check(vg, A, B, _dev(A, dtype), _dev(B, dtype), dtype, M, N, K, transB, ALL)


RAGGED = [("bf16", 2049, 2056, 200, 0), ("bf16", 2303, 2296, 72, 1), ("f16", 2100, 2184, 256, 1), ("f16", 2050, 2064, 384, 0),
          ("bf16", 2175, 2112, 128, 1), ("bf16", 2300, 2200, 64, 0), ("f16", 2111, 2080, 1032, 1), ("f16", 2241, 2312, 120, 0),
          # 192 columns
          ("bf16", 2817, 2888, 64, 0), ("bf16", 3000, 2984, 136, 1), ("f16", 2900, 3064, 384, 0), ("f16", 3072, 2880, 512, 1),
          ("bf16", 2827, 2976, 320, 0), ("f16", 2818, 3072, 128, 1),
          # 256 columns
          ("bf16", 3841, 3848, 72, 0), ("f16", 3900, 4088, 128, 1), ("bf16", 4095, 3904, 256, 1), ("f16", 3999, 3992, 200, 0)]


@pytest.mark.parametrize("dtype,M,N,K,transB", RAGGED)
def test_tiled_kernels_at_ragged_sizes(dtype, M, N, K, transB):
    """Enough tiles for the tiled kernels (of 128 columns in front, then 192 and 256), the sizes no multiples of theirs:
    remainders of one row, of one group of eight columns, and of K below and above one step; K a multiple of 128 runs the
    fused statistics."""
    A, B = _gen(dtype, M, N, K, transB, 11)
    vg = _session(M, N, K, dtype, transB)
    dA, dB = _dev(A, dtype), _dev(B, dtype)
    _check(vg, A, B, dA, dB, dtype, M, N, K, transB, ("run", "run_fused", "fused_deferred"))
    vg.gemm(dA, dB, 0)  # plain product
    check_C(vg.results(), orc.verify(A, B, dtype, transB, e_max=_emax(dtype, K, N)), A, B, dtype, transB)


@pytest.mark.parametrize("dtype,M,N,K,transB", [("bf16", 2049, 2056, 200, 0), ("bf16", 2303, 2296, 72, 1), ("f16", 2100, 2184, 256, 1),
                                                ("f16", 2050, 2312, 64, 0), ("bf16", 2304, 2064, 1032, 0)])
def test_tiled_kernels_with_more_sums_at_ragged_sizes(dtype, M, N, K, transB):
    """Weighted, column and block-wise sums of the 256 x 256 kernel at sizes that are no multiples of it: what lies past the
    last row and column counts as zero in each."""
    A, B = _gen(dtype, M, N, K, transB, 19)
    vg = _session(M, N, K, dtype, transB)
    _check(vg, A, B, _dev(A, dtype), _dev(B, dtype), dtype, M, N, K, transB, ("run_weighted", "run_rc", "blocks"))


# around the line from which operands are copied in front of the tiled kernels, on both sides of it (of both, of B alone; K one
# above and below whole steps, FP8 of every layout); test_gpu_shared_and_copied asks which side a size is on
COPIED = [("bf16", 2049, 2303, 1001, 1), ("f16", 2100, 2183, 1003, 0), ("bf16", 1801, 4097, 513, 0), ("f16", 4000, 3001, 127, 1),
          ("bf16", 2304, 3073, 1024, 0), ("f16", 7479, 1729, 995, 1), ("f8", 2811, 2754, 2047, 1), ("f8e5m2", 2500, 3000, 1500, 0),
          ("f8", 2304, 3072, 2048, 0)]


@pytest.mark.parametrize("dtype,M,N,K,transB", COPIED)
def test_copied_operands(dtype, M, N, K, transB):
    A, B = _gen(dtype, M, N, K, transB, 27)
    dA, dB = _dev(A, dtype), _dev(B, dtype)
    vg = _session(M, N, K, dtype, transB)
    # not zeros where the copies go: what lies behind their rows has to be written
    vg.ws.view(torch.uint8)[vg.ws_bytes // 2:].fill_(0xff)
    _check(vg, A, B, dA, dB, dtype, M, N, K, transB, ALL)
    vg.gemm(dA, dB)
    C = vg.C.clone()
    vg.gemm(dA, dB, 0)  # plain product
    assert torch.equal(vg.C, C)


@pytest.mark.parametrize("dtype,M,N,K,transB", [("bf16", 2049, 2303, 1001, 1), ("f8", 2811, 2754, 2047, 1), ("f16", 3000, 2500, 511, 0)])
def test_copied_rows_give_the_bits_of_the_separate_pass(dtype, M, N, K, transB):
    """The A-side pass on the rows as they are copied against vabft_threshold, S1..S3 folded before and in the pass; what
    the caller passes is not written, and infinities stay in their row and column."""
    A, B = _gen(dtype, M, N, K, transB, 28)
    dA, dB = _dev(A, dtype), _dev(B, dtype)
    vg = _session(M, N, K, dtype, transB)
    vg.encode(dB)
    vg.threshold(dA)
    want = [vg.astat.clone(), vg.expected.clone(), vg.T.clone()]
    for defer in (False, True):
        vg.astat.fill_(float("nan"))
        vg.run_fused(dA, dB, defer_S=defer)
        assert all(torch.equal(x, y) for x, y in zip(want, [vg.astat, vg.expected, vg.T]))
    assert torch.equal(dA.view(torch.uint8), _dev(A, dtype).view(torch.uint8))
    if dtype != "f8":
        dA[M - 1, K - 1] = float("inf")
        dB.abs_().add_(0.1)
        dA[: M - 1].abs_()
        vg.encode(dB)
        vg.gemm_fused(dA, dB)
        bad = ~torch.isfinite(vg.C)
        assert bad[M - 1].all() and not bad[: M - 1].any() and int(vg.nflag.item()) == 1 and int(vg.flags[M - 1].item()) == 1


@pytest.mark.parametrize("dtype,M,N,K,ldc,shift", [
    ("bf16", 2300, 2201, 64, 2201, 0), ("f16", 2049, 2303, 200, 2303, 0), ("bf16", 2100, 2056, 136, 2057, 0),
    ("f16", 2048, 2304, 128, 2304, 1), ("bf16", 3000, 2985, 136, 2985, 0), ("f16", 3900, 4089, 128, 4089, 3)])
def test_tiled_kernels_with_any_columns_and_any_alignment_of_C(dtype, M, N, K, ldc, shift):
    """B stored N x K: the tiled kernels need aligned rows of A and B, but N may be any number and C lie anywhere.  What lies
    around and between the rows of C stays as it is."""
    from paper_2602_08043_amd import binding as vb
    A, B = _gen(dtype, M, N, K, 1, 20)
    vg = _session(M, N, K, dtype, 1)
    vg.problem = vb.make_problem(M, N, K, dtype, 1, K, K, ldc)
    buf = torch.full((M * ldc + shift + 8,), 7.0, dtype=vg.C.dtype, device="cuda")
    full = buf[shift:shift + M * ldc].view(M, ldc)
    vg.C = full[:, :N]
    dA, dB = _dev(A, dtype), _dev(B, dtype)
    o = orc.verify(A, B, dtype, 1, e_max=_emax(dtype, K, N))
    for route in ("plain", "run", "run_fused", "run_weighted", "run_rc", "blocks"):
        buf.fill_(7.0)
        vg.gemm(dA, dB, 0) if route == "plain" else vg.run_blocks(dA, dB) if route == "blocks" else getattr(vg, route)(dA, dB)
        vg.C = full[:, :N].contiguous()
        r = vg.results()
        vg.C = full[:, :N]
        print(f"{route} {dtype} {M}x{N}x{K} ldc={ldc} shift={shift}", flush=True)
        check_C(r, o, A, B, dtype, 1)
        if route not in ("plain", "blocks"):
            check_light(r, o, dtype, M, N, K)
            check_rows(r, o, dtype)
        if route != "plain":
            assert r["nflag"] == 0 and not r["blockflags" if route == "blocks" else "flags"].any()
        assert bool((full[:, N:] == 7.0).all()) and bool((buf[:shift] == 7.0).all()) and bool((buf[shift + M * ldc:] == 7.0).all())


@pytest.mark.parametrize("K", [1920, 2048])
def test_narrow_tiles_at_the_end_of_the_checksum_panel(K):
    """One tile-column folds all of K: as many units as the panel in LDS holds, and one more (a pass of its own)."""
    dtype, M, N = "bf16", 33000, 128
    A, B = _gen(dtype, M, N, K, 1, 13)
    vg = _session(M, N, K, dtype, 1)
    _check(vg, A, B, _dev(A, dtype), _dev(B, dtype), dtype, M, N, K, 1, ("run_fused",))


def test_tiled_kernels_leave_padding_of_C():
    from paper_2602_08043_amd import binding as vb
    dtype, M, N, K = "bf16", 2100, 2056, 136
    A, B = _gen(dtype, M, N, K, 0, 12)
    vg = _session(M, N, K, dtype, 0)
    vg.problem = vb.make_problem(M, N, K, dtype, 0, K, N, N + 8)
    vg.C = torch.full((M + 1, N + 8), 7.0, dtype=torch.bfloat16, device="cuda")
    vg.run_fused(_dev(A, dtype), _dev(B, dtype))
    C = vg.C.float().cpu().numpy()
    assert np.all(C[:, N:] == 7.0) and np.all(C[M:] == 7.0) and int(vg.nflag.item()) == 0


@pytest.mark.parametrize("dtype", ["bf16", "f32", "f64", "f8"])
def test_one_workspace_across_the_change_of_counter_distance(dtype):
    """Arrival counters lie a cache line apart up to 1023 tile-rows (32736 rows in tiles of 32, 65472 of 64) and side by
    side above: problems on both sides of the line share a workspace, one after the other."""
    from paper_2602_08043_amd import binding as vb
    N, K, Mmax, tol = 330, 32, 65536, 1e-13 if dtype == "f64" else 1e-5
    A, B = _gen(dtype, Mmax, N, K, 1, 19)
    dA, dB = _dev(A, dtype), _dev(B, dtype)
    need = vb.vabft_workspace_bytes(vb.make_problem(Mmax, N, K, dtype, 1))
    ws = torch.empty(need + 4096, dtype=torch.uint8, device="cuda")
    vb.vabft_workspace_init(ws.data_ptr(), need, None)
    ws[need:] = 0x5A
    o = orc.verify(A, B, dtype, 1, e_max=_emax(dtype, K, N))
    for M in (32736, 32737, 65472, 65473, 40, 65536, 32700):
        vg = _session(M, N, K, dtype, 1)
        vg.ws, vg.ws_bytes = ws, need
        print(f"shared workspace {dtype} M={M}", flush=True)
        vg.run_fused(dA[:M].contiguous(), dB)
        r = vg.results()
        assert np.all(np.abs(r["rowsum"] - o["rowsum"][:M]) <= tol * o["scale_rowsum"][:M])
        assert np.all(np.abs(r["E"]) <= r["T"]) and r["nflag"] == 0 and not r["flags"].any()
        inj = vg.make_inject(mode=1, faults=[(M - 1, N - 1, 60 if dtype == "f64" else 29)])
        vg.run_fused(dA[:M].contiguous(), dB, inj=inj)
        r = vg.results()
        assert r["nflag"] == 1 and r["flags"][M - 1] == 1 and r["flags"].sum() == 1
        assert bool((ws[need:] == 0x5A).all())


def test_one_workspace_for_fewer_rows():
    """A workspace sized for M rows serves every problem with fewer: the routes change with M, the counters they share
    stay zero and no partial leaves the workspace."""
    from paper_2602_08043_amd import binding as vb
    dtype, N, K, Mmax = "bf16", 2304, 256, 2304
    A, B = _gen(dtype, Mmax, N, K, 1, 10)
    dA, dB = _dev(A, dtype), _dev(B, dtype)
    need = vb.vabft_workspace_bytes(vb.make_problem(Mmax, N, K, dtype, 1))
    ws = torch.empty(need + 4096, dtype=torch.uint8, device="cuda")
    vb.vabft_workspace_init(ws.data_ptr(), need, None)
    ws[need:] = 0x5A
    o = orc.verify(A, B, dtype, 1, e_max=_emax(dtype, K, N))
    for M in (1, 2304, 17, 40, 300, 2304, 1500):
        vg = _session(M, N, K, dtype, 1)
        vg.ws, vg.ws_bytes = ws, need
        vg.run_fused(dA[:M].contiguous(), dB, defer_S=True)
        r = vg.results()
        print(f"shared workspace M={M}", flush=True)
        assert np.all(np.abs(r["rowsum"] - o["rowsum"][:M]) <= 1e-5 * o["scale_rowsum"][:M])
        assert np.all(np.abs(r["expected"] - o["expected"][:M]) <= 1e-5 * o["scale_expected"][:M])
        assert r["nflag"] == 0 and not r["flags"].any()
        assert bool((ws[need:] == 0x5A).all())
