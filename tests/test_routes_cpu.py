"""What a GEMM call runs on, asked on the host (no GPU): the library's own decision for a problem, its operands' addresses and
the room of its workspace."""
import ctypes
import random

import pytest

vb = pytest.importorskip("paper_2602_08043_amd.binding")

DIRECT_16, DIRECT_32, DIRECT_32W, DIRECT_ANY, DIRECT_64, OWN32, OWN64 = range(7)
TILED, CHAINS = -1, 4


def route(dtype, M, N, K, transB=0, *, lda=None, ldb=None, ldc=None, A=4096, B=4096, C=4096, more_sums=0, injects=0, room=None):
    """(A copied, B copied, kernel, workgroups per tile, tiled kernel's form, A-side pass): see vabft_internal_route."""
    lib = vb.load()
    p = vb.make_problem(M, N, K, dtype, transB, lda, ldb, ldc)
    out = (ctypes.c_int32 * 6)()
    ptr = ctypes.c_void_p
    f = lib.vabft_internal_route
    f.restype = None
    f.argtypes = [ctypes.POINTER(vb.Problem), ptr, ptr, ptr, ctypes.c_int32, ctypes.c_int32, ctypes.c_size_t,
                  ctypes.POINTER(ctypes.c_int32)]
    f(p, A, B, C, more_sums, injects, vb.vabft_workspace_bytes(p) if room is None else room, out)
    return tuple(out)


def test_copied_operands_run_on_the_kernel_they_are_priced_for():
    """Copies are made for the 128-wide tiled kernel with K in four chains; no size makes them for another one."""
    copied = 0
    r = random.Random(5)
    problems = [("bf16", 1717, 1961, 5119, 1), ("bf16", 1308, 1402, 10752, 0), ("f16", 1661, 1687, 4441, 1)]
    problems += [(r.choice(["bf16", "f16", "f8", "f8e5m2"]), r.randint(300, 8192), r.randint(300, 11008), r.randint(64, 11008),
                  r.randint(0, 1)) for _ in range(3000)]
    for p in problems:
        a, b, kernel, split, form, _ = route(*p)
        if a or b:
            copied += 1
            assert (kernel, split, form) == (TILED, 1, CHAINS), p
    assert copied > 500
    # rows further apart than the tiled kernels take are not copied for them, but read as they lie
    far = dict(lda=(1 << 22) + 8)
    assert route("bf16", 3000, 3001, 2048, 0)[:3] == (0, 1, TILED)
    assert route("bf16", 3000, 3001, 2048, 0, **far)[:2] == (0, 0)


# measured: as the rows lie / copied (us)
COPIES_PAY = [("bf16", 3708, 1873, 10496, 0), ("f16", 1694, 8971, 5807, 1), ("f16", 5598, 2257, 2431, 0),  # 354 / 165, 479 / 213, 195 / 97
              ("bf16", 2048, 1659, 10987, 1), ("f8", 1792, 5243, 9984, 0), ("f8e5m2", 3584, 2465, 3764, 0)]  # 226 / 134, 268 / 248, 125 / 114
COPIES_LOSE = [("bf16", 1024, 2497, 3584, 0), ("f16", 512, 5219, 9216, 0), ("bf16", 1308, 1402, 10752, 0),  # 49 / 55, 112 / 127, 92 / 121
               ("bf16", 2568, 9722, 448, 0), ("f16", 2560, 7283, 464, 0),  # 67 / 80, 63 / 76
               ("f8", 2048, 2048, 4352, 0), ("f8", 3840, 2304, 2048, 0), ("f8", 2560, 1561, 4096, 1)]  # 57 / 65, 66 / 75, 51 / 61


def test_operands_are_copied_where_that_is_faster():
    for p in COPIES_PAY:
        assert route(*p)[2] == TILED and sum(route(*p)[:2]) > 0, p
    for p in COPIES_LOSE:
        assert route(*p)[:2] == (0, 0), p


FIRST, LAST = 0, 1
# measured fused calls, the pass in front of the tiles / behind them (us)
PASS_ORDER = [("f16", 179, 256, 2560, 0, LAST), ("f32", 7168, 256, 128, 1, LAST),  # 11.9 / 9.6, 19.0 / 14.2
              ("f8e5m2", 8192, 375, 293, 0, LAST), ("f32", 3072, 128, 10467, 0, LAST),  # 24.9 / 18.6, 190 / 113
              ("bf16", 192, 4995, 2145, 0, FIRST), ("f16", 906, 2467, 1092, 1, FIRST), ("f64", 1536, 3072, 80, 1, FIRST),  # 21.0 / 22.7, 26.5 / 29.2, 36.4 / 37.9
              ("f64", 2147, 768, 125, 1, LAST),  # 28.0 / 20.8
              ("f16", 1280, 1792, 1134, 0, FIRST), ("f16", 783, 1589, 7788, 0, FIRST),  # 22.4 / 24.3, 84.6 / 89.8
              ("bf16", 261, 9647, 128, 0, FIRST), ("f32", 3259, 7979, 128, 0, FIRST), ("f64", 552, 3165, 392, 1, FIRST)]  # 12.3 / 14.3, 87 / 94, 41.4 / 43.8


def test_place_of_the_a_side_pass():
    for *p, place in PASS_ORDER:
        assert route(*p)[5] == place, p


# measured fused calls, not shared / shared (us)
SHARED = [("f32", 93, 345, 5527, 0), ("f64", 48, 192, 3840, 1),  # 51 / 16, 39 / 11
          ("bf16", 78, 192, 6871, 0), ("bf16", 1280, 99, 6882, 1),  # 23 / 10, 29 / 20
          ("f16", 4, 1681, 5803, 1), ("f16", 1, 107, 5065, 1), ("bf16", 1792, 80, 3169, 1)]  # 18.2 / 12.1, 13.3 / 9.8, 22.4 / 18.4
NOT_SHARED = [("bf16", 40, 512, 1280, 1), ("f64", 683, 80, 231, 1), ("f8", 48, 6400, 9065, 1),  # 7.9 / 8.5, 12.0 / 12.8, 30 / 36
              ("f16", 30, 3584, 1974, 1)]  # 10.2 / 11.0


def test_workgroups_share_the_k_of_a_tile_where_that_is_faster():
    for p in SHARED:
        assert route(*p)[3] > 1, p
    for p in NOT_SHARED:
        assert route(*p)[3] == 1, p


def test_static_scratch_decides_like_a_workspace_but_for_copies():
    """The call without a workspace (16 MiB and 128 KiB of its own) takes the same kernel, tile and split."""
    r = random.Random(11)
    problems = [("f32", 200, 300, k, 1) for k in range(9_700_000, 10_500_000, 100_000)]  # S1..S3's partials take most of the array
    problems += [(r.choice(list(vb.DTYPE_CODE)), r.randint(1, 3000), r.randint(1, 9000), r.randint(1, 20000), r.randint(0, 1))
                 for _ in range(3000)]
    for p in problems:
        here = route(*p)
        if here[:2] == (0, 0):
            assert route(*p, room=(16 << 20) + (128 << 10)) == here, p
