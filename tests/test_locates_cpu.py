"""Whether the weighted call localises flagged rows in the GEMM's launch: the faster way where the two differ."""
import ctypes

import pytest

vb = pytest.importorskip("paper_2602_08043_amd.binding")

# measured weighted calls: in the compare / in a launch of its own (us)
IN_LAUNCH = [("bf16", 1024, 1024, 1024, 0, 14.6, 15.4), ("bf16", 1024, 1024, 1024, 1, 15.9, 16.7), ("f32", 1000, 1200, 500, 0, 24.4, 25.7),
             ("f8", 1024, 1024, 1024, 1, 16.3, 18.1)]
OWN_LAUNCH = [("f64", 3072, 832, 64, 0, 47.6, 30.4), ("f64", 512, 4928, 62, 0, 45.4, 29.3), ("f64", 528, 5568, 128, 1, 62.3, 42.8),
              ("f64", 909, 3474, 298, 1, 84.5, 63.1), ("f64", 2560, 1920, 384, 0, 118.2, 92.1), ("f64", 1203, 879, 133, 0, 30.6, 24.5),
              ("f64", 227, 2596, 45, 0, 19.6, 15.8), ("f64", 8016, 176, 96, 1, 40.8, 33.1), ("f32", 1408, 1920, 256, 1, 44.3, 34.1)]


@pytest.mark.parametrize("in_launch,problems", [(1, IN_LAUNCH), (0, OWN_LAUNCH)])
def test_where_rows_are_localised(in_launch, problems):
    f = vb.load().vabft_internal_locates
    f.restype, f.argtypes = ctypes.c_int32, [ctypes.POINTER(vb.Problem)] + [ctypes.c_void_p] * 3 + [ctypes.c_size_t]
    for dtype, M, N, K, transB, *_ in problems:
        p = vb.make_problem(M, N, K, dtype, transB)
        assert f(p, 4096, 4096, 4096, vb.vabft_workspace_bytes(p)) == in_launch, (dtype, M, N, K, transB)
