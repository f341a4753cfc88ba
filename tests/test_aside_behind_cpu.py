"""Whether the A-side pass of a fused call on the 16-bit tiled kernels has workgroups behind the tiles: the faster way where the
two differ."""
import ctypes

import pytest

vb = pytest.importorskip("paper_2602_08043_amd.binding")

# measured fused calls: on the operand tiles or in front / behind (us)
BEHIND = [("bf16", 1000, 11008, 4096, 1, 83.6, 81.1), ("bf16", 2688, 3456, 384, 1, 19.6, 16.9), ("f16", 5760, 2304, 4608, 1, 103.5, 102.8),
          ("bf16", 2928, 1792, 768, 0, 18.8, 15.9), ("f16", 5120, 696, 1320, 1, 35.1, 29.6), ("bf16", 7400, 512, 2432, 0, 35.2, 30.6),
          ("f16", 4206, 4672, 1856, 0, 84.2, 78.2), ("bf16", 1421, 10024, 6208, 1, 140.2, 136.1),
          ("bf16", 4224, 1080, 2032, 0, 44.7, 38.3)]
# (a K of which lanes have three pieces of 16 bytes or four, and units that are too few)
NOT_BEHIND = [("f16", 2660, 4992, 1920, 0, 54.8, 59.7), ("f16", 6528, 512, 1792, 1, 28.1, 33.1), ("f16", 4346, 2048, 1792, 1, 38.7, 42.9),
              ("f16", 3193, 2816, 1792, 0, 39.8, 43.2), ("bf16", 4992, 768, 1664, 1, 26.4, 28.5), ("f16", 5888, 768, 1856, 1, 31.9, 34.1),
              ("bf16", 3988, 1280, 1792, 0, 28.3, 29.6), ("f16", 4096, 1280, 1792, 0, 28.9, 30.2), ("bf16", 7680, 768, 4224, 1, 53.6, 74.4),
              ("f16", 3840, 3584, 256, 0, 18.8, 25.6)]


@pytest.mark.parametrize("behind,problems", [(True, BEHIND), (False, NOT_BEHIND)])
def test_where_the_pass_runs(behind, problems):
    f = vb.load().vabft_internal_behind
    f.restype, f.argtypes = ctypes.c_int32, [ctypes.POINTER(vb.Problem)] + [ctypes.c_void_p] * 3 + [ctypes.c_size_t]
    for dtype, M, N, K, transB, *_ in problems:
        p = vb.make_problem(M, N, K, dtype, transB)
        assert (f(p, 4096, 4096, 4096, vb.vabft_workspace_bytes(p)) > 0) == behind, (dtype, M, N, K, transB)
