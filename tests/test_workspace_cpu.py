"""Sizes of the workspace: one that serves M rows serves fewer (same type, layout, N and K)."""
import random

import pytest

vb = pytest.importorskip("paper_2602_08043_amd.binding")


def test_workspace_grows_with_rows():
    r = random.Random(3)
    for _ in range(400):
        dt = r.choice(list(vb.DTYPE_CODE))
        N, K, tb = r.randint(1, 20000), r.randint(1, 5000), r.randint(0, 1)
        rows = sorted(r.choice([1, 16, 17, 32, 33, 64, 255, 256, 2048, r.randint(1, 20000)]) for _ in range(6))
        sizes = [vb.vabft_workspace_bytes(vb.make_problem(M, N, K, dt, tb)) for M in rows]
        assert sizes == sorted(sizes), (dt, N, K, tb, rows, sizes)
