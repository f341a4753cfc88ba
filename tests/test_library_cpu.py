"""Host-side checks of the C-ABI library that need no GPU: it loads, exports every symbol
include/vabft.h declares, and rejects bad arguments before launching anything."""
import os
import re

import pytest

from paper_2602_08043_amd import binding as vb

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(vb.LIB_PATH):
        import __graft_entry__ as ge
        ge.build()
    return vb.load()


def test_exports_match_header(lib):
    header = open(os.path.join(ROOT, "include", "vabft.h")).read()
    declared = set(re.findall(r"\b(vabft_[a-z_]+)\s*\(", header))
    assert declared == set(vb.EXPORTS)
    for name in declared:
        assert hasattr(lib, name), name


def test_struct_layouts_match_header():
    import ctypes
    assert ctypes.sizeof(vb.Problem) == 48
    assert ctypes.sizeof(vb.Inject) == 48
    assert ctypes.sizeof(vb.InjectRec) == 32
    assert vb.Problem.lda.offset == 24 and vb.Inject.seed.offset == 16 and vb.Inject.d_list.offset == 32


def test_status_strings_and_default_emax(lib):
    assert vb.status_string(0) == "ok"
    assert "workspace" in vb.status_string(vb.VABFT_EWORKSPACE)
    # larger of the paper's GPU law and the MI355X-calibrated law, n = max(K, N)
    for n in (128, 512, 4096, 8192, 65536):
        paper, meas = 5.0e-9 * n ** 0.5 + 1.2e-7, 3.0e-9 * n ** 0.5 + 4.2e-7
        assert vb.vabft_default_emax("bf16", n, n) == pytest.approx(max(paper, meas))
        paper, meas = 1.0e-17 * n ** 0.5 + 2.5e-16, 8.0e-18 * n ** 0.5 + 7.0e-16
        assert vb.vabft_default_emax("f64", n, n) == pytest.approx(max(paper, meas))
    assert vb.vabft_default_emax("f16", 4096, 11008) == vb.vabft_default_emax("f32", 11008, 4096)


def test_default_emax_keeps_its_margin_over_the_calibration_table(lib):
    """Every row of the committed calibration table (the paper's protocol run with this library's kernels on
    MI355X; the '+20 %' column is the protocol's own margin): the default lies at least 25 % above it."""
    import os
    path = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "profiles",
                        "emax_calibration_mi355x.md")
    rows = 0
    with open(path) as f:
        for line in f:
            cells = [c.strip() for c in line.strip().strip("|").split("|")]
            if len(cells) < 7 or cells[0] not in ("bf16", "f16", "f32", "f64", "f8", "f8e5m2"):
                continue
            dtype, n, plus20 = cells[0], int(cells[2]), float(cells[6])
            assert vb.vabft_default_emax(dtype, n, n) >= 1.25 * plus20, line
            rows += 1
    assert rows >= 40


def test_workspace_bytes(lib):
    p = vb.make_problem(4096, 4096, 4096, "bf16")
    assert vb.vabft_workspace_bytes(p) >= 16 * 4096 * 4
    assert vb.vabft_workspace_bytes(vb.make_problem(0, 4, 4, "f32")) == 0
    assert vb.vabft_workspace_bytes(vb.make_problem(4, 4, 4, 9)) == 0
    pt = vb.make_problem(4096, 11008, 4096, "bf16", transB=1)
    assert vb.vabft_workspace_bytes(pt) >= 86 * 3 * 4096 * 4


def test_rejects_bad_arguments_without_a_gpu(lib):
    p = vb.make_problem(8, 8, 8, "f32")
    # null pointers
    assert vb.vabft_encode(p, None, None, None, None, None, 0, None, check=False) == vb.VABFT_EINVAL
    assert vb.vabft_threshold(p, None, None, None, 1e-6, 2.5, None, None, None, None, check=False) == vb.VABFT_EINVAL
    assert vb.vabft_gemm_verified(p, None, None, None, None, None, 1, None, None, None, None, None, None, None, None, 0,
                                  None, check=False) == vb.VABFT_EINVAL
    # leading dimension smaller than the row, unknown dtype, bad transB
    for bad in (vb.make_problem(8, 8, 8, "f32", lda=4), vb.make_problem(8, 8, 8, 7), vb.make_problem(8, 8, 8, "f32", transB=2),
                vb.make_problem(8, 8, 8, "f32", transB=1, ldb=7), vb.make_problem(-1, 8, 8, "f32")):
        assert vb.vabft_encode(bad, 16, 16, 16, 16, 16, 1 << 20, None, check=False) == vb.VABFT_EINVAL
    # misaligned element pointer
    assert vb.vabft_encode(p, 18, 16, 16, 16, None, 0, None, check=False) == vb.VABFT_EINVAL
    with pytest.raises(vb.VabftError):
        vb.vabft_encode(p, None, None, None, None, None, 0, None)


_GEMM_CALLS = ["vabft_gemm_verified", "vabft_gemm_verified_fused", "vabft_gemm_verified_fused_static",
               "vabft_gemm_verified_weighted", "vabft_gemm_verified_rc", "vabft_gemm_verified_blocks",
               "vabft_gemm_verified_blocks_k"]


@pytest.mark.parametrize("entry", _GEMM_CALLS)
def test_empty_and_invalid_problems_are_refused_by_every_gemm_call(lib, entry):
    """A size of zero or below, an unknown type and no problem at all come back as EINVAL: nothing is computed from a
    problem (a workspace size, say) before it is known to be one.  In a process of its own, which a trap would end."""
    import subprocess
    import sys
    code = f"""
import ctypes, sys
sys.path.insert(0, {ROOT!r})
from paper_2602_08043_amd import binding as vb
f = getattr(vb.load(), {entry!r})
P = ctypes.POINTER(vb.Problem)
def call(p):
    return f(*[p if t is P else None if issubclass(t, (ctypes.c_void_p, ctypes._Pointer)) else t(1) for t in f.argtypes])
bad = [None]
for M, N, K, dt in ((8, 0, 8, 2), (8, -5, 8, 3), (8, -100, 8, 1), (0, 8, 8, 0), (-1, 8, 8, 4), (8, 8, 0, 3), (8, 8, -3, 5),
                    (8, 8, 8, 6), (8, 8, 8, -1), (0, 0, 0, 0)):
    p = vb.make_problem(8, 8, 8, "f32")
    p.M, p.N, p.K, p.dtype = M, N, K, dt
    bad.append(ctypes.byref(p))
assert [call(p) for p in bad] == [vb.VABFT_EINVAL] * len(bad)
"""
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, (entry, r.returncode, r.stderr[-500:])


def test_deferred_fold_arguments_without_a_gpu(lib):
    """d_S may be NULL for vabft_encode and vabft_gemm_verified_fused (the fold of S1..S3 deferred to the fused
    call): the argument checks then go on to the workspace, which is what these calls lack."""
    p = vb.make_problem(256, 256, 256, "f32")
    assert vb.vabft_encode(p, 16, 16, 16, None, None, 0, None, check=False) == vb.VABFT_EWORKSPACE
    assert vb.vabft_encode(p, 16, 16, 16, 24, None, 0, None, check=False) == vb.VABFT_EWORKSPACE
    # a misaligned d_S is still rejected when it is given
    assert vb.vabft_encode(p, 16, 16, 16, 20, None, 0, None, check=False) == vb.VABFT_EINVAL
    args = dict(d_astat=16, d_expected=16, d_T=16, inj=None, d_rowsum=16, d_E=16, d_flags=16, d_nflag=16, d_injlog=16,
                d_ninj=16, d_workspace=None, workspace_bytes=0)
    assert vb.vabft_gemm_verified_fused(p, 16, 16, 16, 16, None, 1e-6, 2.5, check=False, **args) == vb.VABFT_EWORKSPACE
    assert vb.vabft_gemm_verified_fused(p, 16, 16, 16, None, None, 1e-6, 2.5, check=False, **args) in (
        vb.VABFT_EINVAL, vb.VABFT_EWORKSPACE)
    # the workspace covers the partials of S1..S3 (three doubles per 16 rows of B) beside the GEMM's areas
    small, big = vb.make_problem(256, 256, 256, "f32"), vb.make_problem(256, 256, 16384, "f32")
    assert vb.vabft_workspace_bytes(big) - vb.vabft_workspace_bytes(small) >= (16384 - 256) // 16 * 24


def test_bench_line_stays_short():
    """The benchmark's one JSON line is kept whole only while it is short: its report of a full run in under 5000
    characters, figures of full length in every field it takes over."""
    import json
    import bench
    x = 123.45678901234567
    over = {k: x for k in ("cold_encode_included", "steady_state_B_preencoded", "three_call_route_B_preencoded",
                           "check_with_given_threshold")}
    r = {"name": "c3_bf16_ffn_and_more", "value": x, "ms_per_step": x, "frac_of_peak_whole_path": x, "plain_gemm_tflops": x,
         "plain_gemm_frac_of_peak": x, "overhead_pct": dict(over, method="m" * 100),
         "overhead_pct_interleaved_rounds": dict(over, method="m" * 100), "flags_in_timed_region": 0,
         "roofline": {"bound": "mfma", "achieved": x, "peak": x, "unit": "TFLOP/s", "frac": x, "traffic": 10 ** 9,
                      "kernel": "k" * 60, "avg_launch_ms": x, "measured_mfma_loop_tflops": x, "frac_of_measured_mfma_loop": x},
         "ms": {f"some_route_with_a_name_{i}": x for i in range(9)},
         "quality": {"fault_free_trials": 1000, "false_positive_trials": 0, "threshold_over_actual_mean": x,
                     "worst_row_E_over_T": x, "detection": {str(b): [x] * 9 for b in range(64)}},
         "cpu_baseline": {"value": x, "cores": 16, "kernel_time_s": x, "unit": "TFLOP/s", "sample": "s" * 120}}
    line = json.dumps(dict(bench.rounded(bench.brief(r, full=True)), configs=[bench.rounded(bench.brief(r, full=False))] * 6))
    assert len(line) < 4000, len(line)  # the contract's own fields take under 1000
    assert "method" not in line and "detection" not in line


def test_bench_refuses_more_than_one_gpu():
    """The path is built and measured on one GPU: bench.py --gpus N with N > 1 exits with a message, before
    anything touches a device."""
    import os
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, os.path.join(root, "bench.py"), "--gpus", "2"], capture_output=True, text=True,
                       timeout=120)
    assert r.returncode != 0
    assert "ONE GPU" in r.stderr and r.stdout.strip() == ""


def test_missing_library_fails_loudly(tmp_path):
    """There is no CPU fallback: loading a library that is not there raises, with the build command in the text."""
    missing = str(tmp_path / "libvabft_not_built.so")
    with pytest.raises(ImportError) as e:
        vb.load(missing)
    assert "has not been built" in str(e.value) and "no fallback" in str(e.value)


def test_asm_lint_flags_the_hazards_it_is_built_for():
    """The build-time hazard pass on the generated assembly of the inline-assembly kernels: each of its
    rules fires on a planted case and stays quiet on the padded form of the same sequence."""
    from paper_2602_08043_amd import asm_lint

    def kernel(body):
        return "_ZN5vabft18gemm16_fast_kernelIxEEv:\n" + body + "\n\ts_endpgm\n"

    asm = lambda text: "\t;;#ASMSTART\n\t" + text + "\n\t;;#ASMEND\n"
    # a scalar base written by the vector ALU and read by a load from assembly within five wait states
    bad = kernel("\tv_readfirstlane_b32 s4, v1\n" + asm("global_load_lds_dwordx4 v2, s[4:5] offset:0"))
    good = kernel("\tv_readfirstlane_b32 s4, v1\n\ts_nop 4\n" + asm("global_load_lds_dwordx4 v2, s[4:5] offset:0"))
    assert asm_lint.lint(bad) and not asm_lint.lint(good)
    # ... the same for a plain global load issued from assembly
    bad = kernel("\tv_readfirstlane_b32 s6, v1\n" + asm("global_load_dword v3, v2, s[6:7]"))
    good = kernel("\tv_readfirstlane_b32 s6, v1\n\ts_nop 4\n" + asm("global_load_dword v3, v2, s[6:7]"))
    assert asm_lint.lint(bad) and not asm_lint.lint(good)
    # the load directly behind the move that sets M0
    bad = kernel(asm("s_mov_b32 m0, s9") + asm("global_load_lds_dwordx4 v2, s[4:5] offset:0"))
    good = kernel(asm("s_mov_b32 m0, s9") + asm("v_mfma_f32_16x16x32_bf16 a[0:3], v[4:7], v[8:11], a[0:3]") +
                  asm("global_load_lds_dwordx4 v2, s[4:5] offset:0"))
    assert asm_lint.lint(bad) and not asm_lint.lint(good)
    # an operand of an MFMA from assembly written by the vector ALU within four wait states
    bad = kernel("\tv_cndmask_b32_e32 v4, v20, v21, vcc\n" + asm("v_mfma_f32_16x16x32_bf16 a[0:3], v[4:7], v[8:11], a[0:3]"))
    good = kernel("\tv_cndmask_b32_e32 v4, v20, v21, vcc\n\ts_nop 4\n" +
                  asm("v_mfma_f32_16x16x32_bf16 a[0:3], v[4:7], v[8:11], a[0:3]"))
    assert asm_lint.lint(bad) and not asm_lint.lint(good)
    mfma = asm("v_mfma_f32_16x16x32_bf16 a[4:7], v[4:7], v[8:11], a[4:7]")
    # a vector instruction, or a store, reads an accumulator that an MFMA from assembly wrote within eight wait states
    for read in ("\tv_accvgpr_read_b32 v4, a6\n", asm("v_accvgpr_read_b32 v4, a[6]"), "\tds_write_b128 v3, a[4:7]\n",
                 "\tv_mov_b64_e32 v[2:3], a[6:7]\n"):
        assert asm_lint.lint(kernel(mfma + read)), read
        assert asm_lint.lint(kernel(mfma + "\ts_nop 6\n" + read)), read
        assert not asm_lint.lint(kernel(mfma + "\ts_nop 7\n\ts_nop 1\n" + read)), read
    assert not asm_lint.lint(kernel(mfma + "\tv_accvgpr_read_b32 v4, a8\n"))  # another accumulator
    # an MFMA from assembly accumulates onto a register that a vector instruction wrote within four wait states
    for write in ("\tv_accvgpr_write_b32 a5, v30\n", asm("v_accvgpr_write_b32 a[7], 0")):
        assert asm_lint.lint(kernel(write + mfma)) and asm_lint.lint(kernel(write + "\ts_nop 2\n" + mfma)), write
        assert not asm_lint.lint(kernel(write + "\ts_nop 4\n" + mfma)), write
    assert not asm_lint.lint(kernel("\tv_accvgpr_write_b32 a9, v30\n" + mfma))
    # a kernel that names the registers of the chains (a[128] to a[255]) has one of them in an instruction of the compiler's
    chains = asm("v_accvgpr_write_b32 a[128], 0") + asm("v_accvgpr_read_b32 v4, a[255]")
    assert not asm_lint.lint(kernel(chains + "\tv_accvgpr_write_b32 a127, v1\n\tv_accvgpr_read_b32 v1, a64\n"))
    for use in ("v_accvgpr_write_b32 a130, v1", "v_accvgpr_read_b32 v1, a255", "v_mfma_f32_16x16x32_bf16 a[126:129], v[4:7], v[8:11], a[126:129]",
                "ds_write_b128 v3, a[200:203]", "v_accvgpr_mov_b32 a3, a128", "scratch_load_dword a130, off, s32"):
        assert asm_lint.lint(kernel(chains + "\t" + use + "\n")), use
        assert not asm_lint.lint(kernel("\t" + use + "\n")), use  # (of a kernel that has no such sums)


def test_native_calls_take_every_kind_of_pointer(lib):
    """Tensors, integers, None and ctypes pointers; what is none of them, a wrong count and a number that does not fit are
    Python errors, and nothing is called."""
    import ctypes
    torch = pytest.importorskip("torch")
    p = vb.make_problem(8, 8, 8, "f32")
    t = torch.zeros(64)
    call = lib.call_encode
    for ptr in (t, t.data_ptr(), ctypes.c_void_p(t.data_ptr())):  # as far as the check of the workspace, which is missing
        assert call(p, ptr, ptr, ptr, None, None, 0, None) == vb.VABFT_EWORKSPACE
        assert call(p, ptr, ctypes.c_void_p(None), ptr, None, None, 0, None) == vb.VABFT_EINVAL
    assert call(None, t, t, t, None, None, 0, None) == vb.VABFT_EINVAL
    for bad, error in (((p, "x", t, t, None, None, 0, None), AttributeError), ((p, t), TypeError),
                       ((p, t, t, t, None, None, -1, None), OverflowError), ((b"short", t, t, t, None, None, 0, None), TypeError)):
        with pytest.raises(error):
            call(*bad)
    with pytest.raises(OverflowError):
        lib.call_locate_correct(p, t, t, t, t, t, t, 1 << 40, t, t, t, None)


def test_native_calls_take_what_ctypes_takes_for_a_pointer(lib):
    """byref() with an offset, POINTER instances, arrays, c_size_t and numbers as text as a ctypes call takes them; what that
    refuses (another ctypes type, an array of numpy, another structure of the same size) is refused.  An address off by one byte
    is EINVAL here, an aligned one gets as far as the missing workspace."""
    import ctypes
    import numpy as np
    p = vb.make_problem(8, 8, 8, "f32")
    buf = (ctypes.c_float * 64)()
    at = ctypes.addressof(buf)

    class Subclass(vb.Problem):
        _fields_ = [("more", ctypes.c_int64)]

    def call(ptr, problem=p, size=0):
        return lib.call_encode(problem, ptr, buf, buf, None, None, size, None)

    off = (ctypes.c_float * 8).from_address(at + 1)
    for good, bad in ((ctypes.byref(buf), ctypes.byref(buf, 1)), (buf, off),
                      (ctypes.cast(at, ctypes.POINTER(ctypes.c_float)), ctypes.cast(at + 1, ctypes.POINTER(ctypes.c_float))),
                      (ctypes.c_void_p(at), ctypes.c_void_p(at + 1))):
        assert call(good) == vb.VABFT_EWORKSPACE and call(bad) == vb.VABFT_EINVAL
    assert call(buf, size=ctypes.c_size_t(1 << 20)) == vb.VABFT_EWORKSPACE
    assert call(buf, Subclass(8, 8, 8, vb.VABFT_F32, 0, 0, 8, 8, 8)) == vb.VABFT_EWORKSPACE
    assert lib.call_threshold(p, buf, buf, buf, "1e-6", 2, buf, None, buf, None) == vb.VABFT_EINVAL  # as float() reads it
    for refused in (ctypes.c_int(5), ctypes.c_size_t(at), np.zeros(64, np.float32), np.int64(at), 1.5, [at]):
        with pytest.raises(ctypes.ArgumentError):
            call(refused)
    assert ctypes.sizeof(vb.Inject) == ctypes.sizeof(vb.Problem)
    for other in (vb.Inject(), np.zeros(48, np.uint8), bytearray(48)):
        with pytest.raises(TypeError):
            call(buf, other)
    with pytest.raises(TypeError):
        lib.call_gemm_verified(p, buf, buf, buf, None, None, 0, p, None, None, None, None, None, None, None, 0, None)
    with pytest.raises(TypeError):
        call(buf, size=ctypes.c_int(5))


@pytest.mark.parametrize("method", ["encode", "threshold", "gemm", "gemm_fused", "encode_weighted", "threshold_weighted",
                                    "gemm_weighted", "encode_a", "threshold_cols", "gemm_rc", "encode_blocks",
                                    "threshold_blocks", "gemm_blocks", "check_offline"])
def test_session_operands_are_tensors(lib, method):
    """An address or nothing in the place of a tensor is an error of Python's, not a call with that address."""
    pytest.importorskip("torch")
    from paper_2602_08043_amd.session import VerifiedGemm

    class Any_(VerifiedGemm):
        def __init__(self):
            self.problem = vb.make_problem(8, 8, 8, "f32")
            self.dtype, self.M, self.N, self.K, self.W = "f32", 8, 8, 8, 64

        def __getattr__(self, name):  # any buffer of the session
            return None

        @staticmethod
        def _stream():
            return None

    for wrong in (4096, "x") + ((None,) if method != "check_offline" else ()):
        operands = (wrong, wrong) if method.startswith("gemm") else (wrong,)
        with pytest.raises(AttributeError, match="data_ptr"):
            getattr(Any_(), method)(*operands)
