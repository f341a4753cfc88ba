"""vabft_encode_gemm_fused and vabft_encode_gemm_weighted refuse a wrong argument before they launch anything."""
import math

import pytest

vb = pytest.importorskip("paper_2602_08043_amd.binding")

OK = 1 << 20  # an address, aligned for everything
INVALID, WORKSPACE = vb.VABFT_EINVAL, vb.VABFT_EWORKSPACE


def _inject(**kw):
    inj = vb.Inject()
    inj.mode, inj.rate, inj.bit_lo, inj.bit_hi, inj.log_capacity = 2, 0.5, 0, 31, 0
    for k, v in kw.items():
        setattr(inj, k, v)
    return inj


COMMON = [("dA", None, INVALID), ("dA", OK + 1, INVALID), ("dB", None, INVALID), ("dC", None, INVALID), ("dC", OK + 2, INVALID),
          ("d_Be", None, INVALID), ("d_bstat", OK + 2, INVALID), ("d_S", OK + 4, INVALID), ("e_max", 0.0, INVALID),
          ("e_max", math.nan, INVALID), ("c_sigma", -1.0, INVALID), ("c_sigma", math.inf, INVALID), ("d_astat", None, INVALID),
          ("d_astat", OK + 2, INVALID), ("d_expected", None, INVALID), ("d_T", OK + 1, INVALID), ("d_rowsum", None, INVALID),
          ("d_E", OK + 2, INVALID), ("d_flags", None, INVALID), ("d_nflag", OK + 1, INVALID), ("d_workspace", None, WORKSPACE),
          ("d_workspace", OK + 8, WORKSPACE), ("workspace_bytes", 0, WORKSPACE), ("workspace_bytes", "encode", WORKSPACE)]
FUSED = [("inj", _inject(mode=3), INVALID), ("inj", _inject(rate=1.5), INVALID), ("inj", _inject(bit_hi=32), INVALID),
         ("inj", _inject(log_capacity=4), INVALID)]
WEIGHTED = [("d_Be2", None, INVALID), ("d_S", None, INVALID), ("d_expected2", OK + 2, INVALID), ("d_rowsum2", None, INVALID),
            ("correct", 2, INVALID), ("d_loc", OK + 2, INVALID), ("d_delta", None, INVALID), ("d_ncorrected", OK + 1, INVALID)]


def _arguments(weighted, buffers=None):
    names = ["dA", "dB", "dC", "d_Be"] + (["d_Be2"] if weighted else []) + ["d_bstat", "d_S", "e_max", "c_sigma", "d_astat", "d_expected"]
    names += ["d_expected2", "d_T"] if weighted else ["d_T", "inj"]
    names += ["d_rowsum"] + (["d_rowsum2"] if weighted else []) + ["d_E", "d_flags", "d_nflag"]
    names += ["correct", "d_loc", "d_delta", "d_ncorrected"] if weighted else ["d_injlog", "d_ninj"]
    args = dict.fromkeys(names + ["d_workspace"], OK)
    args.update(buffers or {}, e_max=1e-6, c_sigma=2.5)
    args.update({"correct": 1} if weighted else {"inj": None, "d_injlog": None})
    return args


def _call(weighted, p, args, room, change):
    name, value, _ = change
    args = {**args, "workspace_bytes": room, name: value}
    if args["workspace_bytes"] == "encode":  # room for the encode of B, none for the product's partials
        args["workspace_bytes"] = vb.vabft_workspace_bytes(vb.make_problem(1, p.N, p.K, "f32", p.transB))
        assert args["workspace_bytes"] < room
    call = vb.vabft_encode_gemm_weighted if weighted else vb.vabft_encode_gemm_fused
    room = args.pop("workspace_bytes")
    return call(p, *args.values(), room, None, check=False)


CASES = [(w, c) for w in (False, True) for c in COMMON + (WEIGHTED if w else FUSED)]


@pytest.mark.parametrize("weighted,change", CASES, ids=["%s-%s-%d" % ("weighted" if w else "fused", c[0], i)
                                                        for i, (w, c) in enumerate(CASES)])
def test_status(weighted, change):
    p = vb.make_problem(4096, 512, 64, "f32", 0)
    assert _call(weighted, p, _arguments(weighted), vb.vabft_workspace_bytes(p), change) == change[2]


@pytest.mark.gpu
@pytest.mark.parametrize("weighted", [False, True])
def test_nothing_is_written(weighted):
    import torch

    from paper_2602_08043_amd.session import VerifiedGemm

    for transB in (0, 1):
        v = VerifiedGemm(4096, 512, 64, "f32", transB)
        g = torch.Generator(device="cuda").manual_seed(1)
        A = torch.randn(4096, 64, generator=g, device="cuda")
        B = torch.randn((512, 64) if transB else (64, 512), generator=g, device="cuda")
        outputs = {"dC": v.C, "d_Be": v.Be, "d_bstat": v.bstat, "d_S": v.S, "d_astat": v.astat, "d_expected": v.expected, "d_T": v.T,
                   "d_rowsum": v.rowsum, "d_E": v.E, "d_flags": v.flags, "d_nflag": v.nflag, "d_workspace": v.ws}
        outputs.update({"d_Be2": v.Be2, "d_expected2": v.expected2, "d_rowsum2": v.rowsum2, "d_loc": v.loc, "d_delta": v.delta,
                        "d_ncorrected": v.ncorrected} if weighted else {"d_ninj": v.ninj})
        for t in outputs.values():
            t.zero_()
        args = _arguments(weighted, {k: t.data_ptr() for k, t in {"dA": A, "dB": B, **outputs}.items()})
        for change in COMMON + (WEIGHTED if weighted else FUSED):
            assert _call(weighted, v.problem, args, v.ws_bytes, change) == change[2], change[0]
        torch.cuda.synchronize()
        for k, t in outputs.items():
            assert not bool(t.any()), k
