"""The work whose time this repository watches: verified GEMMs through the public session API.

A case is one pass of one route of the library on device matrices that the program already holds:

  whole    encode of B, then the fused call (statistics of A, threshold, GEMM, compare)
  calls    the same in three calls: encode, threshold, verified GEMM
  encoded  the fused call alone: B is a weight whose checksum column and aggregates were formed once
  correct  weighted encode, weighted threshold, weighted GEMM, localisation and correction
  rc       row and column check of one GEMM
  blocks   block-wise verification over column blocks
  offline  post-hoc check of a stored product (whoever computed it) with B encoded before; some elements of the
           product are corrupted, so that rows are flagged

The fault injector is the test instrument of the library and no work of a user's, so no case switches it on.  The
verification difference E is not returned: on fault-free data it holds nothing but the rounding of the two vectors it
is the difference of, which are both returned.
"""
import math

import torch

from paper_2602_08043_amd.session import VerifiedGemm

C_SIGMA = 2.5
_DTYPE = {"f64": torch.float64, "f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16,
          "f8": torch.float8_e4m3fn, "f8e5m2": torch.float8_e5m2}
_BYTES = {"f64": 8, "f32": 4, "f16": 2, "bf16": 2, "f8": 1, "f8e5m2": 1}
_OUT_BYTES = {"f64": 8, "f32": 4, "f16": 2, "bf16": 2, "f8": 2, "f8e5m2": 2}
_BLOCK = {"f64": 64, "f32": 64, "f16": 256, "bf16": 256, "f8": 256, "f8e5m2": 256}


def _case(name, route, dtype, M, N, K, transB, data="normal", defer=False):
    c = {"route": route, "dtype": dtype, "M": M, "N": N, "K": K, "transB": transB, "data": data, "defer": defer}
    return {"name": name, **c} if name else c


def listed():
    return [
        # a small verified product in the middle of a solver: launches and latency are all there is
        _case("f32_256", "whole", "f32", 256, 256, 256, 0),
        # one decoding step of a served model: a few token rows against a weight encoded when it was loaded
        _case("bf16_decode", "encoded", "bf16", 24, 11008, 4096, 1, "ffn"),
        # a prefill whose token count is no multiple of anything, same weight
        _case("bf16_prefill", "encoded", "bf16", 1000, 11008, 4096, 1, "ffn"),
        # the same layer on a full batch
        _case("bf16_ffn", "encoded", "bf16", 4096, 11008, 4096, 1, "ffn"),
        # square product with both operands new, the benchmark's headline
        _case("bf16_4096", "whole", "bf16", 4096, 4096, 4096, 0, defer=True),
        # the largest product of the benchmark
        _case("f16_8192", "whole", "f16", 8192, 8192, 8192, 0, "uniform", defer=True),
        # sizes from data and not from a model: nothing is aligned
        _case("f16_odd", "whole", "f16", 1021, 1531, 2047, 0),
        # FP32 of ordinary, unround size
        _case("f32_ragged", "whole", "f32", 1000, 1200, 1500, 0),
        # FP64 product of a scientific code
        _case("f64_2048", "whole", "f64", 2048, 2048, 2048, 0, defer=True),
        # FP8 operands, weight layout
        _case("f8_4096", "whole", "f8", 4096, 4096, 4096, 1, defer=True),
        # a product that has to come out right: detection, localisation, correction
        _case("bf16_correct", "correct", "bf16", 1024, 1024, 1024, 0),
        # a product that a library computed, checked where it lies
        _case("bf16_offline", "offline", "bf16", 4096, 4096, 4096, 1),
    ]


# The most operations of a drawn case, per type: what keeps it below the largest listed one.
_MOST = {"bf16": 2e11, "f16": 2e11, "f8": 2e11, "f8e5m2": 2e11, "f32": 4e10, "f64": 1.7e10}


def _size(rng, lo, hi):
    """A size spread over the logarithm of lo..hi: half of them round, half as they fall, one in four of those odd."""
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    if rng.random() < 0.5:
        q = next(q for q in (256, 128, 64, 16, 1) if q <= max(1, v // 2))
        v = max(q, (v + q // 2) // q * q)
    elif rng.random() < 0.25:
        v |= 1
    return max(lo, min(hi, v))


def draw(rng):
    while True:
        route = rng.choice(["whole"] * 4 + ["encoded"] * 4 + ["calls", "correct", "rc", "blocks", "offline"])
        dtype = rng.choice(["bf16"] * 5 + ["f16"] * 3 + ["f32"] * 3 + ["f64", "f8", "f8e5m2"])
        transB = int(rng.random() < (0.8 if route == "encoded" else 0.4))
        M, N, K = _size(rng, 1, 8192), _size(rng, 64, 11008), _size(rng, 64, 11008)
        data = rng.choice(["normal", "uniform"] + (["ffn"] if transB and dtype in ("bf16", "f16") else []))
        if 2.0 * M * N * K <= _MOST[dtype]:
            return _case(None, route, dtype, M, N, K, transB, data, route == "whole" and rng.random() < 0.5)


def _emax(dtype, n):
    """The library's recommended e_max of a check made on accumulator values, for n = max(K, N)."""
    if dtype == "f64":
        return max(1.0e-17 * math.sqrt(n) + 2.5e-16, 8.0e-18 * math.sqrt(n) + 7.0e-16)
    if dtype in ("f8", "f8e5m2"):
        return 6.5e-6
    return max(5.0e-9 * math.sqrt(n) + 1.2e-7, 3.0e-9 * math.sqrt(n) + 4.2e-7)


def _emax_of(case):
    dt, N, K = case["dtype"], case["N"], case["K"]
    if case["route"] == "offline":  # two units in the last place of the stored type
        return {"bf16": 2.0 ** -7, "f16": 2.0 ** -10, "f8": 2.0 ** -10, "f8e5m2": 2.0 ** -10}.get(dt, _emax(dt, max(K, N)))
    if case["route"] == "blocks":
        N = min(N, _BLOCK[dt])
    return _emax(dt, max(K, N))


def _device():
    return torch.device("cuda:0" if torch.cuda.is_available() else "cpu")


def _inputs(case, seed):
    """A and B in storage type and layout, and for the offline route the stored product with its corrupted rows."""
    dev, dt = _device(), case["dtype"]
    M, N, K = case["M"], case["N"], case["K"]
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    gen = torch.float64 if dt == "f64" else torch.float32
    bshape = (N, K) if case["transB"] else (K, N)
    if case["data"] == "uniform":
        A = torch.rand((M, K), generator=g, device=dev, dtype=gen).mul_(2.0).sub_(1.0)
        B = torch.rand(bshape, generator=g, device=dev, dtype=gen).mul_(2.0).sub_(1.0)
    else:
        A = torch.randn((M, K), generator=g, device=dev, dtype=gen)
        B = torch.randn(bshape, generator=g, device=dev, dtype=gen)
        if case["data"] == "ffn":  # activations with outlier channels, weights of a trained layer's size
            A[:, torch.randperm(K, generator=g, device=dev)[:max(1, K // 100)]] *= 20.0
            B.clamp_(-2.0, 2.0).mul_(0.02)
    A, B = A.to(_DTYPE[dt]), B.to(_DTYPE[dt])
    if case["route"] != "offline":
        return A, B, None, None
    Bl = B.to(gen).t() if case["transB"] else B.to(gen)
    C = A.to(gen) @ Bl.contiguous()
    rows = torch.randperm(M, generator=g, device=dev)[:max(1, M // 512)]
    cols = torch.randint(N, rows.shape, generator=g, device=dev)
    C[rows, cols] = 30000.0
    out = torch.float16 if dt in ("f8", "f8e5m2") else _DTYPE[dt]
    return A, B, C.to(out), rows


def prepare(case, seed):
    A, B, C, _ = _inputs(case, seed)
    v = VerifiedGemm(case["M"], case["N"], case["K"], case["dtype"], case["transB"], log_capacity=64)
    if case["route"] in ("encoded", "offline"):
        v.encode(B)
    e_col = _emax(case["dtype"], max(case["K"], case["N"], case["M"]))
    return {"case": case, "v": v, "A": A, "B": B, "C": C, "e_max": _emax_of(case), "e_col": e_col}


def run(state):
    v, A, B, e, route = state["v"], state["A"], state["B"], state["e_max"], state["case"]["route"]
    if route == "whole":
        v.run_fused(A, B, e, C_SIGMA, defer_S=state["case"]["defer"])
    elif route == "calls":
        v.run(A, B, e, C_SIGMA)
    elif route == "encoded":
        v.gemm_fused(A, B, e, C_SIGMA)
    elif route == "correct":
        v.run_weighted(A, B, e, C_SIGMA)
    elif route == "rc":
        v.run_rc(A, B, e, state["e_col"], C_SIGMA)
    elif route == "blocks":
        v.run_blocks(A, B, e, C_SIGMA)
    else:
        v.threshold(A, e, C_SIGMA)
        v.check_offline(state["C"])
    return {k: getattr(v, k) for k in _outputs(state["case"])}


def _outputs(case):
    route = case["route"]
    if route == "blocks":
        return ["C", "Be_blk", "S_blk", "astat", "expected_blk", "T_blk", "rowsum_blk", "blockflags", "nblockflag",
                "flags", "nflag"]
    names = ["astat", "expected", "T", "rowsum", "flags", "nflag"]
    if route != "offline":
        names += ["C"]
    if route in ("whole", "calls", "correct", "rc"):
        names += ["Be", "bstat"]
        if not case["defer"]:
            names += ["S"]
    if route == "correct":
        names += ["Be2", "expected2", "rowsum2", "loc", "delta", "ncorrected"]
    if route == "rc":
        names += ["eA", "acolstat", "SA", "bcolstat", "expected_col", "T_col", "colsum", "colflags", "ncolflag"]
    return names


def work(case):
    """The product's operations and those of the checksums; each matrix of the route once, and its vectors."""
    M, N, K = case["M"], case["N"], case["K"]
    eb, ob, ab = _BYTES[case["dtype"]], _OUT_BYTES[case["dtype"]], 8 if case["dtype"] == "f64" else 4
    if case["route"] == "offline":
        return {"bytes": M * K * eb + M * N * ob + (K + 8 * M) * ab, "flops": 2.0 * M * K + M * N}
    vectors = (8 * M + 4 * K) * ab
    flops = 2.0 * M * N * K + 2.0 * M * K + M * N + (0 if case["route"] == "encoded" else K * N)
    return {"bytes": (M * K + K * N) * eb + M * N * ob + vectors, "flops": flops}


def tolerance(case):
    """The rounding of the stored product, or of FP32 / FP64 sums where the type stores those as they are: four times
    what the path shows against 64 bits."""
    if case["dtype"] == "bf16":
        return {"rel": 7e-3, "max": 1.6e-2}
    if case["dtype"] in ("f16", "f8", "f8e5m2"):
        return {"rel": 9e-4, "max": 2e-3}
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 2e-4}
    return {"rel": 2e-14, "max": 4e-13}


# ---- the same in 64 bits, from the definitions --------------------------------------------------------------------
def _stat(X, dim):
    """(max, min, mean) along a dimension, and the mean and the extrema bound of the variance."""
    mx, mn, mu = X.amax(dim), X.amin(dim), X.mean(dim)
    return torch.stack([mx, mn, mu], 1), mu, ((mx - mu) * (mu - mn)).clamp_min(0.0)


def _aggregates(mu, var):
    return torch.stack([mu.abs().sum(), var.sum(), (mu * mu).sum()])


def _threshold(mu, var, S, n, e_max):
    det = n * mu.abs() * S[0]
    var23 = C_SIGMA * torch.sqrt(n * mu * mu * S[1] + float(n) * n * var * S[2])
    var4 = C_SIGMA * math.sqrt(n) * var.sqrt() * S[1].sqrt()
    return e_max * (det + var23 + var4)


def exact(case, seed):
    A, B, C_stored, bad = _inputs(case, seed)
    M, N, e = case["M"], case["N"], _emax_of(case)
    if case["dtype"] in ("f8", "f8e5m2"):
        A, B = A.float(), B.float()
    A, B = A.double(), B.double()
    B = B.t().contiguous() if case["transB"] else B
    dev, i32 = A.device, torch.int32
    o = {}
    o["astat"], a_mu, a_var = _stat(A, 1)
    o["bstat"], b_mu, b_var = _stat(B, 1)
    o["Be"], o["S"] = B.sum(1), _aggregates(b_mu, b_var)
    o["expected"] = A @ o["Be"]
    o["T"] = _threshold(a_mu, a_var, o["S"], N, e)
    o["flags"], o["nflag"] = torch.zeros(M, dtype=i32, device=dev), torch.zeros(1, dtype=i32, device=dev)
    if case["route"] == "offline":
        o["rowsum"] = C_stored.double().sum(1)
        o["flags"][bad] = 1
        o["nflag"] += bad.numel()
        return {k: o[k] for k in _outputs(case)}
    o["C"] = A @ B
    o["rowsum"] = o["C"].sum(1)
    if case["route"] == "correct":
        w = torch.arange(1, N + 1, dtype=torch.float64, device=dev)
        o["Be2"] = B @ w
        o["expected2"], o["rowsum2"] = A @ o["Be2"], o["C"] @ w
        o["loc"] = torch.full((M,), -1, dtype=i32, device=dev)
        o["delta"], o["ncorrected"] = torch.zeros_like(o["T"]), torch.zeros_like(o["nflag"])
    elif case["route"] == "rc":
        o["eA"], o["colsum"] = A.sum(0), o["C"].sum(0)
        o["acolstat"], ac_mu, ac_var = _stat(A, 0)
        o["bcolstat"], bc_mu, bc_var = _stat(B, 0)
        o["SA"] = _aggregates(ac_mu, ac_var)
        o["expected_col"] = o["eA"] @ B
        o["T_col"] = _threshold(bc_mu, bc_var, o["SA"], M, _emax(case["dtype"], max(case["K"], N, M)))
        o["colflags"], o["ncolflag"] = torch.zeros(N, dtype=i32, device=dev), torch.zeros_like(o["nflag"])
    elif case["route"] == "blocks":
        W = _BLOCK[case["dtype"]]
        parts = {k: [] for k in ("Be_blk", "S_blk", "expected_blk", "T_blk", "rowsum_blk")}
        for t in range(0, N, W):
            Bt = B[:, t:t + W]
            _, mu, var = _stat(Bt, 1)
            S = _aggregates(mu, var)
            Be = Bt.sum(1)
            for k, x in (("Be_blk", Be), ("S_blk", S), ("expected_blk", A @ Be),
                         ("T_blk", _threshold(a_mu, a_var, S, Bt.shape[1], e)), ("rowsum_blk", o["C"][:, t:t + W].sum(1))):
                parts[k].append(x)
        o.update({k: torch.stack(x) for k, x in parts.items()})
        o["blockflags"] = torch.zeros(o["T_blk"].shape, dtype=i32, device=dev)
        o["nblockflag"] = torch.zeros_like(o["nflag"])
    return {k: o[k] for k in _outputs(case)}
