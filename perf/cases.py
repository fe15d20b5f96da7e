"""What the performance of this library is measured on: its own operations at the sizes they are used at.

Three programs use the library.  A trainer quantizes the master weights each step and takes the fused forward with the
objective and the straight-through backward at r = 8/4/2; a calibrator adds the affine re-parameterisation and the
clip factors; a server slices the codes to packed planes once, then reads prompts through the fused forward at the one
bit-width it serves and decodes through the GEMV and the feed-forward stack.  `listed()` holds one point of each path
and direction, from the unit-test layer (16 tokens, 256 x 256) to the layer the headline figure is quoted on; `draw()`
takes other points of the same ranges.  Sizes are those of `synth.py`, the tests and `bench.py`, with ragged token
counts where prompts and samples are ragged.
"""
from __future__ import annotations

import math
import zlib

import torch

import paper_2502_06786_amd as mq

TRAIN_BITS = (8, 4, 2)


def listed():
    return [
        # -- decode: one token step of one matrix, small batches ----------------------------------------------------
        # the smallest call a server makes: one sequence through a square 7B-shaped projection
        {"name": "decode_one", "kind": "gemv", "B": 1, "N": 4096, "K": 4096, "r": 4, "extra": "none", "lend": False},
        # a few sequences through a 7B-shaped gate matrix at two bits
        {"name": "decode_few", "kind": "gemv", "B": 4, "N": 14336, "K": 4096, "r": 2, "extra": "none", "lend": False},
        # a full decode batch through the long rows of a down matrix, scratch memory lent by the server
        {"name": "decode_down", "kind": "gemv", "B": 16, "N": 4096, "K": 14336, "r": 4, "extra": "none", "lend": True},
        # the extra-precision model: int2 plane and overflow list of a 27B-shaped gate matrix (5 % of the weights)
        {"name": "decode_extra", "kind": "gemv", "B": 2, "N": 36864, "K": 4608, "r": 2, "extra": "list", "lend": False},
        # a whole Mix'n'Match stack, int2 at the ends and int8 in the middle (7B-shaped layers)
        {"name": "decode_stack", "kind": "stack", "B": 3, "d": 4096, "F": 14336, "bits": "2,2,4,8,8,4,2,2"},
        # -- prompts and evaluation: the forward alone --------------------------------------------------------------
        # a short prompt at the served bit-width
        {"name": "prompt_short", "kind": "forward", "M": 77, "N": 4096, "K": 4096, "bits": "4", "extra": False},
        # a long prompt, ragged, at two bits
        {"name": "prompt_long", "kind": "forward", "M": 2011, "N": 14336, "K": 4096, "bits": "2", "extra": False},
        # -- training -----------------------------------------------------------------------------------------------
        # the smallest layer: launches and host work
        {"name": "train_tiny", "kind": "train", "M": 16, "N": 256, "K": 256},
        # the layer of the headline figure: 9B-shaped gate, 8192 tokens
        {"name": "train_layer", "kind": "train", "M": 8192, "N": 14336, "K": 3584},
        # the whole gated feed-forward block of the 2B-shaped model, 4096 tokens
        {"name": "train_block", "kind": "block", "M": 4096, "d": 2304, "F": 9216},
        # one calibration step of a 2B-shaped down matrix on one ragged sample
        {"name": "calibrate", "kind": "calibrate", "M": 1999, "N": 2304, "K": 9216},
        # -- model preparation --------------------------------------------------------------------------------------
        # master weights to codes, served planes and overflow list (9B-shaped gate)
        {"name": "planes", "kind": "planes", "N": 14336, "K": 3584, "hot": 0.03},
    ]


def _log(rng, lo, hi, step=1):
    """A multiple of `step` in lo..hi, spread over the logarithm."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(-(-lo // step), min(hi // step, round(v / step))) * step


def draw(rng):
    kind = rng.choice(["gemv"] * 5 + ["forward"] * 4 + ["train"] * 4 + ["stack", "block", "calibrate", "planes"])
    if kind == "gemv":
        while True:
            c = {"kind": kind, "B": rng.randint(1, 16), "N": _log(rng, 896, 73728), "K": _log(rng, 1024, 36864, 128),
                 "r": rng.choice([2, 2, 4, 4, 8, 3, 6]), "extra": "none", "lend": rng.random() < 0.5}
            if rng.random() < 0.25:
                c.update(r=2, extra=rng.choice(["list", "dense"]), lend=False)
            if c["N"] * c["K"] <= 73728 * 4608:
                return c
    if kind == "stack":
        d = _log(rng, 1024, 4608, 128)
        return {"kind": kind, "B": rng.randint(1, 16), "d": d, "F": _log(rng, 2 * d, 3 * d + 2048, 128),
                "bits": ",".join(str(rng.choice([2, 4, 8])) for _ in range(rng.randint(2, 8)))}
    if kind == "planes":
        return {"kind": kind, "N": _log(rng, 512, 14336), "K": _log(rng, 1024, 9216, 16), "hot": rng.choice([0.0, 0.02, 0.05])}
    while True:
        N, K = _log(rng, 896, 14336, 16), _log(rng, 896, 14336, 16)
        if kind == "forward":
            c = {"kind": kind, "M": _log(rng, 17, 4096), "N": N, "K": K, "bits": rng.choice(["2", "4", "8", "3", "8,4,2", "4,2"]),
                 "extra": rng.random() < 0.2}
            work = c["M"] * N * K
        elif kind == "block":
            c = {"kind": kind, "M": _log(rng, 128, 4096), "d": _log(rng, 512, 2304, 16), "F": _log(rng, 1024, 9216, 16)}
            work = 3 * c["M"] * c["d"] * c["F"]
        else:
            c = {"kind": kind, "M": _log(rng, 16, 8192) if kind == "train" else _log(rng, 500, 4096), "N": N, "K": K}
            work = c["M"] * N * K * (1 if kind == "train" else 2)
        if work <= 8192 * 14336 * 3584:
            return c


# --------------------------------------------------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------------------------------------------------
class _Rand:
    """Seeded draws on the GPU."""

    def __init__(self, seed, what):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed((seed * 1_000_003 + zlib.crc32(what.encode())) % (1 << 62))

    def normal(self, *shape, scale=1.0):
        return torch.randn(*shape, generator=self.g, device="cuda").mul_(scale)

    def uniform(self, n, lo, hi):
        return torch.rand(n, generator=self.g, device="cuda") * (hi - lo) + lo

    def weight(self, N, K, scale):
        """fp32 N(0, scale^2), one entry of a thousand eight times as large (the outlier weights of the 9B-shaped layer)."""
        W = self.normal(N, K, scale=scale)
        W[torch.rand(N, K, generator=self.g, device="cuda") < 1e-3] *= 8.0
        return W

    def bf16(self, *shape, scale=1.0):
        return self.normal(*shape, scale=scale).to(torch.bfloat16)

    def codes(self, N, K, first_hot, hot):
        """uint8 codes, a share `hot` of them in first_hot..255 and the rest below (trained extra-precision models)."""
        q = torch.randint(0, first_hot, (N, K), generator=self.g, device="cuda", dtype=torch.uint8)
        top = torch.randint(first_hot, 256, (N, K), generator=self.g, device="cuda", dtype=torch.int16).to(torch.uint8)
        return torch.where(torch.rand(N, K, generator=self.g, device="cuda") < hot, top, q)


def _bits(case):
    return tuple(int(v) for v in case["bits"].split(","))


def _ws(op, M, N, K, nr):
    return torch.empty(max(16, mq.mq_workspace_bytes(op, M, N, K, nr)), dtype=torch.uint8, device="cuda")


def _interleaved(gate, up):
    W = torch.empty(2 * gate.shape[0], gate.shape[1], device="cuda")
    W[0::2], W[1::2] = gate, up
    return W


def prepare(case, seed):
    rnd = _Rand(seed, case["kind"])
    return {"case": case, **_PREPARE[case["kind"]](case, rnd)}


def _prepare_gemv(c, rnd):
    B, N, K, r = c["B"], c["N"], c["K"], c["r"]
    s = {"x": rnd.bf16(B, K), "y": torch.empty(B, N, dtype=torch.bfloat16, device="cuda"), "ovf": None}
    if c["extra"] == "none":
        Q, a, z = mq.mq_quantize_int8(rnd.weight(N, K, 0.02))
        s["plane"] = mq.mq_slice(Q, r, packed=True)
    else:
        # the overflow bucket of an int2 slice starts at code 224
        Q = rnd.codes(N, K, 224, 0.05)
        a, z = rnd.uniform(N, 3e-4, 6e-4), rnd.uniform(N, 100.0, 150.0)
        if c["extra"] == "list":
            s["plane"], s["ovf"] = mq.mq_slice(Q, r, packed=True, extra_precision=True, capacity=N * K // 8)
        else:
            s["plane"] = mq.mq_slice(Q, r, packed=True, extra_precision=True, dense_ep=True)
    s["a"], s["z"] = mq.mq_params_to_bf16(a, z)
    s["ws"] = _ws(mq.MQ_OP_GEMV, B, N, K, r) if c["lend"] else None
    return s


def _prepare_stack(c, rnd):
    B, d, F = c["B"], c["d"], c["F"]
    layers = []
    for r in _bits(c):
        Qg, ag, zg = mq.mq_quantize_int8(rnd.weight(2 * F, d, d ** -0.5))
        # the residual stream keeps its size over the layers, as in a trained model
        Qd, ad, zd = mq.mq_quantize_int8(rnd.weight(d, F, 0.12 * F ** -0.5))
        ag, zg = mq.mq_params_to_bf16(ag, zg)
        ad, zd = mq.mq_params_to_bf16(ad, zd)
        layers.append({"gate_up": mq.mq_slice(Qg, r, packed=True), "down": mq.mq_slice(Qd, r, packed=True),
                       "alpha_gu": ag, "zero_gu": zg, "alpha_dn": ad, "zero_dn": zd, "r": r})
    return {"x": rnd.bf16(B, d), "layers": layers, "y": torch.empty(B, d, dtype=torch.bfloat16, device="cuda"),
            "ws": _ws(mq.MQ_OP_FFN_DECODE, B, F, d, 1)}


def _prepare_forward(c, rnd):
    Q, a, z = mq.mq_quantize_int8(rnd.weight(c["N"], c["K"], 0.02))
    return {"X": rnd.bf16(c["M"], c["K"]), "Q": Q, "a": a, "z": z}


def _prepare_train(c, rnd):
    W, X = rnd.weight(c["N"], c["K"], 0.015), rnd.bf16(c["M"], c["K"])
    # y': the output of the unquantized layer
    return {"W": W, "X": X, "T": X @ W.to(torch.bfloat16).t()}


def _prepare_block(c, rnd):
    M, d, F = c["M"], c["d"], c["F"]
    Qg, ag, zg = mq.mq_quantize_int8(_interleaved(rnd.weight(F, d, d ** -0.5), rnd.weight(F, d, d ** -0.5)))
    Qd, ad, zd = mq.mq_quantize_int8(rnd.weight(d, F, F ** -0.5))
    return {"X": rnd.bf16(M, d), "gu": (Qg, ag, zg), "down": (Qd, ad, zd), "dY": [rnd.bf16(M, d, scale=1e-3) for _ in TRAIN_BITS]}


def _prepare_calibrate(c, rnd):
    M, N, K = c["M"], c["N"], c["K"]
    W, X = rnd.weight(N, K, 0.02), rnd.bf16(M, K)
    return {"W": W, "X": X, "T": X @ W.to(torch.bfloat16).t(), "gamma": rnd.uniform(N, 0.8, 1.0), "beta": rnd.uniform(N, 0.8, 1.0),
            "s": rnd.uniform(K, 0.5, 1.5), "delta": rnd.normal(K, scale=0.05)}


def _prepare_planes(c, rnd):
    W = rnd.normal(c["N"], c["K"], scale=0.02)
    if c["hot"]:
        # the full upper bucket of a trained extra-precision model: this share of the codes, and the top 2 % of the rest,
        # overflow at r = 2
        W = W.clamp_(max=0.06)
        W[torch.rand(W.shape, generator=rnd.g, device="cuda") < c["hot"]] = 0.06
    cap = max(16, int(0.08 * W.numel()))
    ovf = mq.Overflow(c["N"], cap)
    ovf.col_idx.zero_()
    return {"W": W, "ovf": ovf}


_PREPARE = {"gemv": _prepare_gemv, "stack": _prepare_stack, "forward": _prepare_forward, "train": _prepare_train,
            "block": _prepare_block, "calibrate": _prepare_calibrate, "planes": _prepare_planes}


# --------------------------------------------------------------------------------------------------------------------
# one pass
# --------------------------------------------------------------------------------------------------------------------
def run(state):
    return _RUN[state["case"]["kind"]](state, state["case"])


def _run_gemv(s, c):
    if c["extra"] == "dense":
        return mq.mq_gemv_sliced_dense_ep(s["x"], s["plane"], s["a"], s["z"], c["r"], c["K"], y=s["y"])
    if c["lend"]:
        return mq.mq_gemv_sliced_ws(s["x"], s["plane"], s["a"], s["z"], c["r"], c["K"], y=s["y"], ws=s["ws"])
    return mq.mq_gemv_sliced(s["x"], s["plane"], s["a"], s["z"], c["r"], c["K"], ovf=s["ovf"], y=s["y"])


def _run_stack(s, c):
    return mq.mq_ffn_mixnmatch(s["x"], s["layers"], c["F"], silu=True, residual=True, y=s["y"], ws=s["ws"])


def _run_forward(s, c):
    return mq.mq_linear_fwd_multi(s["X"], s["Q"], s["a"], s["z"], _bits(c), extra_precision=c["extra"])


def _run_train(s, c):
    lam = (0.1, 0.1, 1.0)
    Q, a, z = mq.mq_quantize_int8(s["W"])
    losses, dY = mq.mq_linear_fwd_multi_l2(s["X"], Q, a, z, TRAIN_BITS, s["T"], None, lam)
    dX, dW = mq.mq_linear_bwd(s["X"], Q, a, z, dY, None, TRAIN_BITS)
    return {"losses": losses, "dX": dX, "dW": dW}


def _run_block(s, c):
    rs = TRAIN_BITS
    GU, A = mq.mq_linear_fwd_multi_gated(s["X"], *s["gu"], rs)
    Y, dA, dWd = [], [], None
    for i, r in enumerate(rs):
        Y += mq.mq_linear_fwd_multi(A[i], *s["down"], (r,))
    for i, r in enumerate(rs):
        d, dWd = mq.mq_linear_bwd(A[i], *s["down"], [s["dY"][i]], None, (r,), dW=dWd, accumulate_dW=i > 0)
        dA.append(d)
    dX, dWgu = mq.mq_linear_bwd_gated(s["X"], *s["gu"], GU, dA, None, rs)
    return {"Y": Y, "dX": dX, "dWgu": dWgu, "dWd": dWd}


def _run_calibrate(s, c):
    rs = TRAIN_BITS
    Ws, bias = mq.mq_affine_weight(s["W"], s["s"], s["delta"], None)
    Xt = mq.mq_affine_input(s["X"], s["s"], s["delta"])
    Q, a, z = mq.mq_quantize_int8(Ws, s["gamma"], s["beta"])
    losses, dY = mq.mq_linear_fwd_multi_l2(Xt, Q, a, z, rs, s["T"], None, (0.1, 0.1, 1.0), bias=bias)
    dXt, dWs = mq.mq_linear_bwd(Xt, Q, a, z, dY, None, rs)
    dgamma, dbeta = mq.mq_linear_bwd_clip(Ws, Xt, Q, a, z, dY, None, rs, s["gamma"], s["beta"])
    ddelta, ds, dc = mq.mq_affine_bwd(s["X"], dXt, s["W"], dWs, dY, None, s["s"], s["delta"])
    return {"losses": losses, "dX": dXt, "dW": dWs, "dgamma": dgamma, "dbeta": dbeta, "ddelta": ddelta, "ds": ds, "dc": dc}


def _run_planes(s, c):
    Q, a, z = mq.mq_quantize_int8(s["W"])
    planes, ovf = mq.mq_slice_multi(Q, (4, 2), ovf_r=2, ovf=s["ovf"])
    a16, z16 = mq.mq_params_to_bf16(a, z)
    return {"Q": Q, "alpha": a, "zero": z, "planes": planes, "row_ptr": ovf.row_ptr, "col_idx": ovf.col_idx, "nnz": ovf.nnz,
            "a16": a16, "z16": z16}


_RUN = {"gemv": _run_gemv, "stack": _run_stack, "forward": _run_forward, "train": _run_train, "block": _run_block,
        "calibrate": _run_calibrate, "planes": _run_planes}


# --------------------------------------------------------------------------------------------------------------------
# what a pass cannot do without
# --------------------------------------------------------------------------------------------------------------------
def work(case):
    c, kind = case, case["kind"]
    if kind == "gemv":
        B, N, K, r = c["B"], c["N"], c["K"], c["r"]
        byts = N * K * (r + (c["extra"] == "dense")) // 8 + 4 * N + 2 * B * (K + N)
        if c["extra"] == "list":
            byts += 4 * N + 2 * int(0.05 * N * K)
        return {"bytes": byts, "flops": 2 * B * N * K}
    if kind == "stack":
        B, d, F = c["B"], c["d"], c["F"]
        codes = 3 * d * F
        return {"bytes": sum(codes * r // 8 + 4 * (2 * F + d) for r in _bits(c)) + 4 * B * d, "flops": 2 * B * codes * len(_bits(c))}
    if kind == "planes":
        n = c["N"] * c["K"]
        return {"bytes": 4 * n + n + n // 2 + n // 4 + 2 * int((c["hot"] + 0.02 if c["hot"] else 0.0) * n) + 16 * c["N"], "flops": 0}
    n = len(TRAIN_BITS)
    if kind == "block":
        M, d, F = c["M"], c["d"], c["F"]
        # stacked layer: forward and dX per bit-width, one dW; down layers: forward, dX, dW per bit-width
        return {"bytes": 3 * d * F * (1 + 4) + 2 * M * d * (2 + 2 * n), "flops": (4 * n + 2) * M * 2 * F * d + 6 * n * M * d * F}
    M, N, K = c["M"], c["N"], c["K"]
    if kind == "forward":
        nr = len(_bits(c))
        return {"bytes": N * K + 8 * N + 2 * M * K + 2 * nr * M * N, "flops": 2 * nr * M * N * K}
    byts = 4 * N * K + 2 * M * K + 2 * M * N + 2 * M * K + 4 * N * K          # W, X, y' in; dX, dW out
    if kind == "train":
        return {"bytes": byts, "flops": (4 * n + 2) * M * N * K}
    return {"bytes": byts + 16 * (N + K), "flops": (6 * n + 2) * M * N * K}


def tolerance(case):
    """Four times what another order of the sums (the reduced dimension permuted) and a float64 evaluation show.

    Outputs are rounded once to bf16 from fp32 sums: against float64 that is 1.7e-3 of the norm, and two correct
    implementations differ by one step (2^-7 of a value at most) where a sum falls next to a boundary between two bf16
    numbers.  Gradients also see the rounding of their operands; in a stack or a block the roundings of a layer are the
    next one's inputs."""
    kind = case["kind"]
    if kind == "planes":
        return "exact"
    if kind in ("gemv", "forward"):
        return {"rel": 6e-3, "max": 0.032}
    if kind == "stack":
        return {"rel": 0.016, "max": 0.08}
    if kind == "block":
        return {"rel": 0.012, "max": 0.12}
    return {"rel": 6e-3, "max": 0.05}
