"""The work a program has this library do, as timed cases: layer forwards in the three formats, from one
decoded token to the largest prefill, in both packed layouts, and the offline preparation of a layer.

A case is a dict of plain values:
  op      "forward": quantizer + GEMM; "decode": wush_layer_decode (at most 64 tokens); "rtn": transforms +
          weight preparation; "gptq": the GPTQ case of the preparation
  fmt     "mxfp4", "nvfp4" or "int4"
  layout  "tiled" or "canonical" packed operands
  out     "bf16" or "f32" output of the GEMM
  rule    "nosat" or "ocp" (MXFP4 scale rule)
  M, K, N tokens (calibration tokens for the offline cases), input channels, output channels
"""
from __future__ import annotations

import math

import torch

import paper_2512_00956_amd.binding as P

LAMBDA = 1e-2
INT4_STEP = 0.33860793          # grid step over the group's root mean square
CALIBRATION_ROWS = 2048         # rows the prepared layers' transforms are built from

# largest 2 M K N a drawn forward pass may have, by (format, layout): what the largest listed cases take
_FLOP_CAP = {("mxfp4", "tiled"): 7.0e12, ("mxfp4", "canonical"): 1.0e12, ("nvfp4", "tiled"): 2.0e12,
             ("nvfp4", "canonical"): 1.0e12, ("int4", "tiled"): 2.0e12, ("int4", "canonical"): 1.0e12}


def _case(name, op, M, K, N, fmt="mxfp4", layout="tiled", out="bf16", rule="nosat"):
    c = {"op": op, "fmt": fmt, "layout": layout, "out": out, "rule": rule, "M": M, "K": K, "N": N}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one token of one sequence through the QKV projection of an 8B model: launches and latency
        _case("decode_1_token", "decode", 1, 4096, 6144),
        # a small decode batch through the gate+up projection of a 70B model: the weight stream from HBM
        _case("decode_16_tokens_wide", "decode", 16, 8192, 57344),
        # a larger, ragged decode batch through the down projection of an 8B model (few outputs, long K)
        _case("batch_100_tokens", "forward", 100, 14336, 4096),
        # prefill: 8B QKV, where one round of tiles fills the chip; 70B gate+up, the largest layer
        _case("prefill_2048", "forward", 2048, 4096, 6144),
        _case("prefill_8192_wide", "forward", 8192, 8192, 57344),
        # prefill of a caller that keeps the default descriptor (canonical packed operands): 8B down projection
        _case("default_layout_4096", "forward", 4096, 14336, 4096, layout="canonical"),
        # a layer whose sizes fit no tile (K an odd number of 32-blocks, odd N, odd M), FP32 output
        _case("ragged_777", "forward", 777, 1376, 3001, layout="canonical", out="f32", rule="ocp"),
        # the NVFP4 variant: prefill and a small decode batch on a 70B-sized projection
        _case("nvfp4_prefill_4096", "forward", 4096, 8192, 28672, fmt="nvfp4"),
        _case("nvfp4_16_tokens", "forward", 16, 8192, 28672, fmt="nvfp4"),
        # the INT4 variant: prefill of the 8B QKV projection
        _case("int4_prefill_2048", "forward", 2048, 4096, 6144, fmt="int4"),
        # offline, once per layer of a checkpoint: 8B QKV, round-to-nearest and GPTQ
        _case("prepare_rtn", "rtn", 4096, 4096, 6144),
        _case("prepare_gptq", "gptq", 4096, 4096, 6144),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    op = rng.choices(["forward", "decode", "rtn", "gptq"], [12, 3, 2, 1])[0]
    if op == "decode":
        K = 256 * max(1, round(_log(rng, 1024, 28672) / 256))
        N = max(64, round(_log(rng, 512, 57344)))
        return _case(None, op, max(1, round(_log(rng, 1, 64))), K, N, out=rng.choice(["bf16", "bf16", "f32"]),
                     rule=rng.choice(["nosat", "ocp"]))
    if op == "rtn":
        fmt = rng.choice(["mxfp4", "mxfp4", "nvfp4", "int4"])
        layout = rng.choice(["tiled", "canonical"])
        step = 32 if layout == "canonical" else (256 if fmt == "mxfp4" else 64)
        return _case(None, op, round(_log(rng, 512, 8192)), step * max(1, round(_log(rng, 512, 8192) / step)),
                     round(_log(rng, 256, 16384)), fmt=fmt, layout=layout)
    if op == "gptq":
        return _case(None, op, round(_log(rng, 512, 4096)), 256 * round(_log(rng, 512, 3072) / 256),
                     round(_log(rng, 256, 6144)))
    fmt = rng.choices(["mxfp4", "nvfp4", "int4"], [6, 3, 3])[0]
    layout = rng.choices(["tiled", "canonical"], [2, 1])[0]
    step = {"mxfp4": 256, "nvfp4": 64, "int4": 64}[fmt] if layout == "tiled" else (32 if fmt == "mxfp4" else 64)
    M = max(1, round(_log(rng, 1, 8192)))
    K = step * max(1, round(_log(rng, 512, 28672) / step))
    N = max(64, round(_log(rng, 256, 57344)))
    if rng.random() < 0.6:
        N = max(64, N // 64 * 64)
    cap = _FLOP_CAP[fmt, layout]
    if layout == "canonical" and fmt == "mxfp4" and K % 256:
        cap = 3.0e11
    while 2.0 * M * K * N > cap:
        if M >= 64:
            M = max(1, M // 2)
        else:
            N = max(64, N // 2)
    return _case(None, op, M, K, N, fmt=fmt, layout=layout, out=rng.choice(["bf16", "bf16", "bf16", "f32"]),
                 rule=rng.choice(["nosat", "ocp"]))


# ---------------------------------------------------------------------------
# inputs: activations with a per-channel scale spread and a few massive outlier channels, weights with a
# per-row scale spread, everything on the BF16 grid; transforms as a prepared checkpoint holds them
# ---------------------------------------------------------------------------
def _inputs(case, seed):
    M, K, N = case["M"], case["K"], case["N"]
    g = torch.Generator(device="cuda").manual_seed(int(seed))

    def normal(*shape):
        return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32)

    scale = torch.exp(normal(K))
    outliers = torch.randperm(K, generator=g, device="cuda")[:max(1, K // 200)]
    scale[outliers] *= 50.0

    def activations(rows):
        return (normal(rows, K) * scale).bfloat16()

    X = activations(M)
    row_scale = 0.02 * torch.exp(0.5 * normal(N, 1))
    W = torch.empty((N, K), dtype=torch.bfloat16, device="cuda")
    for r in range(0, N, 8192):
        W[r:r + 8192] = (normal(min(8192, N - r), K) * row_scale[r:r + 8192]).bfloat16()
    X_cal = None if case["op"] in ("rtn", "gptq") else activations(min(CALIBRATION_ROWS, max(512, M)))
    return X, W, X_cal


def _block(case):
    return 16 if case["fmt"] == "nvfp4" else 32


def _hadamard(d):
    h = torch.ones((1, 1), dtype=torch.float64)
    while h.shape[0] < d:
        h = torch.cat([torch.cat([h, h], 1), torch.cat([h, -h], 1)])
    return h / math.sqrt(d)


def _moments(A, d):
    """[K/d][d][d] second moments (FP64) of the blocks of A [rows][K]."""
    rows, K = A.shape
    M = torch.zeros((K // d, d, d), dtype=torch.float64, device=A.device)
    for r in range(0, rows, 2048):
        a = A[r:r + 2048].double().reshape(-1, K // d, d).permute(1, 2, 0).contiguous()
        M += torch.bmm(a, a.transpose(1, 2).contiguous())
    return M / rows


def _wush(M_W, M_X, lam):
    """T_wush of every block from its second moments (FP64, on the CPU)."""
    d = M_W.shape[-1]
    eye = torch.eye(d, dtype=torch.float64)

    def factor(m):
        tr = m.diagonal(dim1=1, dim2=2).sum(1)[:, None, None]
        return torch.linalg.cholesky(m + lam * tr / d * eye)

    Wp, Xp = factor(M_W.cpu()), factor(M_X.cpu())
    U, s, _ = torch.linalg.svd(Wp.transpose(1, 2) @ Xp)
    pick = U.abs().argmax(1, keepdim=True)
    U = U * torch.where(torch.gather(U, 1, pick) < 0, -1.0, 1.0)
    return _hadamard(d) @ (s.rsqrt()[:, :, None] * (U.transpose(1, 2) @ Wp.transpose(1, 2)))


def _transforms(case, W, X_cal):
    d = _block(case)
    return _wush(_moments(W[:CALIBRATION_ROWS], d), _moments(X_cal, d), LAMBDA).to(torch.bfloat16).cuda().contiguous()


def _apply(A, T):
    """A [rows][K] with its blocks multiplied by T [K/d][d][d] on the right, transposed: sum_k A[., k] T[j][k] (FP64)."""
    rows, K = A.shape
    d = T.shape[-1]
    a = A.double().reshape(rows, K // d, d).transpose(0, 1).contiguous()
    t = T.double().transpose(1, 2).contiguous()
    return torch.bmm(a, t).transpose(0, 1).reshape(rows, K)


def _activation_scale(X_cal, T):
    """NVFP4 tensor scale of the activations, calibrated with some room above the calibration maximum."""
    return (1.25 * _apply(X_cal, T).abs().max() / (6.0 * 448.0)).float().reshape(1)


# ---------------------------------------------------------------------------
# the calls
# ---------------------------------------------------------------------------
def _layout(case):
    return P.WUSH_LAYOUT_TILED if case["layout"] == "tiled" else P.WUSH_LAYOUT_CANONICAL


def _out(case):
    return P.WUSH_OUT_F32 if case["out"] == "f32" else P.WUSH_OUT_BF16


def _fmt(case):
    return P.default_fmt(scale_rule=P.WUSH_SCALE_OCP_FLOOR if case["rule"] == "ocp" else P.WUSH_SCALE_NOSAT,
                         out_dtype=_out(case), layout=_layout(case))


def _packed(case, rows):
    """Zeroed buffers of a packed [rows][K] operand."""
    K = case["K"]
    if case["fmt"] == "mxfp4":
        cb, sb = P.wush_packed_sizes(rows, K, _fmt(case))
    else:
        cb, sb = P.wush_packed_sizes_nvfp4(rows, K, _layout(case))
    return (torch.zeros(cb, dtype=torch.uint8, device="cuda"), torch.zeros(sb, dtype=torch.uint8, device="cuda"))


def _bytes(n):
    return torch.zeros(n, dtype=torch.uint8, device="cuda")


def _prepare_weight(s):
    case = s["case"]
    if case["fmt"] == "mxfp4":
        P.wush_prepare_weight(s["W"], s["T"], s["Wq"], s["Ws"], s["workspace"], s["fmt"])
    elif case["fmt"] == "nvfp4":
        P.wush_prepare_weight_nvfp4(s["W"], s["T"], s["Wq"], s["Ws"], s["tsw"], s["workspace"], s["layout"])
    else:
        P.wush_prepare_weight_int4(s["W"], s["T"], s["Wq"], s["Ws"], s["workspace"], s["layout"])


def _weight_workspace(case):
    if case["fmt"] == "nvfp4":
        return P.wush_prepare_weight_nvfp4_workspace(case["K"])
    return P.wush_prepare_weight_workspace(case["N"], case["K"])


def prepare(case, seed):
    X, W, X_cal = _inputs(case, seed)
    M, K, N, d = case["M"], case["K"], case["N"], _block(case)
    s = {"case": case, "fmt": _fmt(case), "layout": _layout(case), "out": _out(case), "W": W}
    s["Wq"], s["Ws"] = _packed(case, N)
    s["tsw"] = torch.zeros(1, dtype=torch.float32, device="cuda")
    if case["op"] in ("rtn", "gptq"):
        s["X_cal"] = X
        s["T"] = torch.zeros((K // d, d, d), dtype=torch.bfloat16, device="cuda")
        if case["op"] == "gptq":
            s["workspace"] = _bytes(P.wush_prepare_weight_gptq_workspace(N, K))
        else:
            s["moments"] = _bytes(P.wush_build_transforms_workspace(K))
            s["workspace"] = _bytes(_weight_workspace(case))
        return s
    s["T"] = _transforms(case, W, X_cal)
    s["workspace"] = _bytes(_weight_workspace(case))
    _prepare_weight(s)
    del s["W"], s["workspace"]
    s["X"] = X
    s["Y"] = torch.zeros((M, N), dtype=torch.float32 if case["out"] == "f32" else torch.bfloat16, device="cuda")
    if case["op"] == "decode":
        s["workspace"] = _bytes(P.wush_layer_decode_workspace(K))
        P.wush_layer_decode_init(s["workspace"], K)
        return s
    s["Xq"], s["Xs"] = _packed(case, M)
    if case["fmt"] == "nvfp4":
        s["tsx"] = _activation_scale(X_cal, s["T"])
    return s


def run(s):
    case = s["case"]
    op, fmt, K = case["op"], case["fmt"], case["K"]
    if op == "decode":
        P.wush_layer_decode(s["X"], s["T"], s["Wq"], s["Ws"], s["Y"], s["workspace"], s["fmt"])
        return s["Y"]
    if op == "gptq":
        P.wush_prepare_weight_gptq(s["W"], s["X_cal"], LAMBDA, s["T"], s["Wq"], s["Ws"], s["workspace"], s["fmt"])
        return [s["T"], s["Wq"], s["Ws"]]
    if op == "rtn":
        build = P.wush_build_transforms_nvfp4 if fmt == "nvfp4" else P.wush_build_transforms
        build(s["W"], s["X_cal"], LAMBDA, s["T"], s["moments"])
        _prepare_weight(s)
        return [s["T"], s["Wq"], s["Ws"]] + ([s["tsw"]] if fmt == "nvfp4" else [])
    if fmt == "mxfp4":
        P.wush_quantize_act(s["X"], s["T"], s["Xq"], s["Xs"], s["fmt"])
        P.wush_linear(s["Xq"], s["Xs"], s["Wq"], s["Ws"], s["Y"], s["fmt"], K=K)
    elif fmt == "nvfp4":
        P.wush_quantize_act_nvfp4(s["X"], s["T"], s["tsx"], s["Xq"], s["Xs"], s["layout"])
        P.wush_linear_nvfp4(s["Xq"], s["Xs"], s["tsx"], s["Wq"], s["Ws"], s["tsw"], s["Y"], s["layout"], s["out"], K=K)
    else:
        P.wush_quantize_act_int4(s["X"], s["T"], s["Xq"], s["Xs"], s["layout"])
        P.wush_linear_int4(s["Xq"], s["Xs"], s["Wq"], s["Ws"], s["Y"], s["layout"], s["out"], K=K)
    return [s["Xq"], s["Xs"], s["Y"]]


# ---------------------------------------------------------------------------
# what a pass cannot do without, how far two correct passes may differ, and the 64-bit results
# ---------------------------------------------------------------------------
def work(case):
    M, K, N, d = case["M"], case["K"], case["N"], _block(case)
    per_scale = {"mxfp4": 32, "nvfp4": 16, "int4": 16}[case["fmt"]]     # codes per scale byte
    packed = 0.5 + 1.0 / per_scale
    T = 2.0 * K * d
    if case["op"] in ("rtn", "gptq"):
        # moments of both operands, the block product and the codes; the factorizations of K/d blocks are small.
        flops = 2.0 * (M + N) * K * d + 2.0 * N * K * d
        if case["op"] == "gptq":
            # symmetric Hessian, its Cholesky factor and triangular inverse, inter- and intra-block propagation
            flops = M * K * K + K ** 3 / 3.0 + K ** 3 / 3.0 + N * K * K + 8.0 * N * K * d
        return {"bytes": 2.0 * (M + N) * K + T + packed * N * K, "flops": flops}
    moved = 2.0 * M * K + T + packed * N * K + (4.0 if case["out"] == "f32" else 2.0) * M * N
    if case["op"] == "forward":
        moved += 2.0 * packed * M * K
    return {"bytes": moved, "flops": 2.0 * M * K * N + 2.0 * M * K * d}


def tolerance(case):
    if case["op"] in ("rtn", "gptq"):
        # FP64 throughout: another summation order moves a transform entry across a BF16 rounding boundary
        # or a weight across a code boundary once in a great while (with GPTQ the rest of its row follows)
        return {"rel": 1e-4, "max": 0.01, "differ": 1e-4}
    if case["out"] == "f32":
        return {"rel": 1e-5, "max": 1e-4}      # 32-bit sums of exact products; packed codes and scales are equal
    return {"rel": 4e-3, "max": 0.02}          # BF16 output


def _e2m1(v):
    mids = torch.tensor([0.25, 0.75, 1.25, 1.75, 2.5, 3.5, 5.0], dtype=torch.float64, device=v.device)
    grid = torch.tensor([0.0, 0.5, 1.0, 1.5, 2.0, 3.0, 4.0, 6.0], dtype=torch.float64, device=v.device)
    a = v.abs()
    lo, hi = torch.bucketize(a, mids), torch.bucketize(a, mids, right=True)
    code = torch.where((lo != hi) & (lo % 2 == 1), hi, lo)            # ties to the even code
    return torch.where(torch.signbit(v), -grid[code], grid[code])


def _mxfp4_scale(amax, rule):
    mant, e = torch.frexp(amax)                                        # amax = mant 2^e, mant in [0.5, 1)
    E = e - 3 if rule == "ocp" else torch.where(mant <= 0.75, e - 3, e - 2)
    E = torch.where(amax == 0, -127, E).clamp(-127, 127)
    return torch.ldexp(torch.ones_like(amax), E)


def _quantized(Y, case, ts=None):
    """Values of Y [rows][K] (FP64) after quantization."""
    rows, K = Y.shape
    fmt = case["fmt"]
    G = Y.reshape(rows, K // _block(case), _block(case))
    if fmt == "mxfp4":
        s = _mxfp4_scale(G.abs().amax(-1, keepdim=True), case["rule"])
        q = _e2m1(G / s) * s
    elif fmt == "nvfp4":
        r = (G.abs().amax(-1, keepdim=True) / (6.0 * ts)).clamp(max=448.0)
        _, e = torch.frexp(r)
        step = torch.ldexp(torch.ones_like(r), (e - 1).clamp(min=-6) - 3)
        s = (torch.round(r / step) * step).clamp(max=448.0) * ts
        q = torch.where(s == 0, 0.0, _e2m1(G / torch.where(s == 0, 1.0, s)) * s)
    else:
        s = (INT4_STEP * (G * G).mean(-1, keepdim=True).sqrt()).to(torch.bfloat16).double()
        q = torch.where(s == 0, 0.0, torch.round(G / torch.where(s == 0, 1.0, s)).clamp(-8, 7) * s)
    return q.reshape(rows, K)


def _exact_forward(case, X, W, X_cal):
    T = _transforms(case, W, X_cal)
    Tinv = torch.linalg.inv(T.double().cpu()).to(T.device).transpose(1, 2).contiguous()
    tsx = tsw = None
    if case["fmt"] == "nvfp4":
        tsx = _activation_scale(X_cal, T).double()
        top = torch.stack([_apply(W[r:r + 4096], Tinv).abs().max() for r in range(0, case["N"], 4096)]).max()
        tsw = (top / (6.0 * 448.0)).float().double()
    Xd = torch.cat([_quantized(_apply(X[r:r + 4096], T), case, tsx) for r in range(0, case["M"], 4096)])
    Y = torch.empty((case["M"], case["N"]), dtype=torch.float64, device="cuda")
    for r in range(0, case["N"], 4096):
        Wd = _quantized(_apply(W[r:r + 4096], Tinv), case, tsw)
        Y[:, r:r + 4096] = Xd @ Wd.T.contiguous()
    return Y


def _exact_gptq(case, X, W):
    M, K, N = case["M"], case["K"], case["N"]
    Xd = X.double()
    H = Xd.T.contiguous() @ Xd / M
    Hd = H.cpu()
    Hd += LAMBDA * Hd.trace() / K * torch.eye(K, dtype=torch.float64)
    L = torch.linalg.cholesky(torch.linalg.inv(Hd))
    W, Ld = W.double(), L.cuda()
    T = torch.empty((K // 32, 32, 32), dtype=torch.float64)
    for i in range(K // 32):
        b, rest = slice(32 * i, 32 * i + 32), slice(32 * i + 32, K)
        Wi = W[:, b].contiguous()
        T[i] = _wush((Wi.T.contiguous() @ Wi / N)[None], H[b, b][None], LAMBDA)[0]
        Ti = T[i].to(torch.bfloat16).double()
        Lii = L[b, b]
        Hbar = Ti @ torch.linalg.inv(Lii @ Lii.T) @ Ti.T
        R = torch.linalg.cholesky(torch.linalg.inv(Hbar)).T.contiguous().cuda()
        Y = Wi @ torch.linalg.inv(Ti).cuda()
        s = _mxfp4_scale(Y.abs().amax(1), case["rule"])
        Q = torch.empty_like(Y)
        for r in range(32):
            Q[:, r] = _e2m1(Y[:, r] / s) * s
            Y[:, r + 1:] -= ((Y[:, r] - Q[:, r]) / R[r, r])[:, None] * R[r, r + 1:]
        E = Q @ Ti.cuda() - Wi
        W[:, rest] += E @ (Ld[rest, b] @ torch.linalg.inv(Lii).cuda()).T.contiguous()
    return T


def exact(case, seed):
    X, W, X_cal = _inputs(case, seed)
    if case["op"] == "gptq":
        # Every transform past the first depends on the codes before it, and one code that rounds the other
        # way moves all that follow: beyond some 32 blocks two correct FP64 runs part now and then.
        return [_exact_gptq(case, X, W), None, None] if case["K"] <= 1024 else None
    if case["op"] == "rtn":
        d = _block(case)
        T = _wush(_moments(W, d), _moments(X, d), LAMBDA)
        tsw = []
        if case["fmt"] == "nvfp4":
            Tinv = torch.linalg.inv(T.to(torch.bfloat16).double()).cuda().transpose(1, 2).contiguous()
            tsw = torch.stack([_apply(W[r:r + 4096], Tinv).abs().max() for r in range(0, case["N"], 4096)]).max()
            tsw = [(tsw / (6.0 * 448.0)).reshape(1)]
        return [T, None, None] + tsw
    Y = _exact_forward(case, X, W, X_cal)
    return Y if case["op"] == "decode" else [None, None, Y]
