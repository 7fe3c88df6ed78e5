"""What a user of this library has it do, as cases that can be timed and compared.

A case is one pass through the Python binding of the C ABI, the way the README and bench.py call it: weights are
quantized once and kept (a trainer re-quantizes them per optimizer step: the "train" cases), activations are
quantized on every pass.  Five operations:

  layer    one linear layer with its fused norm: quantize X, FP8 GEMM + norm ("two"), or the one-launch forms
           loka_fp8_linear_norm ("fused", inference: no FP8 copy of X leaves) and loka_fp8_linear_norm_xq ("xq",
           training: codes and scales of X are handed back)
  mlp      two layers chained through the FP8-output epilogue (codes and row scales of the hidden activation)
  train    one training step of a layer: both quantized forms of W, forward, dX = dY W^T, dW = X^T dY
  probe    LoKA-Probe on a layer: FP8 output kept in fp32, BF16 reference GEMM, error statistics
  tracker  the online mean / covariance tracker merges one batch

Values follow synth.py: N(0, 1), Student-t(4) / sqrt 2 (heavy tails) or N(0, 1) with four channels x 100 (outliers)
for activations, N(0, 1/K) for weights, N(0, 0.02^2) for output gradients; drawn on the GPU from the seed.
"""
from __future__ import annotations

import math

import torch

from paper_2605_10886_amd import binding as B

EPS = 1e-5
_RECIPES = {"row": (B.SCALE_ROW, B.SCALE_COL), "tensor": (B.SCALE_TENSOR, B.SCALE_TENSOR),
            "block": (B.SCALE_BLOCK_1x128, B.SCALE_BLOCK_128x128),
            "block_pow2": (B.SCALE_BLOCK_1x128_POW2, B.SCALE_BLOCK_128x128_POW2)}
_MAX_FLOPS = 2.0 * 32768 * 4096 * 4096       # the largest listed case; no drawn case costs more


def _layer(M, K, N, batch=1, norm="layernorm", affine=False, recipe="row", call="two", dist="normal", **name):
    return dict(name, op="layer", M=M, K=K, N=N, batch=batch, norm=norm, affine=affine, recipe=recipe, call=call, dist=dist)


def _mlp(M, K, H, N, norm="layernorm", affine=False, dist="normal", **name):
    return dict(name, op="mlp", M=M, K=K, H=H, N=N, norm=norm, affine=affine, dist=dist)


def _train(M, K, N, norm="layernorm", dist="normal", **name):
    return dict(name, op="train", M=M, K=K, N=N, norm=norm, dist=dist)


def _probe(M, K, N, norm="layernorm", recipe="row", dist="normal", **name):
    return dict(name, op="probe", M=M, K=K, N=N, norm=norm, recipe=recipe, dist=dist)


def _tracker(M, K, **name):
    return dict(name, op="tracker", M=M, K=K)


def listed():
    return [
        # C1 of the benchmark: the smallest call there is; launches and host work count
        _layer(256, 128, 128, name="layer_256x128x128"),
        # the narrowest layer of the paper's throughput study at its batch of 2048, with learned gamma and beta: an
        # ordinary layer of a small-batch step
        _layer(2048, 256, 768, affine=True, name="layer_2048x256x768"),
        # C2: an MLP layer with heavy-tailed input and RMSNorm, in the one-launch form a trainer uses
        _layer(16384, 512, 512, norm="rmsnorm", call="xq", dist="student_t4", name="layer_16384x512x512_xq"),
        # ragged rows, K a multiple of 16 only, N no multiple of anything wider: feature widths as they come
        _layer(5013, 1008, 720, affine=True, name="layer_5013x1008x720"),
        # C3: the skinny up / down pair, hidden activation handed over in FP8
        _mlp(65536, 256, 1024, 256, name="mlp_65536x256x1024x256"),
        # C4: 64 grouped small layers (inference form, nothing but the output leaves)
        _layer(4096, 256, 256, batch=64, norm="rmsnorm", call="fused", name="layer_64x4096x256x256_fused"),
        # blockwise scales at a mid-sized layer with outlier channels: the recipe the dispatcher picks under a tight budget
        _layer(8192, 2048, 2048, recipe="block", dist="normal_outlier4", name="layer_8192x2048x2048_block"),
        # C5: the large layer the benchmark's headline is quoted on
        _layer(32768, 4096, 4096, dist="normal_outlier4", name="layer_32768x4096x4096"),
        # the widest layer of the paper's throughput study
        _layer(2048, 123200, 1024, name="layer_2048x123200x1024"),
        # forward and backward of the C3a layer, weights quantized in the step as after an optimizer update
        _train(65536, 256, 1024, name="train_65536x256x1024"),
        # the probe on a mid-sized layer: BF16 reference GEMM and statistics
        _probe(16384, 1024, 1024, norm="rmsnorm", dist="student_t4", name="probe_16384x1024x1024"),
        # the tracker on a layer input of 1024 features
        _tracker(32768, 1024, name="tracker_32768x1024"),
    ]


def _log(rng, lo, hi, step=1):
    """A multiple of `step` in [lo, hi], spread evenly over the logarithm."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(lo, min(hi, int(round(v / step)) * step))


def _rows(rng, lo, hi, flops_per_row, step=1):
    """Rows of the same kind, so that the case costs no more than the largest listed one."""
    hi = max(lo, min(hi, int(_MAX_FLOPS / flops_per_row)))
    return _log(rng, lo, hi, step)


def draw(rng):
    op = rng.choices(("layer", "fused", "xq", "mlp", "train", "probe", "tracker"), (40, 8, 10, 10, 12, 10, 10))[0]
    dist = rng.choice(("normal", "student_t4", "normal_outlier4"))
    norm = rng.choice(("layernorm", "layernorm", "rmsnorm"))
    affine = rng.random() < 0.4
    if op == "fused":       # whole rows of X in one wave or workgroup: N <= 256 and a short K
        K, N = rng.choice((128, 256, 512)), _log(rng, 64, 256, 16)
        batch = rng.choice((1, 1, 8, 32, 64))
        return _layer(_log(rng, 512, 131072 // batch), K, N, batch, norm, affine, "row", "fused", dist)
    if op == "xq":          # weights that fit the register file of a CU
        K = rng.choice((128, 256, 512, 1024))
        N = _log(rng, 64, min(1024, (1 << 18) // K), 16)
        return _layer(_log(rng, 512, 131072), K, N, 1, norm, affine, "row", "xq", dist)
    if op == "mlp":
        K, H, N = _log(rng, 128, 2048, 128), _log(rng, 128, 4096, 128), _log(rng, 64, 2048, 16)
        return _mlp(_rows(rng, 256, 65536, 2.0 * H * (K + N)), K, H, N, norm, affine, dist)
    if op == "train":       # the batch is a contraction of the weight gradient: scale groups of 128 rows
        K, N = _log(rng, 128, 2048, 128), _log(rng, 128, 2048, 128)
        return _train(_rows(rng, 1024, 65536, 6.0 * K * N, 128), K, N, norm, dist)
    if op == "probe":
        K, N = _log(rng, 64, 4096, 16), _log(rng, 64, 4096, 16)
        return _probe(_rows(rng, 512, 32768, 4.0 * K * N), K, N, norm, "row", dist)
    if op == "tracker":
        K = _log(rng, 64, 4096, 8)
        return _tracker(_rows(rng, 1024, 65536, 1.0 * K * K), K)
    # layers at large: any rows, features a multiple of 16, often (as in practice) of 128
    step = rng.choice((16, 128))
    recipe = rng.choices(("row", "tensor", "block", "block_pow2"), (60, 10, 22, 8))[0]
    norm = rng.choices(("layernorm", "rmsnorm", "none", "blocknorm"), (45, 25, 15, 15))[0]
    if recipe.startswith("block") or norm == "blocknorm":
        step = 128
    K, N = _log(rng, max(64, step), 8192, step), _log(rng, max(64, step), 4096, step)
    if norm == "blocknorm":
        N, affine = max(256, N // 256 * 256), False
    batch = rng.choice((1, 1, 1, 1, 4, 16)) if recipe == "row" else 1
    M = _rows(rng, 64, 65536 // batch, 2.0 * K * N * batch)
    return _layer(M, K, N, batch, norm, affine, recipe, "two", dist)


# ---------------------------------------------------------------------------------------------------- inputs
def _activations(g, rows, cols, dist):
    """[rows, cols] bf16 on the GPU, drawn in slabs (the widest matrix does not need its fp32 copy at once)."""
    x = torch.empty(rows, cols, dtype=torch.bfloat16, device="cuda")
    hot = torch.randperm(cols, generator=g, device="cuda")[:4] if dist == "normal_outlier4" else None
    slab = max(1, min(rows, (1 << 26) // cols))
    for r in range(0, rows, slab):
        n = min(slab, rows - r)
        z = torch.randn(n, cols, generator=g, device="cuda")
        if dist == "student_t4":
            chi = torch.zeros_like(z)
            for _ in range(4):
                c = torch.randn(n, cols, generator=g, device="cuda")
                chi.addcmul_(c, c)
            z.div_(chi.mul_(0.5).sqrt_())            # t_4 / sqrt 2
        elif hot is not None:
            z[:, hot] *= 100.0
        x[r:r + n] = z
    return x


def _weight(g, K, N):
    return (torch.randn(K, N, generator=g, device="cuda") / math.sqrt(K)).to(torch.bfloat16)


def _affine(g, N, norm, on):
    if not on or norm not in ("layernorm", "rmsnorm"):
        return None, None
    gamma = (1.0 + 0.25 * torch.randn(N, generator=g, device="cuda")).to(torch.bfloat16)
    beta = (0.1 * torch.randn(N, generator=g, device="cuda")).to(torch.bfloat16)
    return gamma, beta if norm == "layernorm" else None


def _desc(M, N, K, batch, recipe, norm):
    xm, wm = _RECIPES[recipe]
    block_n, act = (256, B.ACT_HARDSWISH) if norm == "blocknorm" else (0, B.ACT_NONE)
    return B.make_desc(M, N, K, batch, xm, wm, B.NORMS[norm], EPS, block_n=block_n, act=act)


def prepare(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    op, M, K = case["op"], case["M"], case["K"]
    s = {"op": op}
    if op == "tracker":
        mean = 4.0 * torch.rand(K, generator=g, device="cuda") - 2.0
        spread = 0.25 + 1.5 * torch.rand(K, generator=g, device="cuda")
        z = torch.randn(M, K, generator=g, device="cuda")
        z[:, 1:] += 0.6 * z[:, :-1].clone()          # neighbouring features are correlated
        s.update(x=z.mul_(spread).add_(mean).to(torch.bfloat16), n=0, mu=torch.zeros(K, device="cuda"),
                 sigma=torch.zeros(K, K, device="cuda"))
        return s
    N, norm = case["N"], case["norm"]
    if op == "layer":
        batch, recipe = case["batch"], case["recipe"]
        xm, wm = _RECIPES[recipe]
        ws = [B.loka_quantize(_weight(g, K, N), wm, transpose_out=True) for _ in range(batch)]
        s.update(call=case["call"], x=_activations(g, batch * M, K, case["dist"]), x_mode=xm,
                 wq=torch.cat([q for q, _ in ws]), sw=torch.cat([sc for _, sc in ws]),
                 desc=_desc(M, N, K, batch, recipe, norm))
        s["gamma"], s["beta"] = _affine(g, N, norm, case["affine"])
    elif op == "mlp":
        H = case["H"]
        s.update(x=_activations(g, M, K, case["dist"]),
                 up=B.loka_quantize(_weight(g, K, H), B.SCALE_COL, transpose_out=True),
                 down=B.loka_quantize(_weight(g, H, N), B.SCALE_COL, transpose_out=True),
                 desc_up=_desc(M, H, K, 1, "row", norm), desc_down=_desc(M, N, H, 1, "row", norm))
        s["gamma"], s["beta"] = _affine(g, H, norm, case["affine"])
        s["gamma2"], s["beta2"] = _affine(g, N, norm, case["affine"])
    elif op == "train":
        s.update(x=_activations(g, M, K, case["dist"]), w=_weight(g, K, N),
                 dy=(0.02 * torch.randn(M, N, generator=g, device="cuda")).to(torch.bfloat16),
                 desc=_desc(M, N, K, 1, "row", norm), desc_dx=_desc(M, K, N, 1, "row", "none"),
                 desc_dw=_desc(K, N, M, 1, "block", "none"))
    else:
        w = _weight(g, K, N)
        s.update(x=_activations(g, M, K, case["dist"]), w=w, x_mode=_RECIPES[case["recipe"]][0],
                 wq=B.loka_quantize(w, _RECIPES[case["recipe"]][1], transpose_out=True),
                 desc=_desc(M, N, K, 1, case["recipe"], norm))
    return s


# ---------------------------------------------------------------------------------------------------- one pass
def run(s):
    op = s["op"]
    if op == "layer":
        if s["call"] == "fused":
            out, _, _ = B.loka_fp8_linear_norm(s["desc"], s["x"], s["wq"], s["sw"], s["gamma"], s["beta"])
            return {"out": out}
        if s["call"] == "xq":
            out, _, xq, sx = B.loka_fp8_linear_norm_xq(s["desc"], s["x"], s["wq"], s["sw"], s["gamma"], s["beta"])
            return {"out": out, "xq": xq, "sx": sx}
        xq, sx = B.loka_quantize(s["x"], s["x_mode"])
        out, _ = B.loka_fp8_gemm_norm(s["desc"], xq, sx, s["wq"], s["sw"], s["gamma"], s["beta"])
        return {"out": out, "xq": xq, "sx": sx}
    if op == "mlp":
        xq, sx = B.loka_quantize(s["x"], B.SCALE_ROW)
        hq, sh, _ = B.loka_fp8_gemm_norm_fp8out(s["desc_up"], xq, sx, *s["up"], s["gamma"], s["beta"])
        out, _ = B.loka_fp8_gemm_norm(s["desc_down"], hq, sh, *s["down"], s["gamma2"], s["beta2"])
        return {"out": out, "xq": xq, "sx": sx, "hq": hq, "sh": sh}
    if op == "train":
        x, w, dy = s["x"], s["w"], s["dy"]
        wq, sw = B.loka_quantize(w, B.SCALE_COL, transpose_out=True)
        xq, sx = B.loka_quantize(x, B.SCALE_ROW)
        out, _ = B.loka_fp8_gemm_norm(s["desc"], xq, sx, wq, sw)
        wq_k, sw_k = B.loka_quantize(w, B.SCALE_ROW)                                # W as it lies, one scale per k
        dyq, sdy = B.loka_quantize(dy, B.SCALE_ROW)
        dx, _ = B.loka_fp8_gemm_norm(s["desc_dx"], dyq, sdy, wq_k, sw_k)
        xt, sxt = B.loka_quantize(x, B.SCALE_BLOCK_128x1, transpose_out=True)       # groups along the batch
        dyt, sdyt = B.loka_quantize(dy, B.SCALE_BLOCK_128x128, transpose_out=True)
        dw, dw32 = B.loka_fp8_gemm_norm(s["desc_dw"], xt, sxt, dyt, sdyt, want_y=True)
        return {"out": out, "dx": dx, "dw": dw, "dw32": dw32}
    if op == "probe":
        xq, sx = B.loka_quantize(s["x"], s["x_mode"])
        out, y = B.loka_fp8_gemm_norm(s["desc"], xq, sx, *s["wq"], want_y=True)
        yref = B.loka_bf16_gemm(s["desc"], s["x"], s["w"])
        stats, rowmax = B.loka_probe_error(y, yref, sync=False)
        return {"out": out, "y": y, "yref": yref, "stats": stats, "rowmax": rowmax}
    s["n"] = B.loka_tracker_update(s["x"], s["n"], s["mu"], s["sigma"])
    return {"mu": s["mu"], "sigma": s["sigma"]}


# ---------------------------------------------------------------------------------------------------- work, tolerance
def work(case):
    """Bytes that have to be read and written once, and the operations of the matrix products."""
    op, M, K = case["op"], case["M"], case["K"]
    if op == "tracker":
        return {"bytes": 2.0 * M * K + 8.0 * K * (K + 1), "flops": 1.0 * M * K * (K + 1)}
    N = case["N"]
    if op == "layer":
        b = case["batch"]
        codes = 0.0 if case["call"] == "fused" else M * (K + 4.0)
        return {"bytes": b * (2.0 * M * K + codes + N * (K + 4.0) + 2.0 * M * N), "flops": 2.0 * b * M * K * N}
    if op == "mlp":
        H = case["H"]
        return {"bytes": M * (3.0 * K + 4.0) + M * (H + 4.0) + 2.0 * M * N + H * (K + N + 4.0), "flops": 2.0 * M * H * (K + N)}
    if op == "train":
        return {"bytes": 2.0 * (M * K + K * N + M * N) + 2.0 * (M * N + M * K) + 6.0 * K * N, "flops": 6.0 * M * K * N}
    return {"bytes": 2.0 * M * K + K * N * 3.0 + M * N * (2.0 + 4.0 + 4.0) + 4.0 * M, "flops": 4.0 * M * K * N}


def tolerance(case):
    """About four times what each path differs from itself with its products and norms in 64 bits (same codes in):
    bf16 outputs 2e-4 to 5e-4 in the 2-norm and two roundings at most; an mlp's hidden codes flip for 0.1 to 0.25 %
    of the values and carry 1e-3 to 3e-3 into its output; the tracker's fp32 sums 1e-7 to 5e-6.  Codes and scales
    of a quantized activation are the same bytes (no "differ")."""
    op = case["op"]
    if op == "tracker":
        return {"rel": 2e-5, "max": 2.5e-4}
    if op == "mlp":
        return {"rel": 1e-2, "max": 0.5, "differ": 1e-2}
    return {"rel": 2e-3, "max": 3.2e-2}
