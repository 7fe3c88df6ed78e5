"""The static choice between tile sizes and schedules: shapes at the edges of the smaller tiles, rounds of workgroups past
one per slot, the 256 x 256 split-K and BF16 forms with ragged edges, and calls with less scratch than the choice wants."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2605_10886_amd import binding as B
from paper_2605_10886_amd import synth
from test_gpu_gemm_norm import RECIPES, _run_case

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _rows(M, n=24):
    return np.unique(np.concatenate([np.arange(2), np.linspace(0, M - 1, n).round().astype(int), [M - 2, M - 1]]))


@pytest.mark.parametrize("variant,shape,recipe", [
    ("panel32x256", (9001, 256, 528), "row"),          # more tiles than two per CU: several rounds of row panels
    ("panel64x256", (12321, 144, 784), "row"),
    ("panel128x128", (6500, 256, 640), "block"),
    ("panel32x256", (33, 128, 4096), "block"),         # the most tiles a row has at the widest layers, ragged last rows
    ("panel128x128", (129, 272, 4096), "tensor"),
    ("row16x1024", (4099, 400, 1008), "row"),          # 16-row tiles: more tiles than CUs, both halves of the columns ragged
    ("row16x256", (9001, 128, 256), "block_pow2"),
    ("row32x512", (8209, 80, 272), "row"),
    ("panel32_256x256_ragged", (4500, 1200, 1040), "row"),   # ragged in all three, two rounds with a prefetched tile
    ("panel32_256x256_ragged", (66000, 16, 240), "tensor"),  # K shorter than one step
])
@pytest.mark.parametrize("norm", ["layernorm", "none"])
def test_tile_edges_and_rounds(orc, variant, shape, recipe, norm):
    M, K, N = shape
    x, wt = synth.student_t4(M, K, seed=M + N), synth.weight(K, N, seed=K)
    gamma, beta = synth.affine(N, seed=6) if norm == "layernorm" else (None, None)
    _run_case(orc, x, wt, recipe, norm, B.variant_id(variant), gamma, beta, rows=_rows(M), tag=f"{variant} {shape}")


@pytest.mark.parametrize("shape,recipe,ksplit", [((300, 24592, 2320), "row", 12), ((1000, 16384, 1920), "block", 8),
                                                 ((513, 32768, 1024), "block_pow2", 20), ((257, 65552, 272), "tensor", 57)])
def test_split_k_long_ranges(orc, shape, recipe, ksplit):
    # the long-range form of split K, ragged in M, N and K; the first three take 256 x 256 tiles: the workspace holds their
    # number of K ranges (128 x 128 tiles would give 9, 5 and 13)
    M, K, N = shape
    x, wt = synth.student_t4(M, K, seed=M), synth.weight(K, N, seed=N)
    v = B.variant_id("splitk128x128s2")
    desc = B.make_desc(M, N, K, 1, *RECIPES[recipe], B.NORM_RMSNORM, 1e-5, v)
    assert B.lib().loka_fp8_gemm_norm_workspace(ctypes.byref(desc)) == 4 * M * N * ksplit
    _run_case(orc, x, wt, recipe, "rmsnorm", v, rows=_rows(M, 12), tag=f"split-K {shape}")


@pytest.mark.parametrize("shape", [(65536, 8, 16), (66000, 72, 144), (16500, 200, 1008), (65536, 1024, 256), (32768, 4096, 272),
                                   (130, 40, 48), (1000, 4104, 128), (300, 1864, 208), (2048, 4096, 528)])
@pytest.mark.parametrize("batch", [1, 3])
def test_bf16_reference_tiles(shape, batch):
    # 256 x 256 tiles where they fill the chip, 128 x 128 below, K split where those are few; K from one 16-byte chunk up, ragged in M, N and K.
    # fp32 accumulation of exact products against fp64: 2^-24 per addition, K additions at most, relative to sum |x w|
    M, K, N = shape
    if batch > 1 and M * K * N > 1 << 33:
        pytest.skip("the single problem covers the size")
    g = torch.Generator().manual_seed(M + K)
    x = torch.randn(batch, M, K, generator=g).to(torch.bfloat16).to(DEV)
    w = torch.randn(batch, K, N, generator=g).to(torch.bfloat16).to(DEV)
    y = B.loka_bf16_gemm(B.make_desc(M, N, K, batch, norm=B.NORM_NONE), x.view(-1, K), w.view(-1, N)).view(batch, M, N)
    for b in range(batch):
        ref = x[b].double() @ w[b].double()
        bound = x[b].double().abs() @ w[b].double().abs()
        assert bool(((y[b].double() - ref).abs() <= K * 2.0 ** -24 * bound + 1e-30).all())
    # a workspace with room for the transposed weights alone is enough (K is then not split)
    L, d = B.lib(), B.make_desc(M, N, K, batch, norm=B.NORM_NONE)
    small = batch * K * N * 2
    assert small <= L.loka_bf16_gemm_workspace(ctypes.byref(d))
    ws, y2 = torch.empty(small, dtype=torch.uint8, device=DEV), torch.full_like(y, float("nan"))
    args = (ctypes.byref(d), x.data_ptr(), w.data_ptr(), y2.data_ptr(), ws.data_ptr())
    sp = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    assert L.loka_bf16_gemm(*args, small - 1, sp) == B.LOKA_ERR_WORKSPACE
    assert L.loka_bf16_gemm(*args, small, sp) == B.LOKA_OK
    assert bool(((y2[0].double() - y[0].double()).abs() <= K * 2.0 ** -24 * (x[0].double().abs() @ w[0].double().abs()) + 1e-30).all())


@pytest.mark.parametrize("M,K,N,norm,recipe", [(256, 1008, 720, "layernorm", "row"), (2048, 1024, 1024, "rmsnorm", "block"),
                                               (300, 1024, 2320, "none", "row"), (5013, 1008, 1008, "layernorm", "tensor")])
def test_layers_that_need_no_scratch_run_with_any(M, K, N, norm, recipe):
    # N <= 1024 or no row norm: no workspace, a byte less than the query and the query itself are all accepted, and give the
    # same result up to the order of the sums
    L = B.lib()
    x, wt = synth.normal(M, K, seed=3).to(DEV), synth.weight(K, N, seed=4).to(DEV)
    xm, wm = RECIPES[recipe]
    xq, sx = B.loka_quantize(x, xm)
    wq, sw = B.loka_quantize(wt, wm, transpose_out=True)
    desc = B.make_desc(M, N, K, 1, xm, wm, B.NORMS[norm], 1e-5)
    need = L.loka_fp8_gemm_norm_workspace(ctypes.byref(desc))
    sp = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    ws = torch.empty(max(need, 1), dtype=torch.uint8, device=DEV)
    outs = []
    for p, n in ((None, 0), (ws.data_ptr(), max(need - 1, 0)), (ws.data_ptr(), need)):
        out = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device=DEV)
        y = torch.full((M, N), float("nan"), device=DEV)
        assert L.loka_fp8_gemm_norm(ctypes.byref(desc), xq.data_ptr(), sx.data_ptr(), wq.data_ptr(), sw.data_ptr(), None, None,
                                    out.data_ptr(), y.data_ptr(), p, n, sp) == B.LOKA_OK
        if n and n == need:
            assert L.loka_fp8_gemm_norm_check(ctypes.byref(desc), p, 1 << 30, sp) == B.LOKA_OK     # (the header alone is read)
        outs.append((out, y))
    static, _ = B.loka_fp8_gemm_norm_static(desc, xq, sx, wq, sw)
    torch.cuda.synchronize()
    # the variants differ by fp32 summation order (and, blockwise, one rounding per K block): 2^-23 K / 128 of sum |terms|
    ref = outs[-1][1].double()
    for out, y in outs:
        assert float((y.double() - ref).norm() / ref.norm()) <= 2.0 ** -23 * (K / 128 + 8)
        assert float((out.double() - static.double()).norm() / static.double().norm()) <= 1e-3


@pytest.mark.parametrize("shape", [(1, 128, 256), (17, 128, 768), (222, 768, 256), (1000, 1024, 4096), (4100, 256, 512),
                                   (9000, 384, 1024), (20000, 512, 512)])
@pytest.mark.parametrize("recipe", ["tensor", "row", "block"])
def test_blocknorm_on_row_tiles(orc, shape, recipe):
    # BlockNorm by the library's choice: 16-, 32- and 64-row tiles of one group each for few rows, the large kernels above
    M, K, N = shape
    act = B.ACT_HARDSWISH if M % 2 else B.ACT_NONE
    x, wt = synth.student_t4(M, K, seed=M), synth.weight(K, N, seed=N)
    xm, wm = RECIPES[recipe]
    xq, sx = B.loka_quantize(x.to(DEV), xm)
    wq, sw = B.loka_quantize(wt.to(DEV), wm, transpose_out=True)
    desc = B.make_desc(M, N, K, 1, xm, wm, B.NORM_BLOCKNORM, 1e-5, block_n=256, act=act)
    out, y = B.loka_fp8_gemm_norm(desc, xq, sx, wq, sw, want_y=True)
    torch.cuda.synchronize()
    # Y against the exact product of the codes: rounding of the matrix pipe (7 products a group cut at 2^-13 of the largest)
    # and of the fp32 sums, relative to sum |x w|; O against the norm of that Y in fp64: one bf16 rounding and a few fp32 ones
    rows = _rows(M) if M > 4 else np.arange(M)
    idx = torch.from_numpy(rows).to(DEV)
    a = xq[idx].view(torch.float8_e4m3fn).double()
    b = wq.view(torch.float8_e4m3fn).double()
    if recipe == "block":
        a = (a.view(len(rows), K // 128, 128) * sx.view(M, K // 128)[idx].double()[:, :, None]).view(len(rows), K)
        b = (b.view(N // 128, 128, K // 128, 128) * sw.view(K // 128, N // 128).t().double()[:, None, :, None]).view(N, K)
    else:
        a, b = a * (sx if recipe == "tensor" else sx[idx][:, None]).double(), b * (sw if recipe == "tensor" else sw[:, None]).double()
    assert bool(((y[idx].double() - a @ b.T).abs() <= (7 * 2.0 ** -13 + 1e-5) * (a.abs() @ b.abs().T) + 1e-30).all())
    g = y[idx].double().view(len(rows), N // 256, 256)
    o = g / (g.square().mean(-1, keepdim=True) + 1e-5).sqrt()
    if act == B.ACT_HARDSWISH:
        o = o * (o + 3).clamp(0, 6) / 6
    o = o.view(len(rows), N)
    assert bool(((out[idx].double() - o).abs() <= o.abs() * 2.0 ** -8 + 1e-5).all())


@pytest.mark.parametrize("shape", [(222, 768, 256), (300, 1920, 1024)])
@pytest.mark.parametrize("recipe", ["row", "block"])
def test_blocknorm_runs_the_kernel_that_was_profiled(shape, recipe):
    # few rows: without a profile a row tile; after loka_dispatch the kernel that it timed and probed (K is one that the
    # streaming kernel does not take: the large-tile kernel), with that kernel's bits
    M, K, N = shape
    x, w = synth.student_t4(M, K, seed=M).to(DEV), synth.weight(K, N, seed=N).to(DEV)
    xm, wm = RECIPES[recipe]
    xq, sx = B.loka_quantize(x, xm)
    wq, sw = B.loka_quantize(w, wm, transpose_out=True)

    def call(variant):
        desc = B.make_desc(M, N, K, 1, xm, wm, B.NORM_BLOCKNORM, 1e-5, variant, block_n=256)
        return (*B.loka_fp8_gemm_norm(desc, xq, sx, wq, sw, want_y=True), B.loka_default_variant(desc))

    B.loka_dispatch_clear()
    try:
        st, _, table = B.loka_dispatch(B.make_desc(M, N, K, 1, xm, wm, B.NORM_BLOCKNORM, 1e-5, block_n=256), x, w, 0.5)
        assert st == B.LOKA_OK
        out, y, v = call(-1)
        assert v in [r["variant"] for r in table if r["x_mode"] == xm]
        named, named_y, _ = call(v)
        assert torch.equal(out, named) and torch.equal(y, named_y)
    finally:
        B.loka_dispatch_clear()


@pytest.mark.parametrize("variant,shape", [("panel32x256", (1100, 272, 784)), ("panel64x256", (2100, 144, 784)), ("panel128x128", (1300, 256, 640)),
                                           ("panel32_256x256_ragged", (900, 400, 784)), ("splitk128x128s2", (257, 16400, 528))])
def test_new_forms_replay_from_a_graph(variant, shape):
    # the calls of a training step and the split reference, captured once: every replay has new inputs, follows eager work and gives the eager bits
    M, K, N = shape
    desc = B.make_desc(M, N, K, 1, B.SCALE_ROW, B.SCALE_COL, B.NORM_LAYERNORM, 1e-5, B.variant_id(variant))
    x, w = torch.empty(M, K, dtype=torch.bfloat16, device=DEV), torch.empty(K, N, dtype=torch.bfloat16, device=DEV)

    def step():
        wq, sw = B.loka_quantize(w, B.SCALE_COL, transpose_out=True)
        xq, sx = B.loka_quantize(x, B.SCALE_ROW)
        out, _ = B.loka_fp8_gemm_norm(desc, xq, sx, wq, sw)
        return wq, sw, xq, sx, out, B.loka_bf16_gemm(desc, x, w)

    def inputs(seed):
        x.copy_(synth.normal(M, K, seed=seed))
        w.copy_(synth.weight(K, N, seed=seed + 1))

    inputs(1)
    step()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        got = step()
    for seed in range(2, 6):
        inputs(seed)
        want = step()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(got, want))


def test_dispatch_table_lists_every_candidate():
    # one row per recipe and variant that supports the shape, however many variants there are, the chosen one among them
    M, K, N = 256, 128, 128
    x, w = synth.normal(M, K, seed=1).to(DEV), synth.weight(K, N, seed=2).to(DEV)
    B.loka_dispatch_clear()
    st, ch, table = B.loka_dispatch(B.make_desc(M, N, K, norm=B.NORM_LAYERNORM), x, w, 0.1)
    B.loka_dispatch_clear()
    want = set()
    for recipe in ("tensor", "row", "block", "block_pow2"):
        xm, wm = RECIPES[recipe]
        for v in range(B.lib().loka_variant_count()):
            if B.loka_variant_supports(B.make_desc(M, N, K, 1, xm, wm, B.NORM_LAYERNORM, 1e-5), v):
                want.add((xm, wm, v))
    rows = [(r["x_mode"], r["w_mode"], r["variant"]) for r in table]
    assert st == B.LOKA_OK and len(rows) == len(want) and set(rows) == want
    assert (ch["x_mode"], ch["w_mode"], ch["variant"]) in want


@pytest.mark.parametrize("shape", [(300, 1920, 1024), (130, 384, 4096), (8200, 256, 512)])
def test_dispatch_of_wide_blocknorm_layers(shape):
    # groups of 256 in rows of several tiles: bf16 output has no wait to report (FP8 output has), every recipe is a candidate
    M, K, N = shape
    x, w = synth.student_t4(M, K, seed=M).to(DEV), synth.weight(K, N, seed=N).to(DEV)
    B.loka_dispatch_clear()
    try:
        desc = B.make_desc(M, N, K, 1, B.SCALE_ROW, B.SCALE_COL, B.NORM_BLOCKNORM, 1e-5, block_n=256, act=B.ACT_HARDSWISH)
        st, ch, table = B.loka_dispatch(desc, x, w, 0.5)
        assert st == B.LOKA_OK and {r["x_mode"] for r in table} == {RECIPES[r][0] for r in ("tensor", "row", "block", "block_pow2")}
        assert ch["variant"] in [r["variant"] for r in table if r["x_mode"] == ch["x_mode"]]
    finally:
        B.loka_dispatch_clear()


@pytest.mark.parametrize("variant", ["twopass128x128", "splitk128x128", "panel128x128", "panel64x256", "panel32_256x256"])
@pytest.mark.parametrize("norm", ["layernorm", "none"])
def test_strided_outputs_stay_inside_the_workspace(variant, norm):
    # problems further apart than M * N in O: the bits of the contiguous call, nothing written between the problems, and
    # nothing behind the workspace (the guard is long enough for an fp32 staging area with the outputs' stride)
    M, K, N, batch = 130, 1024, 384, 3
    stride = 2 * M * N + 128
    L, v = B.lib(), B.variant_id(variant)
    x, w = synth.normal(batch * M, K, seed=1).to(DEV), synth.weight(K, N, seed=2).to(DEV)
    xq, sx = B.loka_quantize(x, B.SCALE_ROW)
    wq, sw = B.loka_quantize(w, B.SCALE_COL, transpose_out=True)
    desc = B.make_desc(M, N, K, batch, B.SCALE_ROW, B.SCALE_COL, B.NORMS[norm], 1e-5, v)
    desc.strideW = 0
    want, _ = B.loka_fp8_gemm_norm(desc, xq, sx, wq, sw)
    desc.strideO = stride
    need = int(L.loka_fp8_gemm_norm_workspace(ctypes.byref(desc)))
    guard = batch * stride * 4
    ws = torch.full((need + guard,), 0xA5, dtype=torch.uint8, device=DEV)
    out = torch.full((batch * stride,), 7.0, dtype=torch.bfloat16, device=DEV)
    sp = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    assert L.loka_fp8_gemm_norm(ctypes.byref(desc), xq.data_ptr(), sx.data_ptr(), wq.data_ptr(), sw.data_ptr(), None, None,
                                out.data_ptr(), None, ws.data_ptr(), need, sp) == B.LOKA_OK
    torch.cuda.synchronize()
    got = out.view(batch, stride)
    assert torch.equal(got[:, :M * N].reshape(batch * M, N), want)
    assert bool((got[:, M * N:] == 7.0).all()) and bool((ws[need:] == 0xA5).all())
