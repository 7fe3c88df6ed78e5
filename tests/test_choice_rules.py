"""Host rules of the library: which kernel a call takes, and how much scratch it accepts (no GPU needed)."""
import csv
import ctypes
import math
import os
import random
import re
import subprocess

import pytest
import torch

from paper_2605_10886_amd import binding as B
from paper_2605_10886_amd import build


def _check(desc, nbytes):
    """loka_fp8_gemm_norm_check on a clear workspace of `nbytes`: on the device where there is one; without one the size is
    still judged, and an accepted workspace then ends in LOKA_ERR_HIP at the copy of its header."""
    dev = "cuda:0" if torch.cuda.is_available() else "cpu"
    ws = torch.zeros(max(nbytes, 16) + 256, dtype=torch.uint8, device=dev)
    p = (ws.data_ptr() + 255) // 256 * 256
    return B.lib().loka_fp8_gemm_norm_check(ctypes.byref(desc), p, nbytes, None)


# (the FP8-output form needs less than the bf16 call, more, the same, or is the only one of the two that waits)
@pytest.mark.parametrize("M,N,K", [(1024, 2560, 4096), (1000, 1536, 4096), (512, 1024, 2048), (300, 4096, 4096), (2048, 4096, 4096),
                                   (5013, 720, 1024), (65536, 1024, 1024)])
def test_wait_check_takes_the_workspace_of_either_call(M, N, K):
    L, d = B.lib(), B.make_desc(M, N, K, norm=B.NORM_LAYERNORM)
    sizes = [int(L.loka_fp8_gemm_norm_workspace(ctypes.byref(d))), int(L.loka_fp8_gemm_norm_fp8out_workspace(ctypes.byref(d)))]
    for n in sizes:
        assert _check(d, n) != B.LOKA_ERR_WORKSPACE, (sizes, n)


@pytest.fixture(scope="module")
def numbering(tmp_path_factory):
    """(form, G, tiles_n) -> the order in which a panel launch takes its workgroups: logical id of every block, from the header
    that the kernels compile.  None: launch order.  Form 0: 256 x 256 tiles; form 1: smaller ones, up to two workgroups per CU."""
    d = tmp_path_factory.mktemp("numbering")
    src = d / "numbering.hip"
    src.write_text("""#include "gemm_common.h"
#include <cstdio>
int main() {
    for (int tn = 1; tn <= 256; ++tn)
        for (int G = tn; G <= 256; G += tn) {
            std::printf("0 %d %d", G, tn);
            if (loka::panels_may_spread(G, tn)) for (int b = 0; b < G; ++b) std::printf(" %d", loka::xcd_contiguous(b, G));
            std::printf("\\n");
        }
    for (int tn = 1; tn <= 8; ++tn)
        for (int G = tn; G <= 512; G += tn) {
            std::printf("1 %d %d", G, tn);
            for (int b = 0; b < G; ++b) std::printf(" %d", loka::panel_per_xcd(b, G, tn));
            std::printf("\\n");
        }
}
""")
    exe = str(d / "numbering")
    subprocess.run([build._hipcc(), "--cuda-host-only", "-O1", "-std=c++17", "-I", os.path.join(build.HERE, "csrc"), str(src), "-o", exe],
                   check=True, capture_output=True)
    rows = [[int(v) for v in line.split()] for line in subprocess.run([exe], check=True, capture_output=True, text=True).stdout.splitlines()]
    return {tuple(r[:3]): r[3:] or None for r in rows}


def test_panels_are_spread_only_where_their_waits_cannot_fill_an_xcd(numbering):
    large = {k[1:]: v for k, v in numbering.items() if k[0] == 0}
    assert len(large) == sum(256 // tn for tn in range(1, 257))
    for (G, tn), ids in large.items():
        if ids is None:
            assert tn > 8
            continue
        assert sorted(ids) == list(range(G))
        assert 2 * (tn - 1) < 32 and (tn > 8 or 4 * (tn - 1) < 32)
        if tn > 8:                                                # no panel on two XCDs
            homes = [{b % 8 for b in range(G) if ids[b] // tn == panel} for panel in range(G // tn)]
            assert all(len(h) == 1 for h in homes), (G, tn)
    assert large[256, 16] and large[255, 5]
    assert not any(large[g] for g in ((240, 20), (240, 24), (240, 40), (256, 64), (256, 32), (64, 16)))


def test_small_tiles_keep_a_panel_on_one_xcd(numbering):
    # every id once; all panels but the last few (less than one per XCD) on one XCD, their workgroups one behind the other;
    # of the rest an XCD has 7 at most, as many as it can have begun of a panel of 8
    for (form, G, tn), ids in numbering.items():
        if form == 0:
            continue
        assert sorted(ids) == list(range(G))
        whole = G // (8 * tn) * 8
        for x in range(8):
            mine = [ids[b] for b in range(x, G, 8)]
            panels = [i // tn for i in mine]
            assert mine[:whole // 8 * tn] == [p * tn + t for p in range(x, whole, 8) for t in range(tn)], (G, tn, x)
            assert all(p >= whole for p in panels[whole // 8 * tn:]) and len(mine) - whole // 8 * tn <= 7, (G, tn, x)


@pytest.mark.parametrize("form,G,tn,launches,slots", [
    (0, 255, 5, 4, 32), (0, 256, 8, 4, 32), (0, 248, 8, 4, 32), (0, 256, 16, 2, 32), (0, 128, 16, 2, 32), (0, 252, 7, 4, 32),
    (1, 512, 4, 4, 64), (1, 510, 3, 4, 64), (1, 512, 8, 4, 64), (1, 511, 7, 4, 64), (1, 256, 8, 4, 32), (1, 252, 6, 4, 32)])
def test_launches_side_by_side_finish(numbering, form, G, tn, launches, slots):
    # 8 XCDs of 32 CUs; each starts its share of every launch in order, the launches interleaved at random; a panel's
    # workgroups leave once all of them are there.  Nobody may be left waiting.
    ids = numbering[form, G, tn]
    for seed in range(20):
        rng = random.Random(seed)
        todo = [[[ids[b] // tn for b in range(x, G, 8)] for x in range(8)] for _ in range(launches)]
        held, arrived = [[] for _ in range(8)], {}
        left = launches * G
        while left:
            moves = [(n, x) for x in range(8) if len(held[x]) < slots for n in range(launches) if todo[n][x]]
            assert moves, (G, tn, seed, "no slot is free and nobody can finish")
            n, x = rng.choice(moves)
            for _ in range(rng.randrange(1, slots + 1)):          # a run of one launch's workgroups on one XCD
                if not todo[n][x] or len(held[x]) >= slots:
                    break
                key = (n, todo[n][x].pop(0))
                held[x].append(key)
                arrived[key] = arrived.get(key, 0) + 1
                if arrived[key] == tn:
                    for h in held:
                        h[:] = [k for k in h if k != key]
                    left -= tn


def test_block_scales_leave_no_operand_in_flight(tmp_path):
    # The block-scaled main loop, one wave's loads in the order they are requested (they return in it): X(0) W(0) X(1) W(1)
    # X(2), then per step k the scales of block k + 1, X(k + 2) and, behind the wait, W(k + 2).  At the wait X(k + 1) and
    # W(k + 1) have to be there, and no more than that is waited for.
    src = tmp_path / "loads.hip"
    src.write_text("""#include "gemm_common.h"
#include <cstdio>
int main() {
    for (int quad = 0; quad < 2; ++quad)
        for (int k = 0; k < 64; ++k) std::printf("%d ", loka::panel32_scale_loads(quad, k));
}
""")
    exe = str(tmp_path / "loads")
    subprocess.run([build._hipcc(), "--cuda-host-only", "-O1", "-std=c++17", "-I", os.path.join(build.HERE, "csrc"), str(src), "-o", exe],
                   check=True, capture_output=True)
    n = [int(v) for v in subprocess.run([exe], check=True, capture_output=True, text=True).stdout.split()]
    for quad, scales in ((False, n[:64]), (True, n[64:])):
        for ksteps in (4, 5, 8, 16, 64) if not quad else (4, 8, 16, 64):
            sent = [f"{m}{k}" for k in (0, 1) for m in "XW" for _ in range(4)] + ["X2"] * 4
            for k in range(ksteps - 2):
                fetch = 5 if not quad or (k + 1) % 4 == 0 else 1
                sent += [f"s{k + 1}"] * fetch + ([f"X{k + 2}"] * 4 if k else [])
                flying = sent[len(sent) - (4 + scales[k]):]
                assert not {f"X{k + 1}", f"W{k + 1}"} & set(flying), (quad, ksteps, k)
                assert sent[len(sent) - (4 + scales[k]) - 1] == f"W{k + 1}"
                sent += [f"W{k + 2}"] * 4


def test_every_word_of_a_diagonal_tracker_tile_has_one_writer(tmp_path):
    # A diagonal pair's tile on its way out, half by half: every LDS word is written once, by the lane that holds its element or
    # the mirror image of it; two lanes' writes to one word have no order that the kernel may rely on.
    src = tmp_path / "stage.hip"
    src.write_text("""#include "tracker_stage.h"
#include <cstdio>
#include <vector>
using namespace loka;
int main() {
    int bad = 0;
    for (int ps = 0; ps < 2; ++ps) {
        std::vector<int> writers(128 * 256), held(128 * 256, -1);               // held: 256 * tile row + tile column
        auto put = [&](int word, int row, int col) { ++writers.at(word); held[word] = 256 * row + col; };
        for (int wave = 0; wave < 8; ++wave)
            for (int lane = 0; lane < 64; ++lane)
                for (int t = 0; t < 4; ++t)
                    for (int e = 0; e < 2; ++e) {
                        const bool self = trk_self(wave);
                        const int h = lane >> 5, c = lane & 31, ga = trk_group(wave, t < 2 ? 0 : 1), gb = self ? ga : trk_group(wave, 1);
                        const int a = 2 * ga + (t & 1), b = 2 * gb;
                        const bool stores = self ? trk_self_stores(t, e) : trk_pair_holds(t), mirrors = self ? trk_self_mirrors(t, e) : trk_pair_holds(t);
                        for (int r = 0; r < 16; ++r) {
                            const int R = 8 * (r >> 2) + 4 * h + (r & 3), row = 8 * R + a, col = 8 * c + b + e;
                            const TrkAddr d = trk_direct(true, a, b, h, c), m = trk_mirror(a, b + e, h, c);
                            if (stores && r / 8 == ps) put(d.row + trk_direct_step(r & 7) + (d.pos ^ trk_direct_key(true, r & 7)) + e, row, col);
                            if (mirrors && c / 16 == ps) put(m.row + (m.pos ^ trk_mirror_key(r)), col, row);
                        }
                    }
        for (int row = 0; row < 128; ++row)
            for (int col = 0; col < 256; ++col) {
                const int R = row / 8, w = row * 256 + ((col & 7) >> 1) * 64 + ((2 * (col / 8)) ^ (((col & 7) >> 2) * 32) ^ (2 * R)) + (col & 1);
                if (writers[w] != 1 || held[w] != 256 * (128 * ps + row) + col)
                    if (++bad < 20) std::printf("half %d row %d column %d: %d writers, element %d\\n", ps, row, col, writers[w], held[w]);
            }
    }
    return bad ? 1 : 0;
}
""")
    exe = str(tmp_path / "stage")
    subprocess.run([build._hipcc(), "--cuda-host-only", "-O1", "-std=c++17", "-I", os.path.join(build.HERE, "csrc"), str(src), "-o", exe],
                   check=True, capture_output=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


def _device_assembly(src, out):
    """gfx950 assembly of one of the library's sources, by the flags that the library is built with: {kernel: its lines}."""
    subprocess.run([build._hipcc(), *build.HIPCC_FLAGS, *build.EXTRA_FLAGS.get(src, []), "-S", "--cuda-device-only",
                    os.path.join(build.CSRC, src), "-o", str(out)], check=True, capture_output=True)
    kernels, name = {}, None
    for line in out.read_text().splitlines():
        m = re.match(r"(_Z\w+):", line)
        if m:
            name = m.group(1)
            kernels[name] = []
        elif name:
            kernels[name].append(line)
            if "s_endpgm" in line:
                name = None
    return kernels


def test_strips_are_awaited_without_the_stores_behind_them(tmp_path):
    # The strip kernel's loop, rows of up to 256, bf16 output: the operands of the next strip are older than the epilogue's 2 NB
    # stores, which the wait for them leaves in flight; nothing in the loop waits for more than that.
    kernels = _device_assembly("gemm_strip.hip", tmp_path / "strip.s")
    def strip_loop(nb, ks, fused):
        lines = next(v for k, v in kernels.items() if f"gemm_strip_kernelILi{nb}ELi{ks}ELi1ELi8ELb{fused}ELb0E" in k)
        # (the listing names the header of the innermost loop of every block)
        loops, header = {}, None
        for l in lines:
            if re.match(r"\.LBB\w+:|; %bb", l):
                m = re.search(r"Header=(BB\w+)", l)
                header = l[2:l.index(":")] if l.startswith(".LBB") and "Parent Loop" in l else m.group(1) if m else header if l.startswith("; %bb") else None
            loops.setdefault(header, []).append(l)
        loop = next(b for h, b in loops.items() if h and any(f"vmcnt({2 * nb})" in l for l in b))
        assert any("v_mfma" in l for l in loop)
        return loop

    def wait(line):
        m = re.search(r"s_waitcnt.*vmcnt\((\d+)\)", line)
        return int(m.group(1)) if m else None

    for nb, ks in ((4, 2), (4, 4), (8, 2), (8, 4)):
        waits = [wait(l) for l in strip_loop(nb, ks, 0) if wait(l) is not None]
        assert waits and min(waits) == 2 * nb, (nb, ks, waits)


def test_tracker_contraction_keeps_its_values_in_registers(tmp_path):
    # 128 accumulators, a stage in flight and two sets of fragments fill a wave's 256 registers: nothing of it goes to scratch
    _device_assembly("tracker.hip", tmp_path / "tracker.s")
    m = re.search(r"\.amdhsa_kernel \w*tracker_scatter_kernel\w*\n(.*?)\.end_amdhsa_kernel", (tmp_path / "tracker.s").read_text(), re.S)
    assert re.search(r"\.amdhsa_private_segment_fixed_size (\d+)", m.group(1)).group(1) == "0"


@pytest.mark.parametrize("batch,features,ranges", [(65536, 4096, 5), (65536, 2560, 4), (8000, 2048, 6), (32768, 1024, 25), (65536, 256, 128)])
def test_tracker_ranges(batch, features, ranges):
    # scratch: a 256 KB partial tile and its column sums per pair of column tiles and range, and the mean
    tiles = (features + 255) // 256
    want = ranges * tiles * (tiles + 1) // 2 * 256 * (256 * 4 + 8) + tiles * 256 * 4
    assert B.lib().loka_tracker_update_workspace(batch, features) == want


def _chosen(form, M, N, K, norm=B.NORM_LAYERNORM, batch=1):
    """Name of the kernel behind variant = -1 for a call of that form (the library's own rule, a C++ function of the descriptor)."""
    fn = B.lib().loka_default_variant if form == "bf16" else getattr(B.lib(), {"fp8out": "_ZN4loka22variant_fp8out_defaultEPK14loka_gemm_desc",
                           "xq": "_ZN4loka18variant_xq_defaultEPK14loka_gemm_desc"}[form])
    kw = dict(block_n=256) if norm == B.NORM_BLOCKNORM else {}
    v = fn(ctypes.byref(B.make_desc(M, N, K, batch, norm=norm, **kw)))
    return B.loka_variant_name(v) if v >= 0 else None


# the kernel that was measured at least 10 % faster than the other two that have the form
@pytest.mark.parametrize("form,M,N,K,want", [
    ("fp8out", 2048, 64, 128, "strip32"), ("fp8out", 32768, 128, 128, "strip32"), ("fp8out", 65536, 112, 512, "strip32"),
    ("fp8out", 131072, 128, 512, "strip32"), ("fp8out", 16384, 256, 1024, "wreg32"), ("fp8out", 8192, 256, 512, "wreg32"),
    ("fp8out", 65536, 256, 1024, "panel32_256x256"), ("fp8out", 65536, 256, 512, "panel32_256x256"),
    ("fp8out", 2048, 512, 512, "wreg32"), ("fp8out", 65536, 1024, 256, "wreg32"), ("fp8out", 2048, 2048, 512, "panel32_256x256"),
    ("xq", 60000, 256, 512, "panel32_256x256"), ("xq", 60000, 64, 1024, "panel32_256x256"), ("xq", 70000, 256, 1024, "wreg32"),
    ("xq", 80000, 64, 512, "wreg32"), ("xq", 32768, 128, 1024, "wreg32"), ("xq", 131072, 128, 256, "wreg32"),
    ("xq", 4096, 128, 2048, "panel32_256x256")])
def test_forms_choose_by_their_own_times(form, M, N, K, want):
    assert _chosen(form, M, N, K) == want


def test_fp8_output_without_a_row_norm_takes_a_kernel_that_has_it():
    # the large-tile kernel needs a row norm; where it would be the fastest, the call still runs
    for M, N, K in ((65536, 256, 512), (65536, 256, 1024), (131072, 256, 256)):
        assert _chosen("fp8out", M, N, K, B.NORM_NONE) in ("wreg32", "strip32")
        assert _chosen("fp8out", M, N, K, B.NORM_BLOCKNORM) in ("wreg32", "panel32_256x256")
    assert _chosen("fp8out", 512, 4096, 4096, B.NORM_NONE) is None


# bf16 output: the kernel that was measured at least 10 % faster than all others, at shapes where a choice that knows
# neither the norm's share nor the alignment of the rows took one that was 1.2 to 2.9 times slower
@pytest.mark.parametrize("M,N,K,batch,norm,want", [
    (65536, 128, 512, 1, "layernorm", "strip32"), (101163, 240, 512, 1, "layernorm", "strip32"), (13495, 240, 512, 8, "layernorm", "strip32"),
    (4685, 256, 128, 4, "layernorm", "strip32"), (112816, 208, 512, 1, "none", "wreg32"), (31318, 256, 512, 8, "none", "wreg32"),
    (4402, 128, 6272, 1, "rmsnorm", "splitk128x128"), (199, 256, 4352, 16, "rmsnorm", "splitk128x128"),
    (148, 1184, 7856, 16, "none", "splitk128x128s2"), (20937, 128, 4336, 1, "none", "panel128x128"),
    (122, 1184, 2144, 16, "rmsnorm", "panel128x128"), (310, 3072, 3072, 1, "rmsnorm", "panel32x256"),
    (152, 2560, 2816, 16, "layernorm", "panel32_256x256"), (57449, 576, 64, 4, "layernorm", "panel32_256x256_ragged"),
    (31021, 688, 384, 1, "rmsnorm", "row64x1024"), (8616, 64, 2048, 8, "none", "row64x128"), (9214, 128, 128, 1, "none", "row32x128")])
def test_bf16_output_chooses_by_measured_times(M, N, K, batch, norm, want):
    assert _chosen("bf16", M, N, K, B.NORMS[norm], batch) == want


def test_static_choice_over_measured_times():
    # Every variant's time at 1997 shapes: what the choice loses to the fastest variant, in the mean and at its worst shapes, and
    # against what two former sets of figures chose there (the mean alone hides layers that a new set sends to a slower kernel).
    with open(os.path.join(build.ROOT, "profiles", "variant_times.csv")) as f:
        rows = list(csv.DictReader(line for line in f if not line.startswith("#")))
    over, against = [], []
    for r in rows:
        modes = (B.SCALE_BLOCK_1x128, B.SCALE_BLOCK_128x128) if r["scales"] == "block" else (B.SCALE_ROW, B.SCALE_COL)
        d = B.make_desc(int(r["M"]), int(r["N"]), int(r["K"]), int(r["batch"]), *modes, B.NORMS[r["norm"]], 1e-5)
        name = B.loka_variant_name(B.lib().loka_default_variant(ctypes.byref(d)))
        times = {k: float(v) for k, v in r.items() if k not in ("M", "N", "K", "batch", "scales", "norm", "former") and v}
        over.append(math.log(times[name] / min(times.values())))
        against.append(times[name] / times[r["former"].split("/")[0]])
    assert len(rows) == 1997
    assert math.exp(sum(over) / len(over)) < 1.006
    assert math.exp(sorted(over)[int(0.99 * len(over))]) < 1.12
    assert sum(x > 1.05 for x in against) < 0.013 * len(against) and sum(x > 1.2 for x in against) < 0.002 * len(against)
