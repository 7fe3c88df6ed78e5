// Small-layer FP8 GEMM with the row norm fused, one row strip per WAVE: W in LDS, X straight into registers.
//
// For the many small GEMMs of a recommendation model (Section 2.1; K * N <= 128 KB, N <= 256: 256 x 256, 512 x 256,
// 1024 x 128, ...)
// a whole output row fits the accumulators of ONE wave: a wave takes 32 rows of X, multiplies them with all of
// W (resident in LDS for the whole problem, read fragment by fragment), and scales, normalizes and stores its
// 32 x N outputs from registers.  The row statistics need two lanes (l, l ^ 32) and no other wave, so after the
// weights are in place the 8 waves of a workgroup never synchronize: each runs load -> MFMA -> normalize -> store
// at its own pace, and the phases of different waves overlap on the CU.  (The streaming kernel for skinny
// layers splits the row over its 8 waves and runs those phases one after the other behind workgroup barriers;
// measured at 64 x (4096 x 256 x 256) it needs 7.4 us per 128 rows against 3.1 us of HBM time.)
//
// X does not pass through LDS: the MFMA operand of a lane is 32 consecutive K bytes of one row, which two
// 16-byte loads fetch directly (two lanes cover a 64-byte run of the row); the next strip's operands are
// requested before the current strip is multiplied.  Roles and the W row permutation are those of the other
// streaming kernel: W rows -> MFMA rows, X rows -> MFMA columns, so a lane ends with 16 consecutive output
// columns per column block of one output row (= lane % 32).
#include "gemm_common.h"

#include <type_traits>

namespace loka {

typedef float v16f __attribute__((ext_vector_type(16)));


template <int NB, int KS, int NPH>
struct StripCfg {
    static constexpr int NT = NB * 32;                    // columns the accumulators cover
    static constexpr int KB = KS * 64;                    // K bytes per phase = bytes per row of the W slab in LDS
    static constexpr int KBT = NPH * KB;                  // bytes per row of X / W in memory
    static constexpr int SWIN = KB / 16 < 16 ? KB / 16 : 16;
    static constexpr int OFF_W = 0;                       // [NT][KB], 16-byte chunk c of row r at c ^ (r % SWIN)
    static constexpr int OFF_SW = NT * KB;                // [NT] fp32 column scales (0 beyond N)
    static constexpr int OFF_GM = OFF_SW + NT * 4;        // [NT] fp32 gamma (1 when absent)
    static constexpr int OFF_BT = OFF_GM + NT * 4;        // [NT] fp32 beta (0 when absent)
    static constexpr int OFF_T = OFF_BT + NT * 4;         // [8 waves][2 KB] output staging (see the epilogue)
    static constexpr int LDS = OFF_T + 8 * 2048;
    static_assert(LDS <= 160 * 1024, "W, the tables and the staging buffers must fit the LDS");
    // fused quantization with nwv waves, more than 128 columns: K steps of a wave's bf16 strip that wait in LDS, behind the
    // staging buffers: all of them, half, or none (up to 128 columns registers and caches do: 64 x (4096 x 128 x 128),
    // M x N x K, 26.0 us, 27.0 through LDS)
    static constexpr int off_raw(int nwv) { return OFF_T + nwv * 2048; }
    static constexpr int raw_steps(int nwv) {
        return NPH != 1 || NB != 8 ? 0 : off_raw(nwv) + nwv * KS * 4096 <= 160 * 1024 ? KS : off_raw(nwv) + nwv * KS * 2048 <= 160 * 1024 ? KS / 2 : 0;
    }
    static constexpr int lds_fused(int nwv) { return raw_steps(nwv) ? off_raw(nwv) + nwv * raw_steps(nwv) * 4096 : LDS; }
};

// NWV waves per workgroup; BF16IN: X arrives as bf16 and is quantized per row (amax, scale, e4m3 cast: the
// arithmetic of the quantize kernel, bit for bit) on its way into the MFMA operand registers, so the FP8 copy of X
// never exists in memory (Section 3.2: quantization fused with the layer).  A strip's 32 x K bf16 values are a
// second set of 16 KS registers per lane that must stay live through the previous strip's epilogue: with more than 128
// columns it waits in LDS, all or half of it (raw_steps), with K = 512 four waves of up to 512 registers run instead of
// eight of 256.
template <int NB, int KS, int NPH, int NWV, bool BF16IN, bool FP8OUT>
__global__ __launch_bounds__(NWV * 64) void gemm_strip_kernel(const GemmParams p, const int strips_per_problem) {
    using C = StripCfg<NB, KS, NPH>;
    static_assert(!BF16IN || NPH == 1, "fused quantization needs the whole row of X in one pass");
    constexpr int NT = C::NT, KB = C::KB, KBT = C::KBT, KEYMASK = C::SWIN - 1;
    // Up to rows of 256: statistics and stores without branches; with fused quantization the stores everywhere.  Longer rows'
    // operands leave no registers for it: the kernel spills more (M x N x K: 65536 x 128 x 1024 21.5 -> 23.2 us, with FP8
    // output 23.9 -> 25.3 and 64 x (4096 x 256 x 512) 62.6 -> 64.8; but 64 x (4096 x 256 x 256) with FP8 output 48.6 -> 45.6).
    constexpr bool SHORT_ROWS = KS < 8 && NPH == 1, LEAN = SHORT_ROWS || BF16IN;
    // One sequence of stores for layers with and without gamma and beta, so that the next strip's operands, requested before
    // it, can be awaited by count and the stores stay in flight.  With a sequence on each side of a branch the compiler
    // sees a path without any, on which the count does not cover the operands, and drains every store at the next use.
    // (Geometric mean over 160 layers, two sequences -> one: 1.4 % faster; 66481 x 240 x 256, M x N x K, 16.4 -> 15.6 us.)  Not
    // where the branches and registers cost more than that: FP8 output 1.4 to 14 % slower, fused with N <= 128 2.5 to 4 %.
    constexpr bool ONE_PATH = SHORT_ROWS && !FP8OUT && !BF16IN;
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l32 = lane & 31, hk = lane >> 5;
    const bool ln = p.norm == LOKA_NORM_LAYERNORM;
    const bool tensor_x = p.x_mode == LOKA_SCALE_TENSOR, tensor_w = p.w_mode == LOKA_SCALE_TENSOR;
    const float inv_n = 1.0f / static_cast<float>(p.N);
    const bool affine = p.norm != LOKA_NORM_NONE && (p.gamma != nullptr || (p.beta != nullptr && ln));

    float cnt_lane = 0.f;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
        if (nb * 32 + hk * 16 < p.N) cnt_lane += 16.f;     // N % 16 == 0: a run of 16 columns is all in or all out
    const float rc_lane = cnt_lane > 0.f ? __builtin_amdgcn_rcpf(cnt_lane) : 0.f;

    // contiguous range of strips of this workgroup (strip = 32 rows of one problem)
    const int64_t total = static_cast<int64_t>(p.batch) * strips_per_problem;
    int t = static_cast<int>(total * blockIdx.x / gridDim.x);
    const int t1 = static_cast<int>(total * (blockIdx.x + 1) / gridDim.x);

    while (t < t1) {
        const int g = t / strips_per_problem;
        const int seg_end = (g + 1) * strips_per_problem < t1 ? (g + 1) * strips_per_problem : t1;

        // ---- tables of problem g; its weights (the K slab of phase ph) on request
        __syncthreads();                                    // every wave has finished with the previous problem
        const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<uint8_t*>(p.W + static_cast<int64_t>(g) * p.strideW), 0, static_cast<unsigned>(p.N) * KBT, 0x00020000);
        auto load_w = [&](int ph) __attribute__((always_inline)) {
            for (int ld = wave; ld < NT * KB / 1024; ld += NWV) {
                const int byte = ld * 1024 + lane * 16;
                const int row = byte / KB, pos = (byte % KB) >> 4;
                // rows past N lie behind the descriptor's bound (the offset is the per-lane one) and read as zeros
                __builtin_amdgcn_raw_ptr_buffer_load_lds(wr, (__attribute__((address_space(3))) void*)(smem + C::OFF_W + ld * 1024),
                                                         16, row * KBT + ph * KB + ((pos ^ (row & KEYMASK)) << 4), 0, 0, 0);
            }
        };
        {
            const float* swg = p.sw + static_cast<int64_t>(g) * p.strideSw;
            float* swl = reinterpret_cast<float*>(smem + C::OFF_SW);
            float* gml = reinterpret_cast<float*>(smem + C::OFF_GM);
            float* btl = reinterpret_cast<float*>(smem + C::OFF_BT);
            for (int n = threadIdx.x; n < NT; n += NWV * 64) {
                const bool in = n < p.N;
                swl[n] = in ? (tensor_w ? swg[0] : swg[n]) : 0.f;
                gml[n] = (in && p.gamma && p.norm != LOKA_NORM_NONE) ? bf16_bits_to_f32(p.gamma[n]) : 1.f;
                btl[n] = (in && p.beta && ln) ? bf16_bits_to_f32(p.beta[n]) : 0.f;
            }
        }
        if (NPH == 1) {
            load_w(0);
            wait_vmcnt<0>();
            __syncthreads();
        }

        const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<uint8_t*>(p.X + static_cast<int64_t>(g) * p.strideX), 0, static_cast<unsigned>(p.M) * KBT, 0x00020000);
        const float* sxg = p.sx + static_cast<int64_t>(g) * p.strideSx;
        const int s_base = g * strips_per_problem;

        const __amdgpu_buffer_rsrc_t sxr = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(sxg), 0, tensor_x ? 4 : p.M * 4, 0x00020000);
        // operands of strip s, phase ph: row m0 + l32, K bytes [KB ph + 64 j + 32 hk, +32) per K step (rows past M
        // read as zeros)
        auto load_x = [&](int s, int ph, v8i (&x)[KS], float& sxm, bool live) __attribute__((always_inline)) {
            const int m = (s - s_base) * 32 + l32;
            // (short rows: the first row's offset from a scalar register, beyond the descriptor's bound where there is no strip,
            // so that the loads are the same on every path)
            unsigned base = SHORT_ROWS ? (live ? static_cast<unsigned>((s - s_base) * 32) * KBT : 0x80000000u) : 0u;
            if (SHORT_ROWS) asm volatile("; first row" : "+s"(base));
#pragma unroll
            for (int j = 0; j < KS; ++j) {
                const unsigned off = SHORT_ROWS ? base + static_cast<unsigned>(l32 * KBT + (4 * j + 2 * hk) * 16)
                                                : static_cast<unsigned>(m) * KBT + static_cast<unsigned>(ph * KB + (4 * j + 2 * hk) * 16);
                const v4i lo = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(xr, off, 0, 0));
                const v4i hi = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(xr, off + 16u, 0, 0));
                x[j] = v8i{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
            }
            if (SHORT_ROWS) sxm = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(sxr, tensor_x ? 0 : m * 4, 0, 0));
            else sxm = tensor_x ? sxg[0] : (m < p.M ? sxg[m] : 0.f);
        };

        // Fused quantization: the lane's 32 bf16 values per K step (row m0 + l32, K elements [64 j + 32 hk, +32): 64
        // bytes, four loads), then row amax (integer max of the magnitudes, this lane and lane ^ 32 hold the row),
        // scale pair, cast.  Rows past M read as zeros.
        const __amdgpu_buffer_rsrc_t xbr = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<uint16_t*>(BF16IN ? p.xb + static_cast<int64_t>(g) * p.strideX : nullptr), 0,
            static_cast<unsigned>(p.M) * KBT * 2u, 0x00020000);
        auto load_raw = [&](int s, u32x4 (&raw)[KS][4], int j0) __attribute__((always_inline)) {
            int lane_o = lane;
            if (BF16IN && C::raw_steps(NWV) > 0) asm volatile("; per-strip lane id" : "+v"(lane_o));
            const int m = (s - s_base) * 32 + (lane_o & 31);
#pragma unroll
            for (int j = j0; j < KS; ++j) {
                const unsigned off = static_cast<unsigned>(m) * (KBT * 2u) + static_cast<unsigned>((64 * j + 32 * (lane_o >> 5)) * 2);
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    raw[j][q] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(xbr, off + 16u * q, 0, 0));
            }
        };
        // Where LDS has room the raw strip comes through it: loads straight into LDS move whole rows (1 KB runs; 16-byte chunk c
        // of row r at c ^ (r % 16)), each lane then takes its pieces from there.  Requested straight into the lanes that
        // need them a load instruction touches 64 lines for 16 bytes each, and four waves' strips do not stay in the CU's
        // cache until the other pieces are asked for.  With half a strip there (and the other half in 32 registers instead of 64) eight
        // waves fit a CU where four did (M x N x K: 100000 x 240 x 256 32.1 -> 25.2 us, 16 x (4096 x 256 x 256) 21.2 -> 18.0).
        constexpr int KL = BF16IN ? C::raw_steps(NWV) : 0;                // K steps of 64 that come through LDS (the first ones)
        constexpr bool RAWLDS = KL > 0;
        constexpr int ROWB = KBT * 2, ROWL = RAWLDS ? KL * 128 : 128, RLD = KL * 4;
        uint8_t* const rbuf = smem + C::off_raw(NWV) + wave * (KL * 4096);
        auto request_raw = [&](int s) __attribute__((always_inline)) {
            int lane_o = lane;
            asm volatile("; per-strip lane id" : "+v"(lane_o));
            // (load i covers rows i RPL .. + RPL - 1, a power of two, so that the swizzle key of a lane's row is (i RPL) ^ r)
            constexpr int LPR = ROWL / 16, RPL = 64 / LPR;
            const int r = lane_o / LPR, pos = (lane_o % LPR) ^ r;
            const unsigned base = static_cast<unsigned>((s - s_base) * 32 + r) * ROWB;
#pragma unroll
            for (int i = 0; i < RLD; ++i)
                // (rows past M lie behind the descriptor's bound and read as zeros)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(xbr, (__attribute__((address_space(3))) void*)(rbuf + i * 1024), 16,
                                                         base + i * RPL * ROWB + static_cast<unsigned>((pos ^ (i * RPL & 15)) << 4), 0, 0, 0);
        };
        auto read_raw = [&](u32x4 (&raw)[KS][4]) __attribute__((always_inline)) {
            int lane_o = lane;
            asm volatile("; per-strip lane id" : "+v"(lane_o));
            const uint8_t* row = rbuf + (lane_o & 31) * ROWL;
#pragma unroll
            for (int j = 0; j < KL; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    raw[j][q] = *reinterpret_cast<const u32x4*>(row + (((8 * j + 4 * (lane_o >> 5) + q) ^ (lane_o & 15)) << 4));
        };
        auto convert = [&](int s, const u32x4 (&raw)[KS][4], v8i (&x)[KS], float& sxm) __attribute__((always_inline)) {
            // max over the lane's values of the 15 magnitude bits, two per word
            typedef unsigned short us2 __attribute__((ext_vector_type(2)));
            us2 a2 = {0, 0};
#pragma unroll
            for (int j = 0; j < KS; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) a2 = __builtin_elementwise_max(a2, __builtin_bit_cast(us2, raw[j][q][e] & 0x7FFF7FFFu));
                }
            unsigned am = a2[0] > a2[1] ? a2[0] : a2[1];
            const unsigned other = static_cast<unsigned>(__shfl_xor(static_cast<int>(am), 32, 64));
            am = am > other ? am : other;
            float scale, inv;
            group_scale(__uint_as_float(am << 16), scale, inv);
            sxm = scale;
            const int m = (s - s_base) * 32 + l32;
            if (p.sx_out && hk == 0 && m < p.M) p.sx_out[static_cast<int64_t>(g) * p.M + m] = scale;
            auto cast = [&](auto finite_tag) __attribute__((always_inline)) {
                auto four = [&](float a, float b, float c, float d) __attribute__((always_inline)) {
                    return static_cast<int>(decltype(finite_tag)::value ? e4m3x4_finite(a, b, c, d) : e4m3x4(a, b, c, d));
                };
#pragma unroll
                for (int j = 0; j < KS; ++j) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const u32x4 w = raw[j][q];
                        x[j][2 * q] = four(bf16_lo(w.x) * inv, bf16_hi(w.x) * inv, bf16_lo(w.y) * inv, bf16_hi(w.y) * inv);
                        x[j][2 * q + 1] = four(bf16_lo(w.z) * inv, bf16_hi(w.z) * inv, bf16_lo(w.w) * inv, bf16_hi(w.w) * inv);
                    }
                }
            };
            // (four waves: one path, two take 80 registers more)
            if (NWV == 4 || any_not_finite(am)) cast(std::false_type{}); else cast(std::true_type{});
        };

        // MFMAs of one phase of a strip.  Lane-derived LDS addresses restart from an opaque copy of the lane id in
        // every call: W and the tables do not change between strips, and derived from loop invariants their reads
        // would be hoisted out of the strip loop into hundreds of registers.
        auto mma = [&](const v8i (&x)[KS], v16f (&acc)[NB]) __attribute__((always_inline)) {
            int lane_o = lane;
            asm volatile("; per-strip lane id" : "+v"(lane_o));
            const int l32 = lane_o & 31, hk = lane_o >> 5;
            // W fragment addresses: MFMA row rho of a 32-row block is fed W row wperm(rho) (see the file comment);
            // 32 nb rows further down for column block nb (which does not change the swizzle key: SWIN <= 16)
            const int wperm = 16 * ((l32 >> 2) & 1) + 4 * (l32 >> 3) + (l32 & 3);
            const int wkey = wperm & KEYMASK;
            // W fragments are read PF MFMAs ahead of their use (an LDS round trip is several MFMAs long)
            const uint8_t* wbase = smem + C::OFF_W + wperm * KB;
            constexpr int NF = NB * KS, PF = 4;
            v8i wf[PF];
            auto read_w = [&](int f) __attribute__((always_inline)) {           // f = j * NB + nb
                const int j = f / NB, nb = f % NB;
                const v4i lo = *reinterpret_cast<const v4i*>(wbase + nb * 32 * KB + (((4 * j + 2 * hk) ^ wkey) << 4));
                const v4i hi = *reinterpret_cast<const v4i*>(wbase + nb * 32 * KB + (((4 * j + 2 * hk + 1) ^ wkey) << 4));
                wf[f % PF] = v8i{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
            };
#pragma unroll
            for (int f = 0; f < PF - 1 && f < NF; ++f) read_w(f);
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                __builtin_amdgcn_sched_barrier(0);
                if (f + PF - 1 < NF) read_w(f + PF - 1);
                acc[f % NB] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(wf[f % PF], x[f / NB], acc[f % NB], 0, 0, 0, 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        };

        // scales, row statistics, normalization and store of one strip, from registers
        auto epilogue = [&](int s, const float sxm, v16f (&acc)[NB]) __attribute__((always_inline)) {
            int lane_o = lane;
            asm volatile("; per-strip lane id" : "+v"(lane_o));
            const int l32 = lane_o & 31, hk = lane_o >> 5;
            const int m = (s - s_base) * 32 + l32;

            // ---- scales: Y = acc * sx[m] * sw[n]
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                const v4f* sw4 = reinterpret_cast<const v4f*>(smem + C::OFF_SW + (nb * 32 + hk * 16) * 4);
#pragma unroll
                for (int a = 0; a < 4; ++a) {
                    const v4f sc = sw4[a];
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[nb][4 * a + e] *= sc[e] * sxm;
                }
            }
            if (p.y && m < p.M) {
                float* yrow = p.y + static_cast<int64_t>(g) * p.strideO + static_cast<int64_t>(m) * p.N;
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
                    if (nb * 32 + hk * 16 < p.N) {
#pragma unroll
                        for (int a = 0; a < 4; ++a)
                            *reinterpret_cast<v4f*>(yrow + nb * 32 + hk * 16 + 4 * a) =
                                v4f{acc[nb][4 * a], acc[nb][4 * a + 1], acc[nb][4 * a + 2], acc[nb][4 * a + 3]};
                    }
            }

            // ---- row statistics: this lane's columns, then the lane that holds the row's other columns
            float mean = 0.f, rstd = 1.f;
            if (p.norm != LOKA_NORM_NONE) {
                float m2 = 0.f;
                if constexpr (SHORT_ROWS) {                           // (the same bits whatever the output's type)
                    // (branch-free; columns past N hold zeros: they add nothing to the sums, and their centred value is taken as zero)
                    float q4[4] = {0.f, 0.f, 0.f, 0.f};
                    if (ln) {
                        float s4[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                            for (int i = 0; i < 16; ++i) s4[i & 3] += acc[nb][i];
                        const float sum = (s4[0] + s4[1]) + (s4[2] + s4[3]);
                        const float mean_l = sum * rc_lane;
#pragma unroll
                        for (int nb = 0; nb < NB; ++nb) {
                            const float mean_in = nb * 32 + hk * 16 < p.N ? mean_l : 0.f;
#pragma unroll
                            for (int i = 0; i < 16; ++i) { const float d = acc[nb][i] - mean_in; q4[i & 3] = __builtin_fmaf(d, d, q4[i & 3]); }
                        }
                        // the other half of the row is in lane ^ 32: identical bits on both
                        mean = half_lanes_sum(sum) * inv_n;
                        const float d = mean_l - mean;
                        m2 = half_lanes_sum(__builtin_fmaf(cnt_lane * d, d, (q4[0] + q4[1]) + (q4[2] + q4[3])));
                    } else {
#pragma unroll
                        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                            for (int i = 0; i < 16; ++i) q4[i & 3] = __builtin_fmaf(acc[nb][i], acc[nb][i], q4[i & 3]);
                        m2 = half_lanes_sum((q4[0] + q4[1]) + (q4[2] + q4[3]));
                    }
                } else {
                    if (ln) {
                        float n_ = cnt_lane, sum = 0.f;
#pragma unroll
                        for (int nb = 0; nb < NB; ++nb)
                            if (nb * 32 + hk * 16 < p.N) {
#pragma unroll
                                for (int i = 0; i < 16; ++i) sum += acc[nb][i];
                            }
                        mean = n_ > 0.f ? sum * __builtin_amdgcn_rcpf(n_) : 0.f;
#pragma unroll
                        for (int nb = 0; nb < NB; ++nb)
                            if (nb * 32 + hk * 16 < p.N) {
#pragma unroll
                                for (int i = 0; i < 16; ++i) { const float d = acc[nb][i] - mean; m2 = __builtin_fmaf(d, d, m2); }
                            }
                        // symmetric Chan merge: identical bits on both lanes
                        const float nb_ = wave_shfl_xor(n_, 32), mb = wave_shfl_xor(mean, 32), m2b = wave_shfl_xor(m2, 32);
                        const float nn = n_ + nb_;
                        if (nn > 0.f) {
                            const float d = mb - mean;
                            const float rn = __builtin_amdgcn_rcpf(nn);
                            const float newmean = (n_ * mean + nb_ * mb) * rn;
                            m2 = m2 + m2b + d * d * (n_ * nb_ * rn);
                            mean = newmean;
                        }
                    } else {
#pragma unroll
                        for (int nb = 0; nb < NB; ++nb)
                            if (nb * 32 + hk * 16 < p.N) {
#pragma unroll
                                for (int i = 0; i < 16; ++i) m2 = __builtin_fmaf(acc[nb][i], acc[nb][i], m2);
                            }
                        m2 += wave_shfl_xor(m2, 32);
                    }
                }
                rstd = __builtin_amdgcn_rsqf(m2 * inv_n + p.eps);
            }
            const float nmr = -mean * rstd;

            // ---- normalize, affine, bf16.  A lane holds 16 consecutive columns (32 bytes) of ONE row per column
            // block; stored from there an instruction writes 16-byte pieces 32 bytes apart in 32 rows.  Each wave
            // instead passes the 32 x 64-byte block through 2 KB of its own LDS (16-byte chunk c of row r at
            // position c ^ (r / 4 % 4): conflict-free both ways) and stores it with 4 lanes per row: 16 full 64-byte
            // runs per instruction.  LDS executes one wave's instructions in order: no barrier, one buffer.
            uint8_t* const tbuf = smem + C::OFF_T + wave * 2048;
            const int t_wr = l32 * 64, t_key = (l32 >> 2) & 3;
            const int t_row = lane_o >> 2, t_c = lane_o & 3;                   // store side: row (+ 16 j), chunk
            // (buffer stores relative to the strip's first row: the descriptor ends with the last row that exists, columns past
            // N get an offset beyond it; every strip issues the same stores, no branch among them.)
            const int row0 = (s - s_base) * 32, rows_here = p.M - row0 < 32 ? p.M - row0 : 32;
            const __amdgpu_buffer_rsrc_t orsrc =
                FP8OUT ? __builtin_amdgcn_make_buffer_rsrc(p.outq + static_cast<int64_t>(g) * p.strideO + static_cast<int64_t>(row0) * p.N, 0,
                                                           rows_here * p.N, 0x00020000)
                       : __builtin_amdgcn_make_buffer_rsrc(p.out + static_cast<int64_t>(g) * p.strideO + static_cast<int64_t>(row0) * p.N, 0,
                                                           rows_here * p.N * 2, 0x00020000);
            uint16_t* const obase = p.out + static_cast<int64_t>(g) * p.strideO + static_cast<int64_t>((s - s_base) * 32) * p.N;
            uint8_t* const qbase = p.outq + static_cast<int64_t>(g) * p.strideO + static_cast<int64_t>((s - s_base) * 32) * p.N;
            auto put = [&](const u32x4 v, int r, int ccol) __attribute__((always_inline)) {
                constexpr int ES = FP8OUT ? 1 : 2;                              // bytes per value
                if constexpr (LEAN) {
                    __builtin_amdgcn_raw_buffer_store_b128(v, orsrc, ccol < p.N ? (r * p.N + ccol) * ES : 0x7FFFFFF0, 0, 0);
                } else {
                    if ((s - s_base) * 32 + r < p.M && ccol < p.N) {
                        if (FP8OUT) *reinterpret_cast<u32x4*>(qbase + static_cast<int64_t>(r) * p.N + ccol) = v;
                        else *reinterpret_cast<u32x4*>(obase + static_cast<int64_t>(r) * p.N + ccol) = v;
                    }
                }
            };
            // The affine step (without gamma and beta it is x * 1 + 0: skipped, same bits, no table reads)
            auto affine_step = [&](float (&o)[8], int nb, int half) __attribute__((always_inline)) {
                const int col = nb * 32 + hk * 16;
                const v4f* g4 = reinterpret_cast<const v4f*>(smem + C::OFF_GM + col * 4);
                const v4f* b4 = reinterpret_cast<const v4f*>(smem + C::OFF_BT + col * 4);
                const v4f gq0 = g4[2 * half], gq1 = g4[2 * half + 1], bq0 = b4[2 * half], bq1 = b4[2 * half + 1];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    o[e] = __builtin_fmaf(o[e], gq0[e], bq0[e]);
                    o[4 + e] = __builtin_fmaf(o[4 + e], gq1[e], bq1[e]);
                }
            };
            // (affine: a compile-time constant per path, or (ONE_PATH) the run-time flag)
            auto normalize_store = [&](auto affine) __attribute__((always_inline)) {
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    float o[2][8];
#pragma unroll
                    for (int half = 0; half < 2; ++half)
#pragma unroll
                        for (int e = 0; e < 8; ++e) o[half][e] = __builtin_fmaf(acc[nb][8 * half + e], rstd, nmr);
                    if (affine) { affine_step(o[0], nb, 0); affine_step(o[1], nb, 1); }
#pragma unroll
                    for (int half = 0; half < 2; ++half) {
                        u32x4 pk;
                        pk.x = pack_bf16x2(o[half][0], o[half][1]); pk.y = pack_bf16x2(o[half][2], o[half][3]);
                        pk.z = pack_bf16x2(o[half][4], o[half][5]); pk.w = pack_bf16x2(o[half][6], o[half][7]);
                        *reinterpret_cast<u32x4*>(tbuf + t_wr + (((2 * hk + half) ^ t_key) << 4)) = pk;
                    }
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        const int r = 16 * j + t_row;
                        const u32x4 pk = *reinterpret_cast<const u32x4*>(tbuf + r * 64 + ((t_c ^ ((r >> 2) & 3)) << 4));
                        const int ccol = nb * 32 + t_c * 8;
                        put(pk, r, ccol);
                    }
                }
            };
            // FP8 output for the next layer (Section 3.2: quantization fused before the output is written): the
            // bf16 values above, quantized per row exactly as the quantize entry point would quantize the stored bf16
            // tensor.  The whole row lives in this lane and lane ^ 32, so the row amax needs one exchange; the values
            // are then computed a second time (keeping 128 packed values would not fit beside the accumulators),
            // cast, and leave through the same staging buffer, two column blocks (64 codes per row) at a time.
            auto normalize_store_fp8 = [&](auto affine) __attribute__((always_inline)) {
                auto packed8 = [&](int nb, int half) __attribute__((always_inline)) {
                    float o[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) o[e] = __builtin_fmaf(acc[nb][8 * half + e], rstd, nmr);
                    if (affine) affine_step(o, nb, half);
                    u32x4 pk;
                    pk.x = pack_bf16x2(o[0], o[1]); pk.y = pack_bf16x2(o[2], o[3]);
                    pk.z = pack_bf16x2(o[4], o[5]); pk.w = pack_bf16x2(o[6], o[7]);
                    return pk;
                };
                unsigned am = 0u;
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
                    if (nb * 32 + hk * 16 < p.N) {
#pragma unroll
                        for (int half = 0; half < 2; ++half) {
                            const u32x4 pk = packed8(nb, half);
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                const unsigned lo = pk[e] & 0x7FFFu, hi = (pk[e] >> 16) & 0x7FFFu;
                                am = am > lo ? am : lo;
                                am = am > hi ? am : hi;
                            }
                        }
                    }
                const unsigned other = static_cast<unsigned>(__shfl_xor(static_cast<int>(am), 32, 64));
                am = am > other ? am : other;
                float scale, inv;
                group_scale(__uint_as_float(am << 16), scale, inv);
                if (hk == 0 && m < p.M) p.outs[static_cast<int64_t>(g) * p.M + m] = scale;
#pragma unroll
                for (int nbp = 0; nbp < NB / 2; ++nbp) {
#pragma unroll
                    for (int q = 0; q < 2; ++q) {
                        const int nb = 2 * nbp + q;
                        const u32x4 p0 = packed8(nb, 0), p1 = packed8(nb, 1);
                        u32x4 ck;
                        ck.x = e4m3x4(bf16_lo(p0.x) * inv, bf16_hi(p0.x) * inv, bf16_lo(p0.y) * inv, bf16_hi(p0.y) * inv);
                        ck.y = e4m3x4(bf16_lo(p0.z) * inv, bf16_hi(p0.z) * inv, bf16_lo(p0.w) * inv, bf16_hi(p0.w) * inv);
                        ck.z = e4m3x4(bf16_lo(p1.x) * inv, bf16_hi(p1.x) * inv, bf16_lo(p1.y) * inv, bf16_hi(p1.y) * inv);
                        ck.w = e4m3x4(bf16_lo(p1.z) * inv, bf16_hi(p1.z) * inv, bf16_lo(p1.w) * inv, bf16_hi(p1.w) * inv);
                        *reinterpret_cast<u32x4*>(tbuf + t_wr + (((2 * q + hk) ^ t_key) << 4)) = ck;
                    }
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        const int r = 16 * j + t_row;
                        const u32x4 ck = *reinterpret_cast<const u32x4*>(tbuf + r * 64 + ((t_c ^ ((r >> 2) & 3)) << 4));
                        const int ccol = nbp * 64 + t_c * 16;
                        put(ck, r, ccol);
                    }
                }
            };
            // (an instantiation of its own: in one kernel with the bf16 form the larger shapes spill more)
            if (FP8OUT) {
                if (affine) normalize_store_fp8(std::true_type{}); else normalize_store_fp8(std::false_type{});
            } else {
                if constexpr (ONE_PATH) normalize_store(affine);
                // (fused: each path ends in a line of its own; with their last stores merged into one tail 64 x (4096 x 256 x 256),
                // M x N x K, takes 65.2 us instead of 65.0)
                else if (affine) { normalize_store(std::true_type{}); if (BF16IN) asm volatile("; stored, affine"); }
                else { normalize_store(std::false_type{}); if (BF16IN) asm volatile("; stored"); }
            }
        };

        // ---- this wave's strips of the segment
        v8i x[KS];
        float sxm = 0.f;
        if (NPH == 1 && BF16IN) {
            // as below, with the raw strip in a register set of its own: requested right after the previous strip's
            // values have been cast, in flight through that strip's MFMAs and epilogue
            u32x4 raw[KS][4];
            int s = t + wave;
            if (s < seg_end) {
                if (RAWLDS) request_raw(s);
                load_raw(s, raw, KL);
            }
            if (RAWLDS) wait_vmcnt<0>();
            while (s < seg_end) {
                const bool more = s + NWV < seg_end;
                if (RAWLDS) {
                    read_raw(raw);
                    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // the strip has been read: its place is free
                    // (With half of the strip in registers convert waits for what has just been requested too: the compiler
                    // does not know how much is younger than that half.  Requested behind the MFMAs instead, 64 x (4096 x
                    // 256 x 256), M x N x K, takes 58.2 us where it takes 59.6, but as long, 64.9, on buffers that no cache
                    // holds, and there 11 of 124 layers were 2 to 8 % slower, 43 faster.)
                    if (more) request_raw(s + NWV);
                }
                convert(s, raw, x, sxm);
                if (more) load_raw(s + NWV, raw, KL);
                __builtin_amdgcn_sched_barrier(0);
                v16f acc[NB];
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                    for (int i = 0; i < 16; ++i) acc[nb][i] = 0.f;
                mma(x, acc);
                epilogue(s, sxm, acc);
                // what comes through LDS is there: of this wave's operations only the epilogue's 2 NB stores are younger
                if (RAWLDS) wait_vmcnt<2 * NB>();
                s += NWV;
            }
        } else if (NPH == 1) {
            // W is complete in LDS: the waves run on their own.  The next strip's operands are requested into the
            // same registers right after the last MFMA (x is dead then) and arrive during the epilogue.
            // (short rows: requested whether or not there is one - past the end beyond the descriptor, which reads zeros - and,
            // ONE_PATH, awaited by count: of this wave's operations only the epilogue's stores are younger)
            int s = t + wave;
            if (s < seg_end) load_x(s, 0, x, sxm, true);
            if constexpr (SHORT_ROWS) wait_vmcnt<0>();
            while (s < seg_end) {
                v16f acc[NB];
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                    for (int i = 0; i < 16; ++i) acc[nb][i] = 0.f;
                mma(x, acc);
                const float sx_cur = sxm;
                if constexpr (SHORT_ROWS) load_x(s + NWV, 0, x, sxm, s + NWV < seg_end);
                else if (s + NWV < seg_end) load_x(s + NWV, 0, x, sxm, true);
                __builtin_amdgcn_sched_barrier(0);
                epilogue(s, sx_cur, acc);
                if constexpr (ONE_PATH) wait_vmcnt<2 * NB>();
                s += NWV;
            }
        } else {
            // W is longer than the LDS: rounds of 8 strips (one per wave), and per round NPH phases in which all
            // waves multiply the same K slab of W; the epilogues still run unsynchronized
            const int rounds = (seg_end - t + NWV - 1) / NWV;
            for (int r = 0; r < rounds; ++r) {
                const int s = t + NWV * r + wave;
                const bool active = s < seg_end;
                v16f acc[NB];
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                    for (int i = 0; i < 16; ++i) acc[nb][i] = 0.f;
                for (int ph = 0; ph < NPH; ++ph) {
                    __syncthreads();                            // every wave has read the previous slab (and the tables are written)
                    load_w(ph);
                    if (active) load_x(s, ph, x, sxm, true);
                    wait_vmcnt<0>();
                    __syncthreads();
                    if (active) mma(x, acc);
                }
                if (active) epilogue(s, sxm, acc);
            }
        }
        t = seg_end;
    }
}

// ---------------------------------------------------------------------------------------------- host side
namespace {

struct StripInst {
    int nb, ks, nph;
    const void* fn;
    const void* fn_fused;      // bf16 X, quantization fused (single-phase instances only)
    const void* fn_q;          // e4m3 output
    size_t lds, lds_fused;
    void (*launch)(const GemmParams&, int, dim3, hipStream_t);
};

// waves of a fused-quantization instance: 8 where accumulators, the raw strip (or the half of it that is not in LDS) and the
// operands fit 256 registers, K <= 256; else 4 with up to 512 each (eight that spill were slower: 64 x (4096 x 256 x 256),
// M x N x K, 94 us where four took 65 and eight with half the strip in LDS take 63)
constexpr int fused_waves(int ks) { return ks <= 4 ? 8 : 4; }

template <int NB, int KS, int NPH>
void launch_strip(const GemmParams& p, int spp, dim3 grid, hipStream_t s) {
    if (p.xb) {
        if constexpr (NPH == 1 && KS <= 8)                      // (K = 1024: the raw strip alone would be 256 registers)
            gemm_strip_kernel<NB, KS, NPH, fused_waves(KS), true, false><<<grid, fused_waves(KS) * 64, StripCfg<NB, KS, NPH>::lds_fused(fused_waves(KS)), s>>>(p, spp);
    } else if (p.outq) {
        gemm_strip_kernel<NB, KS, NPH, 8, false, true><<<grid, 512, StripCfg<NB, KS, NPH>::LDS, s>>>(p, spp);
    } else {
        gemm_strip_kernel<NB, KS, NPH, 8, false, false><<<grid, 512, StripCfg<NB, KS, NPH>::LDS, s>>>(p, spp);
    }
}

template <int NB, int KS, int NPH>
const void* strip_fused_fn() {
    if constexpr (NPH == 1 && KS <= 8) return reinterpret_cast<const void*>(&gemm_strip_kernel<NB, KS, NPH, fused_waves(KS), true, false>);
    else return nullptr;
}

#define LOKA_STRIP(NB, KS, NPH)                                                                                     \
    {NB, KS, NPH, reinterpret_cast<const void*>(&gemm_strip_kernel<NB, KS, NPH, 8, false, false>), strip_fused_fn<NB, KS, NPH>(), \
     reinterpret_cast<const void*>(&gemm_strip_kernel<NB, KS, NPH, 8, false, true>), StripCfg<NB, KS, NPH>::LDS, StripCfg<NB, KS, NPH>::lds_fused(fused_waves(KS)), \
     &launch_strip<NB, KS, NPH>}

// column blocks, K steps per phase, phases (K = 64 KS NPH; one phase when W fits the LDS)
const StripInst kStrip[] = {LOKA_STRIP(4, 2, 1), LOKA_STRIP(4, 4, 1), LOKA_STRIP(4, 8, 1), LOKA_STRIP(4, 16, 1),
                            LOKA_STRIP(8, 2, 1), LOKA_STRIP(8, 4, 1), LOKA_STRIP(8, 8, 1), LOKA_STRIP(8, 8, 2)};

const StripInst* strip_pick(int64_t N, int64_t K) {
    if (K % 64 || N > 256) return nullptr;
    const int ks = static_cast<int>(K / 64), nb = N <= 128 ? 4 : 8;
    for (const StripInst& w : kStrip)
        if (w.nb == nb && w.ks * w.nph == ks) return &w;
    return nullptr;
}

}  // namespace

bool strip_supports(int64_t M, int64_t N, int64_t K) {
    return strip_pick(N, K) != nullptr && M * K < (int64_t(1) << 31) && M < (int64_t(1) << 26);
}

// Workgroups to launch and the kernel's entry (for the dynamic-LDS attribute); 0 when unsupported.
bool strip_supports_fused(int64_t M, int64_t N, int64_t K) {
    const StripInst* w = strip_pick(N, K);
    return w != nullptr && w->fn_fused != nullptr && strip_supports(M, N, K) && M * K < (int64_t(1) << 30);
}

int strip_plan(int64_t M, int64_t N, int64_t K, int64_t batch, int cus, bool bf16_in, bool fp8_out, const void** fn,
               size_t* lds) {
    const StripInst* w = strip_pick(N, K);
    if (!w || (bf16_in && (!w->fn_fused || fp8_out))) return 0;
    *fn = bf16_in ? w->fn_fused : fp8_out ? w->fn_q : w->fn;
    *lds = bf16_in ? w->lds_fused : w->lds;
    const int64_t strips = batch * ((M + 31) / 32);
    // (one strip per workgroup while CUs are free, though only one wave of it then works: measured with fused quantization,
    // M x N x K: 1311 x 112 x 256 10.4 -> 7.2 us, 9815 x 112 x 128 8.6 -> 6.8, 32 x (1348 x 128 x 256) 17.9 -> 13.2)
    return static_cast<int>(strips < cus ? strips : cus);
}

void strip_launch(const GemmParams& p, dim3 grid, hipStream_t s) {
    const StripInst* w = strip_pick(p.N, p.KB);
    w->launch(p, (p.M + 31) / 32, grid, s);
}

}  // namespace loka
