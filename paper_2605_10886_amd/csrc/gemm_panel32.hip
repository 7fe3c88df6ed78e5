// Large-tile FP8 GEMM with the row norm fused across workgroups: 256 x 256 tiles, 8 waves, persistent
// panel-synchronous schedule (see gemm.hip for the schedule's description; this file is its throughput-oriented
// instantiation).
//
// Matrix instruction: v_mfma_f32_16x16x128_f8f6f4 where the accumulators take nothing but products (one scale per row,
// column or tensor, power-of-two block scales), v_mfma_f32_32x32x64_f8f6f4 where block scales rescale them, 32x32x16 for the
// BF16 reference.  From registers the 32 x 32 form issues back to back at 98 % of the FP8 rate in one wave where the
// 16 x 16 form reaches 70 - 80 %, but only while the operands do not change: on changing operands the chip holds the first to
// 2.3 - 2.5 PFLOP/s and the second to 3.7 - 4.0.  Whole launches, M x N x K, us, 32 x 32 x 64 -> 16 x 16 x 128 (with the
// main loop below): 32768 x 4096 x 4096 472 -> 451, without a norm 460 -> 434, with FP8 output 468 -> 446; 16384 x 2048 x 8192
// 213 -> 202; 2048 x 1024 x 123200 in K ranges 245 -> 230; 12000 x 2560 x 3072 93.7 -> 90.8; 8192 x 2048 x 2048 36.5 -> 35.7;
// K = 256 and 512 the same within 1 % where a workgroup has several tiles.  The exchange into the 32 x 32 layout costs 0.3 - 0.6 us a
// tile: a launch of one round of few K steps is 2 - 5 % longer (over 496 shapes beside the former form, medians: one round to 4 K steps
// 1.04, to 16 1.02, more 0.99; two rounds 1.02, 0.98, 0.96; more 1.00, 0.98, 0.97).  Power-of-two block scales 32768 x 4096 x 4096
// 511 -> 488, 8192 x 2048 x 2048 38.5 -> 36.6.
//
// Work split: waves 0..3 own rows 0..127 of the tile, waves 4..7 rows 128..255; wave w % 4 owns columns
// [64 (w % 4), +64).  Per K step of 128 bytes a wave runs 8 (row tiles of 16) x 4 (column tiles of 16) = 32 MFMAs, or
// 4 x 2 tiles of 32 x 2 K halves of 64 = 16, from 12 operand fragments of 8 registers.
//
// Operand roles are swapped as in gemm.hip (W rows -> MFMA rows, X rows -> MFMA columns).  In the 32 x 32 form MFMA row
// rho = 8a + 4h + b (a = 0..3, h = lane / 32, b = 0..3) is fed W row 16h + 4a + b of the 32-row tile, so a
// lane ends with 16 CONSECUTIVE output columns (accumulator element i <-> column 16h + i) of one output
// row m = lane % 32, and the two lanes that share a row cover 32 consecutive columns.
//
// LDS: rows of 128 bytes, chunk c of row r at position c ^ key(r); X rows are read 16 consecutive rows at a
// time (key = (r >> 1) & 7); the W read pattern above touches rows {16h + 4a + b} with a in a pair
// {0,1} or {2,3} per 16 lanes: key = bits (1, 2, 4) of r.  Both give 16 lanes x 16 bytes on 64 distinct banks.
#include "gemm_common.h"

#include <type_traits>

namespace loka {

typedef float v16f __attribute__((ext_vector_type(16)));

// BW: 0 = one scale per row / column / tensor (applied in the epilogue); 1 = block scales, accumulators rescaled
// per K block; 2 = power-of-two block scales handed to the matrix cores (scaled MFMA), nothing to rescale.
// FP8OUT: instead of bf16 O the tile leaves as e4m3 codes with one scale per output row, exactly what a rowwise
// quantization of the bf16 output would give.  Without an affine step the normalized value (y - mean) * rstd grows
// with y, and so does its bf16 rounding: the row's largest magnitude is reached at the row's largest or smallest
// y, so the row minimum and maximum travel with the row statistics in the ONE exchange between the workgroups of a
// panel and every workgroup derives the row scale from them.  With gamma / beta the extremum can sit anywhere: the
// tile is normalized first and the row amax of the result crosses the workgroups in a second exchange.
// F8: 0 = bf16 output, 1 = FP8 output without gamma / beta (one exchange), 2 = FP8 output with gamma / beta, BlockNorm
// or an activation (the row amax of the result crosses the workgroups in a second exchange; an instantiation of its
// own because it keeps the packed normalized tile in registers).
// Quantize prologue (QPRO instantiation; GemmParams::qpro): when a tile spans the whole output row (N <= 256), the 256
// rows of X a tile reads are read by no other workgroup, so the workgroup can quantize them itself - rowwise, exactly
// as the quantize entry point would (row amax, scale = amax / 448, code = e4m3(x * (448 / amax)); same helper
// functions, same bits) - write codes and row scales where the caller wants them, and then stream them back like any
// FP8 input (they come from this XCD's L2).  One launch instead of two; the only ordering needed is inside the
// workgroup: every wave waits for its stores to be acknowledged before the barrier in front of the first read.
// Wave w takes rows [32 w, +32) of each of the workgroup's tiles, RG rows at a time (16 loads of 16 bytes per lane in
// flight, the next group requested before the current one is converted); a row is LPR loads of a whole wave
// (K = 512 LPR elements).
template <int LPR>
__device__ __forceinline__ void panel32_quantize_own_rows(const GemmParams& p, int tile_first, int tile_stride, int total_tiles,
                                                          int wave) {
    constexpr int RG = 16 / LPR;                 // rows per group
    constexpr int NG = 32 / RG;                  // groups per tile and wave
    typedef unsigned short us2 __attribute__((ext_vector_type(2)));
    int lv = static_cast<int>(threadIdx.x) & 63;
    asm volatile("; lane id" : "+v"(lv));
    const int K = p.KB;                          // elements per row (= bytes per row of codes)
    u32x4 raw[2][RG][LPR];
    // group q of the workgroup's tile sequence: tile tile_first + (q / NG) * tile_stride, rows 32 wave + (q % NG) * RG + [0, RG)
    const int ntiles = tile_first < total_tiles ? (total_tiles - 1 - tile_first) / tile_stride + 1 : 0;
    const int ngroups = ntiles * NG;
    auto locate = [&](int q, int& g, int& m0) __attribute__((always_inline)) {
        const int tile = tile_first + (q / NG) * tile_stride;
        g = tile / p.tiles_m;                    // (tiles_n == 1)
        m0 = (tile - g * p.tiles_m) * 256 + 32 * wave + (q % NG) * RG;
    };
    auto fetch = [&](int q, u32x4 (&dst)[RG][LPR]) __attribute__((always_inline)) {
        int g, m0;
        locate(q, g, m0);
        const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<uint16_t*>(p.xb + static_cast<int64_t>(g) * p.strideX), 0, static_cast<unsigned>(p.M) * (2u * K), 0x00020000);
#pragma unroll
        for (int rr = 0; rr < RG; ++rr)
#pragma unroll
            for (int i = 0; i < LPR; ++i)
                // (rows past M lie beyond the descriptor's bound and read as zeros)
                dst[rr][i] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                                           xr, static_cast<unsigned>(m0 + rr) * (2u * K) + static_cast<unsigned>((i * 64 + lv) * 16), 0, 0));
    };
    auto convert = [&](int q, const u32x4 (&src)[RG][LPR]) __attribute__((always_inline)) {
        int g, m0;
        locate(q, g, m0);
        uint8_t* const xq = const_cast<uint8_t*>(p.X) + static_cast<int64_t>(g) * p.strideX;
        float* const sxo = const_cast<float*>(p.sx) + static_cast<int64_t>(g) * p.strideSx;
        // row amax: packed 16-bit maxima of the magnitudes (exact)
        unsigned mine = 0u;
#pragma unroll
        for (int rr = 0; rr < RG; ++rr) {
            us2 a2 = {0, 0};
#pragma unroll
            for (int i = 0; i < LPR; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) a2 = __builtin_elementwise_max(a2, __builtin_bit_cast(us2, src[rr][i][e] & 0x7FFF7FFFu));
            const unsigned a = lanes_max_bits<64>(a2[0] > a2[1] ? a2[0] : a2[1]);
            mine = (lv & 15) == rr ? a : mine;   // lane rr of 16 keeps row rr's amax: one division pair per lane, not per row and lane
        }
        float scale_l, inv_l;
        group_scale(__uint_as_float(mine << 16), scale_l, inv_l);
        if (lv < RG && m0 + lv < p.M) sxo[m0 + lv] = scale_l;
        static_assert(RG <= 16, "one row per lane of 16");
        float inv_b[RG];
        row_broadcasts<RG>(inv_l, inv_b);
#pragma unroll
        for (int rr = 0; rr < RG; ++rr) {
            const float inv = inv_b[rr];
            const bool live = m0 + rr < p.M;
#pragma unroll
            for (int i = 0; i < LPR; ++i) {
                const u32x4 w = src[rr][i];
                u32x2 o;
                o.x = e4m3x4(bf16_lo(w.x) * inv, bf16_hi(w.x) * inv, bf16_lo(w.y) * inv, bf16_hi(w.y) * inv);
                o.y = e4m3x4(bf16_lo(w.z) * inv, bf16_hi(w.z) * inv, bf16_lo(w.w) * inv, bf16_hi(w.w) * inv);
                if (live) *reinterpret_cast<u32x2*>(xq + static_cast<int64_t>(m0 + rr) * K + (i * 64 + lv) * 8) = o;
            }
        }
    };
    if (ngroups > 0) fetch(0, raw[0]);
    for (int q = 0; q < ngroups; q += 2) {
        // (two groups per iteration so that the buffers keep compile-time names)
        if (q + 1 < ngroups) { fetch(q + 1, raw[1]); wait_vmcnt<RG * LPR>(); } else wait_vmcnt<0>();
        convert(q, raw[0]);
        if (q + 1 < ngroups) {
            // ("at most RG * LPR operations outstanding" covers group q + 1 although the stores of group q are in
            // flight too: loads return in order, so whatever part of the completed operations are stores, the completed
            // loads are the oldest ones, and there are at least as many of them as group q + 1 has)
            if (q + 2 < ngroups) { fetch(q + 2, raw[0]); wait_vmcnt<RG * LPR>(); } else wait_vmcnt<0>();
            convert(q + 1, raw[1]);
        }
    }
    wait_vmcnt<0>();                             // codes and scales are in L2 before this wave passes the barrier
}

// Two forms leave as fp32 and normalize nothing (PART): EPI_SPLITK, one K range of one tile per workgroup, and BF16, the
// reference GEMM (KB = 2 K bytes per row, two v_mfma_f32_32x32x16_bf16 in the place of each FP8 instruction: the same
// bytes per fragment and the same matrix-pipe time per K step of 128 bytes, so the same main loop keeps the pipe full).
// RAGK: K need not be a multiple of the 128-byte step: in the last step the lanes whose 16-byte chunk lies past the end
// of the row read zeros, in both operands.
// YOUT false: the caller wants no fp32 Y, and the code that would store it is left out (230 instead of 242 registers;
// in the 32 x 32 form, quantize + GEMM at 32768 x 4096 x 4096, beside a kernel that stored Y straight from registers: 1.1 and 0.5 % slower with the code in, 0.3 and
// 0.4 % without it).
template <int EPI, int BW, int F8, bool QPRO = false, bool BF16 = false, bool RAGK = (EPI == EPI_SPLITK || BF16) && BW == 0, bool YOUT = true, bool QUAD = false>
__global__ __launch_bounds__(512) void gemm_panel32_kernel(const GemmParams p) {
    constexpr bool FP8OUT = F8 != 0;
    constexpr bool SPLITK = EPI == EPI_SPLITK, PART = SPLITK || BF16;
    static_assert(!PART || (!FP8OUT && !QPRO), "partial sums and the reference GEMM leave as fp32");
    constexpr bool BLOCKWISE = BW != 0;
    // Matrix instruction: 16 x 16 x 128 where the accumulators take nothing but products (see LOKA_PAIR)
    constexpr bool SQ16 = BW != 1 && !BF16;
    constexpr int BM = 256, BN = 256, NW = 8, WM = 128, WN = 64, MI = 4, NI = 2;
    constexpr int ES = 256 * 128;           // one ring entry: 256 rows x 128 bytes of X or of W
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wave_m = wave >> 2, wave_n = wave & 3;
    const bool grp_b = wave >= 4;           // the second wave of each SIMD
    const int l32 = lane & 31, hk = lane >> 5;

    const int total_tiles = p.tiles_m * p.tiles_n * p.batch;
    // (split K: ids run range by range, so an XCD's workgroups contract the same K range of neighbouring tiles)
    const int id = EPI == EPI_PANEL_SYNC && !panels_may_spread(gridDim.x, p.tiles_n) ? static_cast<int>(blockIdx.x)
                                                                                     : xcd_contiguous(blockIdx.x, gridDim.x);
    const int tile_first = SPLITK ? id % total_tiles : id, tile_stride = SPLITK ? total_tiles : gridDim.x;
    const int ks = SPLITK ? id / total_tiles : 0, k_lo = SPLITK ? ks * p.k_per_split : 0, kb0 = k_lo * 128;
    if (EPI == EPI_PANEL_SYNC) {
        // the workspace remembers which launch used it last (a wait that runs out records the same value beside it)
        if (p.header && blockIdx.x == 0 && threadIdx.x == 0)
            __hip_atomic_store(p.header, p.nonce, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    // loop-invariant lane offsets
    const int ld_row = lane >> 3, ld_pos = lane & 7;
    const int x_chunk = ((ld_pos ^ (ld_row >> 1)) << 4) ^ ((wave & 1) << 6);
    const int w_chunk = ((ld_pos ^ ((ld_row >> 1) & 3)) << 4) ^ (((wave >> 1) & 1) << 6);
    const int x_lane_off = ld_row * p.KB + x_chunk;
    const int w_lane_off = ld_row * p.KB + w_chunk;
    // chunks that exist in a ragged last K step
    const bool x_in = !RAGK || x_chunk < (p.KB & 127), w_in = !RAGK || w_chunk < (p.KB & 127);
    // fragment read offsets inside a stage: K half s uses chunks 4s + 2hk, 4s + 2hk + 1
    const int xrow = wave_m * WM + l32;                                    // + 32 mi
    const int xkey = (xrow >> 1) & 7;
    const int x_off0 = xrow * 128 + (((2 * hk) ^ xkey) << 4), x_off1 = xrow * 128 + (((2 * hk + 1) ^ xkey) << 4);
    const int wperm = 16 * ((l32 >> 2) & 1) + 4 * (l32 >> 3) + (l32 & 3);  // W row of the 32-row tile this lane feeds
    const int wrow = wave_n * WN + wperm;                                  // + 32 ni
    const int wkey = ((wrow >> 1) & 1) | (((wrow >> 2) & 1) << 1) | (((wrow >> 4) & 1) << 2);
    const int w_off0 = wrow * 128 + (((2 * hk) ^ wkey) << 4), w_off1 = wrow * 128 + (((2 * hk + 1) ^ wkey) << 4);
    const int ksteps_all = RAGK ? (p.KB + 127) / 128 : p.KB / 128;
    const int ksteps = SPLITK && ksteps_all - k_lo > p.k_per_split ? p.k_per_split : ksteps_all - k_lo;

    // n fastest where the tiles of a row panel run together, else in bands
    auto locate = [&](int t, int& tm_, int& tn_, int& g_) __attribute__((always_inline)) {
        g_ = t / (p.tiles_m * p.tiles_n);
        t -= g_ * p.tiles_m * p.tiles_n;
        if (PART) {
            banded_tile(t, p.tiles_m, p.tiles_n, tm_, tn_);
        } else {
            tm_ = t / p.tiles_n;
            tn_ = t - tm_ * p.tiles_n;
        }
    };
    // buffer descriptors of the tile whose operands are being streamed (bounds = the rows that exist: rows
    // past the end of X or W read as zeros)
    __amdgpu_buffer_rsrc_t x_rsrc, w_rsrc;
    uint8_t *x_base, *w_base;
    int x_bytes, w_bytes;
    auto set_rsrc = [&](int tile_id) __attribute__((always_inline)) {
        int tm_, tn_, g_;
        locate(tile_id, tm_, tn_, g_);
        const int m0_ = tm_ * BM, n0_ = tn_ * BN;
        const int x_rows = p.M - m0_ < BM ? p.M - m0_ : BM, w_rows = p.N - n0_ < BN ? p.N - n0_ : BN;
        x_base = const_cast<uint8_t*>(p.X + static_cast<int64_t>(g_) * p.strideX + static_cast<int64_t>(m0_) * p.KB);
        w_base = const_cast<uint8_t*>(p.W + static_cast<int64_t>(g_) * p.strideW + static_cast<int64_t>(n0_) * p.KB);
        x_bytes = x_rows * p.KB; w_bytes = w_rows * p.KB;
        x_rsrc = __builtin_amdgcn_make_buffer_rsrc(x_base, 0, x_bytes, 0x00020000);
        w_rsrc = __builtin_amdgcn_make_buffer_rsrc(w_base, 0, w_bytes, 0x00020000);
    };
    // ... or of nothing: what is requested then reads as zeros
    auto limit_rsrc = [&](bool more) __attribute__((always_inline)) {
        x_rsrc = __builtin_amdgcn_make_buffer_rsrc(x_base, 0, more ? x_bytes : 0, 0x00020000);
        w_rsrc = __builtin_amdgcn_make_buffer_rsrc(w_base, 0, more ? w_bytes : 0, 0x00020000);
    };
    bool prefetched = false;        // ring entries X(0) W(0) X(1) W(1) of `tile` were requested during the previous epilogue
    if (QPRO) {
        if (p.KB == 512) panel32_quantize_own_rows<1>(p, tile_first, tile_stride, total_tiles, wave);
        else if (p.KB == 1024) panel32_quantize_own_rows<2>(p, tile_first, tile_stride, total_tiles, wave);
        else panel32_quantize_own_rows<4>(p, tile_first, tile_stride, total_tiles, wave);
        __syncthreads();
    }

  for (int tile = tile_first; tile < total_tiles; tile += tile_stride) {
    int tm, tn, g;
    locate(tile, tm, tn, g);
    const int m0 = tm * BM, n0 = tn * BN;
    const float* sxg = p.sx + static_cast<int64_t>(g) * p.strideSx;
    const float* swg = p.sw + static_cast<int64_t>(g) * p.strideSw;
    if (!prefetched) set_rsrc(tile);
    // this wave's share of one ring entry (the X or the W rows of K step kb / 128) is four loads of 1 KB:
    // row groups wave, wave + 8, wave + 16, wave + 24; load j of an entry
    // (ragged rows: the offset is chosen per load from an opaque copy, or the choices of the first steps are kept from tile to
    // tile and spilled)
    auto issue_x1 = [&](int slot, int kb, int j) __attribute__((always_inline)) {
        const int grp = wave + j * NW;
        int x_lane = x_lane_off;
        if (RAGK) asm volatile("; lane offset" : "+v"(x_lane));
        __builtin_amdgcn_raw_ptr_buffer_load_lds(
            x_rsrc, (__attribute__((address_space(3))) void*)(smem + slot * ES + grp * 1024), 16,
            !RAGK || kb + kb0 + 128 <= p.KB || x_in ? x_lane : 0x7FFFFFFF, grp * 8 * p.KB + kb + kb0, 0, 0);
    };
    auto issue_w1 = [&](int slot, int kb, int j) __attribute__((always_inline)) {
        const int grp = wave + j * NW;
        int w_lane = w_lane_off;
        if (RAGK) asm volatile("; lane offset" : "+v"(w_lane));
        __builtin_amdgcn_raw_ptr_buffer_load_lds(
            w_rsrc, (__attribute__((address_space(3))) void*)(smem + slot * ES + grp * 1024), 16,
            !RAGK || kb + kb0 + 128 <= p.KB || w_in ? w_lane : 0x7FFFFFFF, grp * 8 * p.KB + kb + kb0, 0, 0);
    };
    auto issue_x = [&](int slot, int kb) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 4; ++j) issue_x1(slot, kb, j);
    };
    auto issue_w = [&](int slot, int kb) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 4; ++j) issue_w1(slot, kb, j);
    };

    v16f acc[MI][NI];
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[mi][ni][i] = 0.f;

    // Blockwise scales (1 x 128 for X, 128 x 128 for W): the accumulators are kept in units of the CURRENT K
    // block's scale s(kb) = sx[m, kb] * sw[kb, n / 128] (one value per lane and row tile: a wave's 64 columns lie
    // inside one 128-column block).  Entering block kb they are multiplied by s(kb - 1) / s(kb), the MFMAs of
    // the block then accumulate raw code products on top, and the epilogue multiplies by the last s: the sum
    // over kb of s(kb) * P(kb) without a second set of accumulators for the per-block partial products P.  The
    // 16 multiplies per tile and K step sit in front of the tile's first MFMA of the step (the vector ALU is idle
    // there).  One extra fp32 rounding of the running sum per K step (and a 1-ulp reciprocal in the ratio):
    // K / 128 * 2^-23 relative to sum |terms|, two orders below the matrix pipe's own truncation.
    // The scales of block k + 1 are fetched at the start of step k and used at its end.
    // Power-of-two block scales (BW == 2): every scale is 2^(e - 127) with e its fp32 exponent field, which is the
    // 8-bit scale format of the scaled MFMA: the instruction multiplies the products of a 32-element K run by
    // 2^(ea - 127) * 2^(eb - 127), ea / eb taken from the lane that holds the run.  A lane's X fragment is one
    // row's run (scale of that row and K block), a W fragment's 32 rows lie in one 128-column block (one scale
    // for the wave).  The accumulators then hold the scaled sum itself and the epilogue multiplies by nothing.
    // X's block scales lie [row][K block]: a lane reading one value per K step touches a cache line of its own each
    // time (as many L2 requests per step as the operands themselves need).  When a row's scales are 16-byte aligned
    // (K a multiple of 512) a lane fetches four K blocks at once, every fourth step (QUAD, an instantiation of its own: 541
    // against 555 us at 32768 x 4096 x 4096, 488 against 523 with power-of-two scales).
    float s_cur[MI], r_sc[MI], sx_nx[MI], sw_nx = 0.f;
    v4f sx_q[MI];
    int sc_x[MI], sc_w = 127;
    const int bw_nb = ((n0 + wave_n * WN < p.N ? n0 + wave_n * WN : p.N - 1) >> 7), bw_nblk = p.N >> 7;
    const float* const sx_tile = sxg + static_cast<int64_t>(m0) * ksteps_all + k_lo;
    unsigned sx_off[MI];                                     // this lane's rows in them, in bytes
    auto load_sx1 = [&](int mi, int k) __attribute__((always_inline)) {
        return *reinterpret_cast<const float*>(reinterpret_cast<const char*>(sx_tile + k) + sx_off[mi]);
    };
    auto load_sx4 = [&](int mi, int k) __attribute__((always_inline)) {
        return *reinterpret_cast<const v4f*>(reinterpret_cast<const char*>(sx_tile + k) + sx_off[mi]);
    };
    // the first block's scales
    auto bw_first = [&]() __attribute__((always_inline)) {
        if (!BLOCKWISE) return;
        const float sw0 = swg[static_cast<int64_t>(k_lo) * bw_nblk + bw_nb];
        float sx0[MI];
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) {
            const int r = wave_m * WM + mi * 32 + l32;
            sx_off[mi] = static_cast<unsigned>(m0 + r < p.M ? r : p.M - 1 - m0) * static_cast<unsigned>(ksteps_all * 4);
            if (QUAD) sx_q[mi] = load_sx4(mi, 0);
            else sx0[mi] = load_sx1(mi, 0);
        }
        if (!prefetched && ksteps > 1) { issue_x(3, 128); issue_w(4, 128); }
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) {
            if (QUAD) sx0[mi] = sx_q[mi][0];
            if (BW == 1) { s_cur[mi] = sx0[mi] * sw0; r_sc[mi] = 1.f; }
            else sc_x[mi] = static_cast<int>(__float_as_uint(sx0[mi]) >> 23);
        }
        if (BW == 2) sc_w = static_cast<int>(__float_as_uint(sw0) >> 23);
    };
    // requests the scales of block k + 1 (panel32_scale_loads(QUAD, k) loads)
    auto bw_fetch = [&](int k) __attribute__((always_inline)) {
        if (!BLOCKWISE) return;
        sw_nx = swg[static_cast<int64_t>(k_lo + k + 1) * bw_nblk + bw_nb];
        if (!QUAD) {
#pragma unroll
            for (int mi = 0; mi < MI; ++mi) sx_nx[mi] = load_sx1(mi, k + 1);
        } else if (((k + 1) & 3) == 0) {
#pragma unroll
            for (int mi = 0; mi < MI; ++mi) sx_q[mi] = load_sx4(mi, k + 1);
        }
    };
    // takes them, at the end of step k: the ratio to the last step's, or the exponents
    auto bw_use = [&](int k) __attribute__((always_inline)) {
        if (!BLOCKWISE) return;
        if (BW == 2) sc_w = static_cast<int>(__float_as_uint(sw_nx) >> 23);
        const int j = (k + 1) & 3;
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) {
            float sx;
            if (QUAD) {
                const float lo = j & 1 ? sx_q[mi][1] : sx_q[mi][0], hi = j & 1 ? sx_q[mi][3] : sx_q[mi][2];
                sx = j & 2 ? hi : lo;
            } else {
                sx = sx_nx[mi];
            }
            if (BW == 1) {
                const float s_new = sx * sw_nx;
                r_sc[mi] = s_cur[mi] * __builtin_amdgcn_rcpf(s_new);
                s_cur[mi] = s_new;
            } else {
                sc_x[mi] = static_cast<int>(__float_as_uint(sx) >> 23);
            }
        }
    };

    // Fragments of one K half (64 bytes): 2 W (two sets, double buffered) and 4 X (one set, refilled in place
    // as soon as the two MFMAs that use a fragment have been issued) of 8 registers each.
    v8i bx[MI], aw[2][NI];
    auto read_w = [&](int slot, int s, int set) __attribute__((always_inline)) {
        const uint8_t* ws = smem + slot * ES;
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) {
            const v4i lo = *reinterpret_cast<const v4i*>(ws + (w_off0 ^ (s << 6)) + ni * 32 * 128);
            const v4i hi = *reinterpret_cast<const v4i*>(ws + (w_off1 ^ (s << 6)) + ni * 32 * 128);
            aw[set][ni] = v8i{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        }
    };
    auto read_x = [&](int slot, int s, int mi) __attribute__((always_inline)) {
        const uint8_t* xs = smem + slot * ES + mi * 32 * 128;
        const v4i lo = *reinterpret_cast<const v4i*>(xs + (x_off0 ^ (s << 6)));
        const v4i hi = *reinterpret_cast<const v4i*>(xs + (x_off1 ^ (s << 6)));
        bx[mi] = v8i{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    };
    auto mfma_one = [&](int mi, int ni, int set) __attribute__((always_inline)) {
        if constexpr (BF16) {
            const v8i a = aw[set][ni], b = bx[mi];
            acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, v4i{a[0], a[1], a[2], a[3]}),
                                                                  __builtin_bit_cast(v8bf, v4i{b[0], b[1], b[2], b[3]}), acc[mi][ni], 0, 0, 0);
            acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, v4i{a[4], a[5], a[6], a[7]}),
                                                                  __builtin_bit_cast(v8bf, v4i{b[4], b[5], b[6], b[7]}), acc[mi][ni], 0, 0, 0);
        } else
            acc[mi][ni] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(aw[set][ni], bx[mi], acc[mi][ni], 0, 0, 0, 0, 0, 0);
    };
    auto mfma_row = [&](int mi, int set) __attribute__((always_inline)) {
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) mfma_one(mi, ni, set);
    };
    // MFMAs of the K half whose W fragments are in SET, with the LDS reads of K half S_READ of the entries in
    // slots SLOT_X / SLOT_W, and this wave's four loads of one new ring entry (LD: 0 none, 1 an X entry, 2 a W
    // entry; into ld_slot, K offset ld_kb), spread between them in source order.  The matrix pipe then always
    // has an instruction queued: a burst of LDS reads or of loads keeps a wave in the issue stage for hundreds
    // of cycles (the load path accepts 64 bytes per clock per CU).  The two waves of a SIMD (w, w + 4) issue
    // their loads in different gaps, so one of them is always free to feed the pipe.
#define LOKA_HALF_STEP(SLOT_X, SLOT_W, S_READ, SET, LD, RESC)                              \
    do {                                                                             \
        __builtin_amdgcn_sched_barrier(0);                                           \
        read_w(SLOT_W, S_READ, (SET) ^ 1);                                           \
        _Pragma("unroll") for (int mi = 0; mi < MI; ++mi) {                          \
            __builtin_amdgcn_sched_barrier(0);                                       \
            if (BW == 1 && (RESC)) {                                                 \
                _Pragma("unroll") for (int ni = 0; ni < NI; ++ni)                    \
                    _Pragma("unroll") for (int i = 0; i < 16; ++i) acc[mi][ni][i] *= r_sc[mi]; \
            }                                                                        \
            mfma_one(mi, 0, SET);                                                    \
            __builtin_amdgcn_sched_barrier(0);                                       \
            if ((LD) == 1 && ld_x && (BLOCKWISE || !grp_b)) issue_x1(ld_x_slot, ld_x_kb, mi); \
            if ((LD) == 2 && ld_w && (BLOCKWISE || !grp_b)) issue_w1(ld_w_slot, ld_w_kb, mi);       \
            __builtin_amdgcn_sched_barrier(0);                                       \
            mfma_one(mi, 1, SET);                                                    \
            __builtin_amdgcn_sched_barrier(0);                                       \
            read_x(SLOT_X, S_READ, mi);                                              \
            if ((LD) == 1 && ld_x && !BLOCKWISE && grp_b) issue_x1(ld_x_slot, ld_x_kb, mi);        \
            if ((LD) == 2 && ld_w && !BLOCKWISE && grp_b) issue_w1(ld_w_slot, ld_w_kb, mi);        \
        }                                                                            \
        __builtin_amdgcn_sched_barrier(0);                                           \
    } while (0)

    // The same by 16 x 16 x 128 instructions, which sustain 3.7 - 4.0 PFLOP/s on changing operands from registers where the 32 x 32 x 64
    // form sustains 2.3 - 2.5.  A K step is four pairs of X fragments (16 rows each; pair = row tile mi), a pair eight
    // instructions: the step's four W fragments (32 registers) against both.  A pair's two X fragments are read while the
    // pair before it is multiplied (two sets of 16 registers); a W fragment is replaced by the next step's behind its
    // last instruction, in the step's last pair, and used again six instructions later.  So the last pair of a step reads
    // of the next one only, and the step's barrier stands in front of it.
    // acc16[mi][ni][2 t + x]: X rows 32 mi + 16 x + [0, 16), W rows of fragment (ni, t); lane (l16, q) holds the rows 4 q + r.  W row
    // 16 hk + 8 t + 4 s + r of the 32 is row 4 (2 hk + s) + r of fragment t: exchanging the odd rows of 16 lanes of x = 0 with the
    // even ones of x = 1 afterwards (one swap per two registers) leaves what the 32 x 32 form leaves, 16 consecutive
    // columns of row l % 32 in every lane, and one epilogue serves both.
    v4f acc16[MI][NI][4];
    v8i xf[2][2], wf[4];
    int sc_pair[2] = {127, 127};                             // (BW == 2) exponents of the pair's two row blocks
    // Lane (l16, kg) takes the chunks kg and kg + 4 of its row, X row l16 (+ 16 per fragment), W row w16 (+ 8 and + 32 per
    // fragment; neither changes the swizzle).  (From an opaque copy of the lane id: not kept from tile to tile.)
    const int lane16 = lane_id();
    const int l16 = lane16 & 15, kg = lane16 >> 4, w16 = wave_n * WN + 16 * (l16 >> 3) + 4 * ((l16 >> 2) & 1) + (l16 & 3);
    const int x_at = (wave_m * WM + l16) * 128 + ((kg ^ ((l16 >> 1) & 7)) << 4);
    const int w_at = w16 * 128 + ((kg ^ (((w16 >> 1) & 1) | (((w16 >> 2) & 1) << 1) | (((w16 >> 4) & 1) << 2))) << 4);
    if constexpr (SQ16) {
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                for (int u = 0; u < 4; ++u) acc16[mi][ni][u] = v4f{0.f, 0.f, 0.f, 0.f};
    }
    auto read16 = [&](const uint8_t* entry, int off) __attribute__((always_inline)) {
        const v4i lo = *reinterpret_cast<const v4i*>(entry + off);
        const v4i hi = *reinterpret_cast<const v4i*>(entry + (off ^ 64));
        return v8i{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    };
    auto read_x16 = [&](int slot, int pair, int x) __attribute__((always_inline)) {
        xf[pair & 1][x] = read16(smem + slot * ES + (32 * pair + 16 * x) * 128, x_at);
    };
    auto read_w16 = [&](int slot, int j) __attribute__((always_inline)) {
        wf[j] = read16(smem + slot * ES + (32 * (j >> 1) + 8 * (j & 1)) * 128, w_at);
    };
    auto mfma16 = [&](int mi, int x, int j) __attribute__((always_inline)) {
        v4f& a = acc16[mi][j >> 1][2 * (j & 1) + x];
        if constexpr (BW == 2) a = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(wf[j], xf[mi & 1][x], a, 0, 0, 0, sc_w, 0, sc_pair[x]);
        else a = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(wf[j], xf[mi & 1][x], a, 0, 0, 0, 0, 0, 0);
    };
    // Power-of-two block scales: a lane holds those of row l % 32 of every row tile, and needs those of rows l16 and 16 + l16: a
    // swap.  (Scales of any value multiply the accumulators between the instructions.  So did the 16 x 16 form, at most two
    // instructions ahead: 32768 x 4096 x 4096 555 -> 554 us, 2048 x 1024 x 32768 84.7 -> 84.0, but 16384 x 1024 x 1024 26.3 -> 27.0
    // and 65536 x 256 x 512 20.5 -> 21.1.)
    auto pair_scales = [&](int mi) __attribute__((always_inline)) {
        if constexpr (BW == 2) {
            const u32_pair r = __builtin_amdgcn_permlane16_swap(static_cast<unsigned>(sc_x[mi]), static_cast<unsigned>(sc_x[mi]), false, false);
            sc_pair[0] = static_cast<int>(r.x);
            sc_pair[1] = static_cast<int>(r.y);
        }
    };
    // Pair MI_ of a step; reads pair RP (-1: none) of the entry in slot RX and, NEXT, the W fragments of the entry in slot RW; this
    // wave's four loads LD as in LOKA_HALF_STEP.
#define LOKA_PAIR(MI_, RX, RP, NEXT, RW, LD)                                               \
    do {                                                                             \
        __builtin_amdgcn_sched_barrier(0);                                           \
        pair_scales(MI_);                                                            \
        _Pragma("unroll") for (int j = 0; j < 4; ++j) {                              \
            __builtin_amdgcn_sched_barrier(0);                                       \
            mfma16(MI_, 0, j);                                                       \
            __builtin_amdgcn_sched_barrier(0);                                       \
            if ((LD) == 1 && ld_x && (BLOCKWISE || !grp_b)) issue_x1(ld_x_slot, ld_x_kb, j);        \
            if ((LD) == 2 && ld_w && (BLOCKWISE || !grp_b)) issue_w1(ld_w_slot, ld_w_kb, j);        \
            if ((RP) >= 0 && (j & 1) == 0) read_x16(RX, RP, j >> 1);                 \
            __builtin_amdgcn_sched_barrier(0);                                       \
            mfma16(MI_, 1, j);                                                       \
            __builtin_amdgcn_sched_barrier(0);                                       \
            if (NEXT) read_w16(RW, j);                                               \
            if ((LD) == 1 && ld_x && !BLOCKWISE && grp_b) issue_x1(ld_x_slot, ld_x_kb, j);         \
            if ((LD) == 2 && ld_w && !BLOCKWISE && grp_b) issue_w1(ld_w_slot, ld_w_kb, j);         \
        }                                                                            \
        __builtin_amdgcn_sched_barrier(0);                                           \
    } while (0)

    // ---- main loop.  LDS holds a ring of five 32 KB entries X(0) W(0) X(1) W(1) X(2) ...; entry e lives in
    // slot e % 5.  One barrier per K step, when every wave has read X(k) and W(k) completely and every wave's share of
    // X(k + 1), W(k + 1) has landed: in the step's middle in the 32 x 32 form, which reads a half step ahead; in front of its last
    // quarter in the 16 x 16 form, whose pairs read one pair ahead and whose last pair reads X(k + 1) and W(k + 1).
    // The slot of X(k) then takes W(k + 2) (requested behind the barrier), the slot of W(k) takes X(k + 3) (first half, or
    // second quarter, of step k + 1): an X entry is requested 1.5 steps before its first read, a W entry one step (half the
    // bytes of a stage: the round trip through L2 under load is ~1 us for 64 KB, ~0.6 us for 32 KB; a step is ~1.2 us).
    // All of a wave's loads return in issue order, so "vmcnt(4)" = everything but the newest entry's share.
    auto mod5 = [](int v) { return v >= 5 ? v - 5 : v; };
    // entry e of a tile lives in slot (e + 1) % 5: slot 0, which the epilogue uses as scratch, is the last to fill
    if (!prefetched) {
        issue_x(1, 0);
        issue_w(2, 0);
        if (!BLOCKWISE && ksteps > 1) { issue_x(3, 128); issue_w(4, 128); }
    }
    // (block scales: requested between the operands of the first two steps, which they would hold up by a round trip in front.  The
    // compiler, which cannot count across the condition on the second step's, waits for those along with the scales.  Requested
    // on every path, zeros where there are none, and awaited by count: 8192 x 2048 x 2048 with its quantization 53.7 ->
    // 53.8 us, and over 149 layers 1.9 % slower in the geometric mean, with power-of-two scales the same.)
    bw_first();
    if (!BLOCKWISE && ksteps > 2) issue_x(0, 256);     // (block scales: in the first step)
    if (BLOCKWISE) {
        if (ksteps > 1) __builtin_amdgcn_s_waitcnt(0x0F78); else __builtin_amdgcn_s_waitcnt(0x0F70);
    } else if (ksteps > 2) {
        // loads return in issue order, so "at most 4 (12) outstanding" covers X(0), W(0) whatever else (the
        // previous tile's stores) is still in flight
        if (prefetched) __builtin_amdgcn_s_waitcnt(0x0F74); else __builtin_amdgcn_s_waitcnt(0x0F7C);
    } else if (ksteps > 1 && !prefetched) {
        __builtin_amdgcn_s_waitcnt(0x0F78);
    } else {
        __builtin_amdgcn_s_waitcnt(0x0F70);
    }
    lds_barrier();
    if constexpr (SQ16) {
#pragma unroll
        for (int j = 0; j < 4; ++j) read_w16(2, j);
        read_x16(1, 0, 0);
        read_x16(1, 0, 1);
    } else {
        read_w(2, 0, 0);
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) read_x(1, 0, mi);
    }
    int e5 = 1;                                                 // slot of X(k)
    // (the last K step is peeled: MFMAs under a condition inside the loop make the compiler copy accumulators)
    for (int k = 0; k + 1 < ksteps; ++k) {
        const int sw_cur = mod5(e5 + 1), sx_nxt = mod5(e5 + 2), sw_nxt = mod5(e5 + 3);
        // Block scales: every step requests the same loads in the same places (those past the last step read zeros into
        // free slots, both waves of a SIMD use the same gap), so that the compiler can count how many are younger than a
        // block's scales.  Under a condition it has to assume that none is, and waits for everything in flight at their
        // use: the ring had no depth then.  32768 x 4096 x 4096 604 -> 541 us, power-of-two scales 550 -> 488; 8192 x 2048 x
        // 2048 (one tile per CU) 47.5 -> 44 and 44.5 -> 40.3.
        const bool more = k + 2 < ksteps;
        const bool ld_x = BLOCKWISE || (k >= 1 && more), ld_w = BLOCKWISE || more;
        const int ld_x_slot = mod5(e5 + 4), ld_x_kb = (k + 2) * 128;    // X(k + 2) -> the slot W(k - 1) left
        const int ld_w_slot = e5, ld_w_kb = (k + 2) * 128;              // W(k + 2) -> the slot X(k) leaves
        if (BLOCKWISE) limit_rsrc(more);
        bw_fetch(k);
        if constexpr (SQ16) {
            LOKA_PAIR(0, e5, 1, false, 0, 0);
            LOKA_PAIR(1, e5, 2, false, 0, 1);
            LOKA_PAIR(2, e5, 3, false, 0, 0);
        } else {
            LOKA_HALF_STEP(e5, sw_cur, 1, 0, 1, 1);
        }
        // all but this step's newest loads: X(k + 2) (4) and, blockwise, the scales of block k + 1 (1 or MI + 1)
        if (!ld_w) __builtin_amdgcn_s_waitcnt(0x0F70);
        else if (!BLOCKWISE) __builtin_amdgcn_s_waitcnt(0x0F74);
        else if (panel32_scale_loads(QUAD, k) == 1) __builtin_amdgcn_s_waitcnt(0x0F75);
        else __builtin_amdgcn_s_waitcnt(0x0F79);
        lds_barrier();                                          // (also waits for this wave's LDS reads)
        if constexpr (SQ16) {
            LOKA_PAIR(3, sx_nxt, 0, true, sw_nxt, 2);
        } else {
            LOKA_HALF_STEP(sx_nxt, sw_nxt, 0, 1, 2, 0);
        }
        bw_use(k);
        e5 = sx_nxt;
    }
    {
        const bool ld_x = false, ld_w = false;
        const int ld_x_slot = 0, ld_x_kb = 0, ld_w_slot = 0, ld_w_kb = 0;
        if constexpr (SQ16) {
            LOKA_PAIR(0, e5, 1, false, 0, 0);
            LOKA_PAIR(1, e5, 2, false, 0, 0);
            LOKA_PAIR(2, e5, 3, false, 0, 0);
        } else {
            LOKA_HALF_STEP(e5, mod5(e5 + 1), 1, 0, 0, 1);
        }
        (void)ld_x; (void)ld_w; (void)ld_x_slot; (void)ld_x_kb; (void)ld_w_slot; (void)ld_w_kb;
    }
    {   // Epilogue scope.  Lane- and thread-derived offsets restart from opaque copies of the ids: derived from
        // loop-invariant values the compiler would compute them once before the tile loop and keep dozens of
        // registers live through the main loop.
    const int lane_o = lane_id(), tid_o = wave * 64 + lane_o;
    const int lane = lane_o, l32 = lane & 31, hk = lane >> 5;
    const unsigned tid = static_cast<unsigned>(tid_o);
    (void)lane;
    int n_o = p.N;                                          // (1 / N likewise: recomputed per tile, not kept in a register)
    asm volatile("; row length" : "+s"(n_o));
    const float inv_n = 1.0f / static_cast<float>(n_o);
    // scales of this lane's rows and columns: requested before the last eight MFMAs so that the round trip
    // through L2 is covered (the fragment registers of the other K half are free by now)
    // lane: rows m(mi) = m0 + 128 wave_m + 32 mi + l32; columns ncol(ni) + [0, 16), ncol = n0 + 64 wave_n + 32 ni + 16 hk
    const bool tensor_x = p.x_mode == LOKA_SCALE_TENSOR, tensor_w = p.w_mode == LOKA_SCALE_TENSOR;
    int ncol[NI];
#pragma unroll
    for (int ni = 0; ni < NI; ++ni) ncol[ni] = n0 + wave_n * WN + ni * 32 + hk * 16;     // N % 16 == 0: a run of 16 is all in or all out
    v4f s4q[NI][2];                                         // SQ16: columns 4 q .. of fragment (ni, t), row l16 of (mi, x): 24
    float sxq[MI][2];                                       // registers, 36 in the layout behind the exchange
    if constexpr (SQ16 && !BLOCKWISE) {
        // (buffer loads: one 32-bit offset per lane; columns past the last read as zeros)
        const int q = lane >> 4, r16 = lane & 15;
        const __amdgpu_buffer_rsrc_t sw_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(swg), 0, tensor_w ? 4 : n_o * 4, 0x00020000);
        const float sw_all = swg[0];
        // (the rows' descriptor starts at the tile: the scales of all of X can be more bytes than 32 bits count.  Rows past the last
        // take the first one's scale: a bound that follows from M costs one more round of argument loads at the start, 2 % of
        // a launch of one round.  With FP8 output it starts at a multiple of 2^20 rows, in which the tile lies, and ends with M:
        // 8192 x 1024 x 2048 31.2 us, from the tile on 31.6.)
        constexpr int kScaleRows = FP8OUT ? 1 << 20 : BM;
        static_assert(kScaleRows % BM == 0, "a tile's rows have one descriptor");
        const int m_at = FP8OUT ? m0 & (kScaleRows - 1) : 0, m_base = m0 - m_at, m_left = p.M - m_base;
        const int sx_bytes = !FP8OUT ? BM * 4 : tensor_x ? 4 : (m_left < kScaleRows ? m_left : kScaleRows) * 4;
        const __amdgpu_buffer_rsrc_t sx_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(tensor_x ? sxg : sxg + m_base), 0, sx_bytes, 0x00020000);
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const int c = n0 + wave_n * WN + ni * 32 + 16 * (q >> 1) + 8 * t + 4 * (q & 1);
                s4q[ni][t] = __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(sw_rsrc, c * 4, 0, 0));
                s4q[ni][t] = tensor_w ? v4f{sw_all, sw_all, sw_all, sw_all} : s4q[ni][t];
            }
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int x = 0; x < 2; ++x) {
                const int r = m_at + wave_m * WM + mi * 32 + 16 * x + r16;
                sxq[mi][x] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(sx_rsrc, tensor_x || (!FP8OUT && r >= m_left) ? 0 : r * 4, 0, 0));
            }
    }
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (SQ16) {
        const bool ld_x = false, ld_w = false;
        const int ld_x_slot = 0, ld_x_kb = 0, ld_w_slot = 0, ld_w_kb = 0;
        LOKA_PAIR(3, 0, -1, false, 0, 0);
        (void)ld_x; (void)ld_w; (void)ld_x_slot; (void)ld_x_kb; (void)ld_w_slot; (void)ld_w_kb;
    } else {
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) mfma_row(mi, 1);
    }
#undef LOKA_HALF_STEP
#undef LOKA_PAIR
    if (BLOCKWISE) wait_vmcnt<0>();                         // (the zeros requested past the last K step are in)
    __syncthreads();                                        // LDS is free for the epilogue
    // the next tile's first four ring entries stream in while this tile's statistics are exchanged
    prefetched = tile + tile_stride < total_tiles;
    if (prefetched) {
        set_rsrc(tile + tile_stride);
        issue_x(1, 0);
        issue_w(2, 0);
        if (ksteps > 1) { issue_x(3, 128); issue_w(4, 128); }
    }

    // ------------------------------------------------------------------ epilogue
    float2* red = reinterpret_cast<float2*>(smem);                                 // [4][BM] (mean, M2) of a wave's columns
    float2* fin = red + BM * 4;                                                    // [BM] (mean, rstd)
    float* finq = reinterpret_cast<float*>(fin + BM);                              // [BM] 448 / amax of the output row (FP8OUT)
    float* red2 = reinterpret_cast<float*>(smem + 16384);                          // [BM][4][2] (min, max) (FP8OUT); the
                                                                                   // transpose buffers take its place later
    const int64_t obase = static_cast<int64_t>(g) * p.strideO;
    if constexpr (SQ16) {
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const float v0 = BLOCKWISE ? acc16[mi][ni][2 * t][r] : acc16[mi][ni][2 * t][r] * (s4q[ni][t][r] * sxq[mi][0]);
                        const float v1 = BLOCKWISE ? acc16[mi][ni][2 * t + 1][r] : acc16[mi][ni][2 * t + 1][r] * (s4q[ni][t][r] * sxq[mi][1]);
                        const u32_pair sw = __builtin_amdgcn_permlane16_swap(__float_as_uint(v0), __float_as_uint(v1), false, false);
                        acc[mi][ni][8 * t + r] = __uint_as_float(sw.x);
                        acc[mi][ni][8 * t + 4 + r] = __uint_as_float(sw.y);
                    }
    }
    if (BW == 1) {
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
#pragma unroll
            for (int mi = 0; mi < MI; ++mi)
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[mi][ni][i] *= s_cur[mi];
    }
    // fp32 tile: split K's share of this range (its scales are factors of every term), the reference's Y, or the pre-norm Y
    // a caller asked for.  Each wave passes a 32 x 32 sub-tile through 4 KB of its own LDS (128-byte rows, 16-byte chunk c
    // of row r at position c ^ (r / 2 % 8)) and stores it with 8 lanes per row: whole 128-byte lines instead of 16 bytes in
    // each of 64 (16384 x 1024 x 1024 with Y, 67 MB: 47.2 -> 36.3 us).
    if (PART || (YOUT && p.y)) {
        float* const dst = SPLITK ? p.part + (static_cast<int64_t>(ks) * p.batch + g) * p.M * p.N : p.y + obase;
        uint8_t* const fbuf = smem + wave * 4096;
        const int f_row = lane >> 3, f_c = lane & 7;
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) {
#pragma unroll
                for (int a = 0; a < 4; ++a)
                    *reinterpret_cast<v4f*>(fbuf + l32 * 128 + (((4 * hk + a) ^ ((l32 >> 1) & 7)) << 4)) =
                        v4f{acc[mi][ni][4 * a], acc[mi][ni][4 * a + 1], acc[mi][ni][4 * a + 2], acc[mi][ni][4 * a + 3]};
                const int col = n0 + wave_n * WN + ni * 32 + f_c * 4;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int r = 8 * j + f_row, m = m0 + wave_m * WM + mi * 32 + r;
                    const v4f v = *reinterpret_cast<const v4f*>(fbuf + r * 128 + ((f_c ^ ((r >> 1) & 7)) << 4));
                    if (m < p.M && col < p.N) *reinterpret_cast<v4f*>(dst + static_cast<int64_t>(m) * p.N + col) = v;
                }
            }
        lds_barrier();
        if constexpr (PART) continue;
    }

    float mean_r[MI], rstd_r[MI];
    const bool ln = p.norm == LOKA_NORM_LAYERNORM;
    // FP8 output with gamma / beta: the row amax is only known after the affine step, and crosses the workgroups in
    // a second exchange (below); the row extremes of the pre-norm values are then of no use
    constexpr bool affine_q = F8 == 2;
    float iq_r[MI];
    if (p.norm == LOKA_NORM_NONE) {
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) { mean_r[mi] = 0.f; rstd_r[mi] = 1.f; iq_r[mi] = 1.f; }
    } else {
        // In every wave per row: mean and centred squares of its 64 columns (LayerNorm) or the sum of squares.  Without branches and
        // LDS exchanges: columns past N hold zeros, which add nothing to the sums (their centred value is taken as
        // zero), and the two lanes of a row add up by half swaps.  The counts of the waves' columns add up to the tile's,
        // so the tile's mean is the plain sum of n_w mean_w over n, its centred squares that of m2_w + n_w (mean_w - mean)^2.
        // (M x N x K, us, with branches, shuffles and pairwise merges before: 16384 x 3072 x 1024 100.1 -> 98.3, 8192 x 2048 x 2048
        // 36.0 -> 35.7, 65536 x 256 x 512 20.5 -> 20.2, 32768 x 4096 x 4096 477 -> 474)
        const int n_tile = n_o - n0 < BN ? n_o - n0 : BN;
        auto cols_of = [&](int w) __attribute__((always_inline)) {
            const int c = n_tile - w * WN;
            return static_cast<float>(c < 0 ? 0 : c < WN ? c : WN);
        };
        const float n_wave = cols_of(wave_n), rn_wave = n_wave > 0.f ? __builtin_amdgcn_rcpf(n_wave) : 0.f;
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) {
            float mean = 0.f, q[4] = {0.f, 0.f, 0.f, 0.f};
            if (ln) {
                float t[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                    for (int i = 0; i < 16; ++i) t[i & 3] += acc[mi][ni][i];
                mean = half_lanes_sum((t[0] + t[1]) + (t[2] + t[3])) * rn_wave;
#pragma unroll
                for (int ni = 0; ni < NI; ++ni) {
                    const float mean_in = ncol[ni] < n_o ? mean : 0.f;
#pragma unroll
                    for (int i = 0; i < 16; ++i) { const float d = acc[mi][ni][i] - mean_in; q[i & 3] = __builtin_fmaf(d, d, q[i & 3]); }
                }
            } else {
#pragma unroll
                for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                    for (int i = 0; i < 16; ++i) q[i & 3] = __builtin_fmaf(acc[mi][ni][i], acc[mi][ni][i], q[i & 3]);
            }
            const float m2 = half_lanes_sum((q[0] + q[1]) + (q[2] + q[3]));
            if (hk == 0) red[wave_n * BM + wave_m * WM + mi * 32 + l32] = make_float2(mean, m2);
            if (FP8OUT && !affine_q) {
                float lo = __builtin_inff(), hi = -__builtin_inff();
#pragma unroll
                for (int ni = 0; ni < NI; ++ni)
                    if (ncol[ni] < p.N) {
#pragma unroll
                        for (int i = 0; i < 16; ++i) {
                            lo = __builtin_fminf(lo, acc[mi][ni][i]);
                            hi = __builtin_fmaxf(hi, acc[mi][ni][i]);
                        }
                    }
                lo = -half_lanes_max(-lo);
                hi = half_lanes_max(hi);
                if (hk == 0) {
                    float* r2 = red2 + ((wave_m * WM + mi * 32 + l32) * 4 + wave_n) * 2;
                    r2[0] = lo; r2[1] = hi;
                }
            }
        }
        __syncthreads();
        // tile statistics per row: thread r < 256 folds the four column waves in order
        float t_mean = 0.f, t_m2 = 0.f, t_lo = __builtin_inff(), t_hi = -__builtin_inff();
        if (tid < BM) {
            float2 part[4];
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                part[w] = red[w * BM + tid];
                t_mean = __builtin_fmaf(cols_of(w), part[w].x, t_mean);
            }
            t_mean *= __builtin_amdgcn_rcpf(static_cast<float>(n_tile));
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const float d = part[w].x - t_mean;
                t_m2 += __builtin_fmaf(cols_of(w) * d, d, part[w].y);
                if (FP8OUT && !affine_q) {
                    t_lo = __builtin_fminf(t_lo, red2[(tid * 4 + w) * 2]);
                    t_hi = __builtin_fmaxf(t_hi, red2[(tid * 4 + w) * 2 + 1]);
                }
            }
        }
        // FP8OUT: the row scale from the row's extreme pre-norm values, through the very operations the
        // normalization applies to every element (one fused multiply-add, bf16 rounding)
        auto row_scale = [&](int r, float mean, float rstd, float lo, float hi) __attribute__((always_inline)) {
            const float nmr = -mean * rstd;
            const unsigned pk = pack_bf16x2(__builtin_fmaf(lo, rstd, nmr), __builtin_fmaf(hi, rstd, nmr));
            const unsigned a = pk & 0x7FFFu, b = (pk >> 16) & 0x7FFFu;
            float scale, inv;
            group_scale(__uint_as_float((a > b ? a : b) << 16), scale, inv);
            if (!(rstd == rstd)) scale = rstd;                    // poisoned row: the scale says so
            finq[r] = inv;
            if (tn == 0 && m0 + r < p.M) p.outs[static_cast<int64_t>(g) * p.M + m0 + r] = scale;
        };
        const bool blocknorm = p.norm == LOKA_NORM_BLOCKNORM;   // groups of 256 columns = this tile: nothing to exchange
        bool arrived = true;                                    // false: a wait for the panel's other tiles ran out
        int* const lds_word = reinterpret_cast<int*>(smem + 16000);   // (free between finq and red2)
        if (EPI == EPI_PANEL_SYNC && !blocknorm && p.tiles_n > 1) {
            // publish (mean, M2) of this tile per row, signal, wait for the panel's other tiles, merge all tiles
            const int panel = g * p.tiles_m + tm;
            // Exchange area of a panel: [tiles_n][256 rows] records of 8 bytes, so that a tile's 256 threads write
            // one contiguous 2 KB run and the merging threads of consecutive rows read consecutive records (a
            // row-major [row][tile] layout makes every lane of a load touch a cache line of its own, and the 256
            // workgroups' merges then queue at the L2 channels).  (min, max) per row and tile: a second array of the
            // same shape behind the statistics of all panels.
            unsigned long long* pbase = reinterpret_cast<unsigned long long*>(p.part) + static_cast<int64_t>(panel) * p.tiles_n * BM;
            const int64_t mm_off = static_cast<int64_t>(p.batch) * p.tiles_m * p.tiles_n * BM;
            if (tid < BM) {
                unsigned long long* dst = pbase + tn * BM + tid;
                __hip_atomic_store(dst, static_cast<unsigned long long>(__float_as_uint(t_mean)) |
                                            (static_cast<unsigned long long>(__float_as_uint(t_m2)) << 32),
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (FP8OUT && !affine_q)
                    __hip_atomic_store(dst + mm_off, static_cast<unsigned long long>(__float_as_uint(t_lo)) |
                                                         (static_cast<unsigned long long>(__float_as_uint(t_hi)) << 32),
                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            arrived = panel_publish_and_wait(p, p.flags + static_cast<int64_t>(panel) * p.tiles_n, tn, p.tiles_n, lds_word, wave == 0);
            // two threads per row, each folds a contiguous half of the row's tiles in order (device-coherent
            // 8-byte loads), symmetric merge of the halves: identical bits in every workgroup of the panel
            {
                const int r = static_cast<int>(tid) >> 1, sub = static_cast<int>(tid) & 1;
                const unsigned long long* src = pbase + r;
                const int TH = (p.tiles_n + 1) >> 1;
                float n_ = 0.f, mean = 0.f, m2 = 0.f, lo = __builtin_inff(), hi = -__builtin_inff();
                for (int t0 = sub * TH; t0 < (sub + 1) * TH && t0 < p.tiles_n; t0 += 8) {
                    unsigned long long raw[8], raw2[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        int tt = t0 + u;
                        tt = tt < p.tiles_n ? tt : p.tiles_n - 1;
                        raw[u] = __hip_atomic_load(src + tt * BM, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        if (FP8OUT && !affine_q) raw2[u] = __hip_atomic_load(src + mm_off + tt * BM, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    }
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const int tt = t0 + u;
                        if (tt < (sub + 1) * TH && tt < p.tiles_n) {
                            const float a = __uint_as_float(static_cast<unsigned>(raw[u]));
                            const float b2 = __uint_as_float(static_cast<unsigned>(raw[u] >> 32));
                            const int wcols = (tt + 1) * BN <= p.N ? BN : p.N - tt * BN;
                            if (ln) merge_stats(n_, mean, m2, static_cast<float>(wcols), a, b2);
                            else m2 += b2;
                            if (FP8OUT && !affine_q) {
                                lo = __builtin_fminf(lo, __uint_as_float(static_cast<unsigned>(raw2[u])));
                                hi = __builtin_fmaxf(hi, __uint_as_float(static_cast<unsigned>(raw2[u] >> 32)));
                            }
                        }
                    }
                }
                // (the other thread's, by a move within the quad)
                auto other = [](float v) __attribute__((always_inline)) {
                    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xF, 0xF, true));
                };
                const float nb = other(n_), mb = other(mean), m2b = other(m2);
                if (ln) {
                    const float nn = n_ + nb;
                    if (nn > 0.f) {
                        const float d = mb - mean;
                        const float rn = __builtin_amdgcn_rcpf(nn);
                        const float newmean = (n_ * mean + nb * mb) * rn;
                        m2 = m2 + m2b + d * d * (n_ * nb * rn);
                        mean = newmean;
                    }
                } else {
                    m2 = m2 + m2b;
                }
                if (FP8OUT && !affine_q) {
                    lo = __builtin_fminf(lo, other(lo));
                    hi = __builtin_fmaxf(hi, other(hi));
                }
                if (sub == 0) {
                    // (a wait that ran out: the statistics are not to be trusted; the tile's rows leave as NaN, their
                    // FP8 row scale as NaN)
                    const float2 f = arrived ? make_float2(ln ? mean : 0.f, __builtin_amdgcn_rsqf(m2 * inv_n + p.eps))
                                             : make_float2(__builtin_nanf(""), __builtin_nanf(""));
                    fin[r] = f;
                    if (FP8OUT && !affine_q) row_scale(r, f.x, f.y, lo, hi);
                }
            }
        } else {
            // the tile spans the whole row (N <= 256): finalize here
            if (tid < BM) {
                const float2 f = make_float2(ln ? t_mean : 0.f, __builtin_amdgcn_rsqf(t_m2 * (blocknorm ? 1.0f / BN : inv_n) + p.eps));
                fin[tid] = f;
                if (FP8OUT && !affine_q) row_scale(static_cast<int>(tid), f.x, f.y, t_lo, t_hi);
            }
        }
        __syncthreads();
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) {
            const float2 f = fin[wave_m * WM + mi * 32 + l32];
            mean_r[mi] = f.x;
            rstd_r[mi] = f.y;
            if (FP8OUT && !affine_q) iq_r[mi] = finq[wave_m * WM + mi * 32 + l32];
        }
    }
    float nmr_r[MI];
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) nmr_r[mi] = -mean_r[mi] * rstd_r[mi];

    // ---- normalize, affine, bf16 store.  A lane holds 16 consecutive columns of ONE row per 32 x 32 sub-tile;
    // stored from there, an instruction would touch 32 rows with 32 bytes each.  Each wave instead passes the
    // sub-tile through 2 KB of its own LDS (64-byte rows, 16-byte chunk c of row r at position c ^ (r / 4 % 4):
    // conflict-free both ways) and stores it with 4 lanes per row: 16 full 64-byte runs per instruction.
    // LDS executes one wave's instructions in order, so the same buffer serves every sub-tile without a barrier.
    const bool has_g = p.gamma != nullptr && (ln || p.norm == LOKA_NORM_RMSNORM), has_b = p.beta != nullptr && ln;
    const bool hswish = p.act == LOKA_ACT_HARDSWISH;
    // gamma and beta of this lane's 16 columns of sub-tile ni (1 and 0 where absent or past N)
    auto load_affine = [&](int ni, float (&gm)[16], float (&bt)[16]) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < 16; ++e) { gm[e] = 1.f; bt[e] = 0.f; }
        if (ncol[ni] >= p.N) return;
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            if (has_g) {
                const u32x4 w = *reinterpret_cast<const u32x4*>(p.gamma + ncol[ni] + 8 * half);
                float* q = gm + 8 * half;
                q[0] = bf16_lo(w.x); q[1] = bf16_hi(w.x); q[2] = bf16_lo(w.y); q[3] = bf16_hi(w.y);
                q[4] = bf16_lo(w.z); q[5] = bf16_hi(w.z); q[6] = bf16_lo(w.w); q[7] = bf16_hi(w.w);
            }
            if (has_b) {
                const u32x4 w = *reinterpret_cast<const u32x4*>(p.beta + ncol[ni] + 8 * half);
                float* q = bt + 8 * half;
                q[0] = bf16_lo(w.x); q[1] = bf16_hi(w.x); q[2] = bf16_lo(w.y); q[3] = bf16_hi(w.y);
                q[4] = bf16_lo(w.z); q[5] = bf16_hi(w.z); q[6] = bf16_lo(w.w); q[7] = bf16_hi(w.w);
            }
        }
    };
    uint8_t* const tbuf = smem + 16384 + wave * 2048;
    const int t_wr = l32 * 64, t_key = (l32 >> 2) & 3;
    const int t_row = lane >> 2, t_c = lane & 3;                       // store side: row (+ 16 j), chunk
    if (FP8OUT) {
        (void)hswish;
        // With gamma / beta: the normalized bf16 values replace the accumulators (64 packed registers), their row
        // amax crosses the waves through LDS and the workgroups through a second exchange (records in the area the
        // row extremes use otherwise, a second arrival counter per panel), and the cast follows.
        unsigned opk[MI][NI][4][2];
        if (affine_q) {
            unsigned am[MI];
#pragma unroll
            for (int mi = 0; mi < MI; ++mi) am[mi] = 0u;
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) {
                float gm[16], bt[16];
                load_affine(ni, gm, bt);
#pragma unroll
                for (int mi = 0; mi < MI; ++mi)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        float o[4];
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            o[e] = __builtin_fmaf(acc[mi][ni][4 * q + e], rstd_r[mi], nmr_r[mi]);
                            if (has_g || has_b) o[e] = __builtin_fmaf(o[e], gm[4 * q + e], bt[4 * q + e]);
                            if (hswish) o[e] = o[e] * __builtin_fminf(__builtin_fmaxf(o[e] + 3.0f, 0.0f), 6.0f) * (1.0f / 6.0f);
                        }
                        const unsigned p0 = pack_bf16x2(o[0], o[1]), p1 = pack_bf16x2(o[2], o[3]);
                        opk[mi][ni][q][0] = p0; opk[mi][ni][q][1] = p1;
                        if (ncol[ni] < p.N) {
                            const unsigned a0 = p0 & 0x7FFFu, a1 = (p0 >> 16) & 0x7FFFu, a2 = p1 & 0x7FFFu, a3 = (p1 >> 16) & 0x7FFFu;
                            const unsigned a01 = a0 > a1 ? a0 : a1, a23 = a2 > a3 ? a2 : a3;
                            const unsigned a = a01 > a23 ? a01 : a23;
                            am[mi] = am[mi] > a ? am[mi] : a;
                        }
                    }
            }
            unsigned* amw = reinterpret_cast<unsigned*>(smem + 16384);        // [BM][4]: row amax per column wave
#pragma unroll
            for (int mi = 0; mi < MI; ++mi) {
                const unsigned other = static_cast<unsigned>(__shfl_xor(static_cast<int>(am[mi]), 32, 64));
                am[mi] = am[mi] > other ? am[mi] : other;
                if (hk == 0) amw[(wave_m * WM + mi * 32 + l32) * 4 + wave_n] = am[mi];
            }
            __syncthreads();
            unsigned t_am = 0u;
            if (tid < BM) {
#pragma unroll
                for (int w = 0; w < 4; ++w) { const unsigned a = amw[tid * 4 + w]; t_am = t_am > a ? t_am : a; }
            }
            bool amax_ok = true;
            auto row_scale_am = [&](int r, unsigned a) __attribute__((always_inline)) {
                float scale, inv;
                group_scale(__uint_as_float(a << 16), scale, inv);
                if (!amax_ok) scale = __builtin_nanf("");           // the wait for the other tiles' amax ran out
                finq[r] = inv;
                if (tn == 0 && m0 + r < p.M) p.outs[static_cast<int64_t>(g) * p.M + m0 + r] = scale;
            };
            if (p.tiles_n > 1) {
                const int panel = g * p.tiles_m + tm;
                const int64_t mm_off = static_cast<int64_t>(p.batch) * p.tiles_m * p.tiles_n * BM;
                unsigned long long* pam = reinterpret_cast<unsigned long long*>(p.part) + mm_off +
                                          static_cast<int64_t>(panel) * p.tiles_n * BM;
                if (tid < BM) {
                    __hip_atomic_store(pam + tn * BM + tid, static_cast<unsigned long long>(t_am), __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
                }
                // (the second set of arrival words of the panel)
                const bool arrived2 = panel_publish_and_wait(
                    p, p.flags + (static_cast<int64_t>(p.batch) * p.tiles_m + panel) * p.tiles_n, tn, p.tiles_n,
                    reinterpret_cast<int*>(smem + 16000), wave == 0);
                amax_ok = arrived2;
                {
                    const int r = static_cast<int>(tid) >> 1, sub = static_cast<int>(tid) & 1;
                    const int TH = (p.tiles_n + 1) >> 1;
                    unsigned a = 0u;
                    for (int t0 = sub * TH; t0 < (sub + 1) * TH && t0 < p.tiles_n; t0 += 8) {
                        unsigned long long raw[8];
#pragma unroll
                        for (int u = 0; u < 8; ++u) {
                            int tt = t0 + u;
                            tt = tt < p.tiles_n ? tt : p.tiles_n - 1;
                            raw[u] = __hip_atomic_load(pam + tt * BM + r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        }
#pragma unroll
                        for (int u = 0; u < 8; ++u) {
                            const unsigned v = static_cast<unsigned>(raw[u]);      // (a clamped index repeats a tile: harmless for a maximum)
                            a = a > v ? a : v;
                        }
                    }
                    const unsigned other = static_cast<unsigned>(__shfl_xor(static_cast<int>(a), 1, 64));
                    a = a > other ? a : other;
                    if (sub == 0) row_scale_am(r, a);
                }
            } else if (tid < BM) {
                row_scale_am(static_cast<int>(tid), t_am);
            }
            __syncthreads();
#pragma unroll
            for (int mi = 0; mi < MI; ++mi) iq_r[mi] = finq[wave_m * WM + mi * 32 + l32];
            __syncthreads();                  // amw (aliasing the transpose buffers) and finq are read
        }
        // 16 codes per lane and sub-tile; the wave's 64 columns of 32 rows pass through the transpose buffer at once
        // (64-byte rows of codes) and leave as full 64-byte runs, 4 lanes per row
        const int col = n0 + wave_n * WN + t_c * 16;
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) {
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) {
                unsigned ck[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    unsigned p0, p1;
                    if (affine_q) {
                        p0 = opk[mi][ni][q][0]; p1 = opk[mi][ni][q][1];
                    } else {
                        float o[4];
#pragma unroll
                        for (int e = 0; e < 4; ++e) o[e] = __builtin_fmaf(acc[mi][ni][4 * q + e], rstd_r[mi], nmr_r[mi]);
                        p0 = pack_bf16x2(o[0], o[1]); p1 = pack_bf16x2(o[2], o[3]);
                    }
                    ck[q] = e4m3x4(bf16_lo(p0) * iq_r[mi], bf16_hi(p0) * iq_r[mi], bf16_lo(p1) * iq_r[mi], bf16_hi(p1) * iq_r[mi]);
                }
                *reinterpret_cast<u32x4*>(tbuf + t_wr + (((2 * ni + hk) ^ t_key) << 4)) = u32x4{ck[0], ck[1], ck[2], ck[3]};
            }
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int r = 16 * j + t_row;
                const u32x4 ck = *reinterpret_cast<const u32x4*>(tbuf + r * 64 + ((t_c ^ ((r >> 2) & 3)) << 4));
                const int m = m0 + wave_m * WM + mi * 32 + r;
                if (m < p.M && col < p.N)
                    __builtin_nontemporal_store(ck, reinterpret_cast<u32x4*>(p.outq + obase + static_cast<int64_t>(m) * p.N + col));
            }
        }
    } else {
#pragma unroll
    for (int ni = 0; ni < NI; ++ni) {
        float gm[16], bt[16];
        load_affine(ni, gm, bt);
        const int col = n0 + wave_n * WN + ni * 32 + t_c * 8;         // store side: this lane's 8 columns
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) {
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                float o[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    // (y - mean) * rstd as one fused multiply-add, the affine part as another
                    o[e] = __builtin_fmaf(acc[mi][ni][8 * half + e], rstd_r[mi], nmr_r[mi]);
                    if (has_g || has_b) o[e] = __builtin_fmaf(o[e], gm[8 * half + e], bt[8 * half + e]);
                    if (hswish) o[e] = o[e] * __builtin_fminf(__builtin_fmaxf(o[e] + 3.0f, 0.0f), 6.0f) * (1.0f / 6.0f);
                }
                u32x4 pk;
                pk.x = pack_bf16x2(o[0], o[1]); pk.y = pack_bf16x2(o[2], o[3]);
                pk.z = pack_bf16x2(o[4], o[5]); pk.w = pack_bf16x2(o[6], o[7]);
                *reinterpret_cast<u32x4*>(tbuf + t_wr + (((2 * hk + half) ^ t_key) << 4)) = pk;
            }
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int r = 16 * j + t_row;
                const u32x4 pk = *reinterpret_cast<const u32x4*>(tbuf + r * 64 + ((t_c ^ ((r >> 2) & 3)) << 4));
                const int m = m0 + wave_m * WM + mi * 32 + r;
                if (m < p.M && col < p.N)
                    __builtin_nontemporal_store(pk, reinterpret_cast<u32x4*>(p.out + obase + static_cast<int64_t>(m) * p.N + col));
            }
        }
    }
    }
    }
    lds_barrier();              // the epilogue's scratch (slot 0) is read: the next tile may load into it.  The
                                // stores stay in flight.
  }
}

constexpr size_t kPanel32Lds = 5 * 256 * 128;   // the ring; the epilogue's scratch aliases it

// The normalized value is not a growing function of the pre-norm value along the row: gamma / beta take part (the
// kernel ignores gamma outside LayerNorm / RMSNorm and beta outside LayerNorm), or the row is normalized group by
// group (BlockNorm), or an activation follows.  The FP8-output launch then takes the form with the second exchange.
bool panel32_affine(const GemmParams& p) {
    const bool ln = p.norm == LOKA_NORM_LAYERNORM;
    return (p.gamma != nullptr && (ln || p.norm == LOKA_NORM_RMSNORM)) || (p.beta != nullptr && ln) ||
           p.norm == LOKA_NORM_BLOCKNORM || p.act != LOKA_ACT_NONE;
}
// X's block scales four K blocks at a time: a row's scales are whole 16-byte runs, and so are a K range's
bool panel32_quad(int KB, int k_per_split) { return KB % 512 == 0 && k_per_split % 4 == 0; }
namespace {
using Panel32Fn = void (*)(GemmParams);
template <int EPI, bool YOUT>
Panel32Fn panel32_block_fn(int bw, bool quad) {
    return bw == 2 ? (quad ? &gemm_panel32_kernel<EPI, 2, 0, false, false, false, YOUT, true> : &gemm_panel32_kernel<EPI, 2, 0, false, false, false, YOUT, false>)
                   : (quad ? &gemm_panel32_kernel<EPI, 1, 0, false, false, false, YOUT, true> : &gemm_panel32_kernel<EPI, 1, 0, false, false, false, YOUT, false>);
}
// bw: 0 plain scales, 1 block scales, 2 power-of-two block scales (see the kernel); fp8out with bw == 0 only
Panel32Fn panel32_pick(int bw, bool fp8out, bool affine, bool qpro, bool want_y, bool quad) {
    if (qpro) return (bw != 0 || fp8out) ? nullptr : &gemm_panel32_kernel<EPI_PANEL_SYNC, 0, 0, true>;
    if (fp8out) return bw != 0 ? nullptr : affine ? &gemm_panel32_kernel<EPI_PANEL_SYNC, 0, 2> : &gemm_panel32_kernel<EPI_PANEL_SYNC, 0, 1>;
    if (bw) return want_y ? panel32_block_fn<EPI_PANEL_SYNC, true>(bw, quad) : panel32_block_fn<EPI_PANEL_SYNC, false>(bw, quad);
    return want_y ? &gemm_panel32_kernel<EPI_PANEL_SYNC, 0, 0> : &gemm_panel32_kernel<EPI_PANEL_SYNC, 0, 0, false, false, false, false>;
}
// split K and the BF16 reference GEMM: fp32 out
Panel32Fn panel32_part_pick(int bw, bool bf16, bool quad) {
    return bf16 ? &gemm_panel32_kernel<EPI_ROW_IN_TILE, 0, 0, false, true> : bw ? panel32_block_fn<EPI_SPLITK, true>(bw, quad) : &gemm_panel32_kernel<EPI_SPLITK, 0, 0>;
}
}  // namespace
const void* panel32_fn(int bw, bool fp8out, bool affine, bool qpro, bool want_y, bool quad) {
    return reinterpret_cast<const void*>(panel32_pick(bw, fp8out, affine, qpro, want_y, quad));
}
// a K that is no multiple of 128 (plain scales, bf16 output)
const void* panel32_ragged_fn() { return reinterpret_cast<const void*>(&gemm_panel32_kernel<EPI_PANEL_SYNC, 0, 0, false, false, true>); }
void panel32_ragged_launch(const GemmParams& p, dim3 grid, hipStream_t s) {
    gemm_panel32_kernel<EPI_PANEL_SYNC, 0, 0, false, false, true><<<grid, 512, kPanel32Lds, s>>>(p);
}
const void* panel32_part_fn(int bw, bool bf16, bool quad) { return reinterpret_cast<const void*>(panel32_part_pick(bw, bf16, quad)); }
void panel32_part_launch(const GemmParams& p, int bw, bool bf16, dim3 grid, hipStream_t s) {
    panel32_part_pick(bw, bf16, panel32_quad(p.KB, p.k_per_split))<<<grid, 512, kPanel32Lds, s>>>(p);
}
size_t panel32_lds() { return kPanel32Lds; }
void panel32_launch(const GemmParams& p, int bw, dim3 grid, hipStream_t s) {
    panel32_pick(bw, p.outq != nullptr, panel32_affine(p), p.qpro != 0, p.y != nullptr, panel32_quad(p.KB, 0))<<<grid, 512, kPanel32Lds, s>>>(p);
}

}  // namespace loka
