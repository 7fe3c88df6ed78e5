// amax -> scale -> OCP e4m3 cast of bf16 matrices (bandwidth-bound streaming kernels).
//
// ROW and BLOCK_1x128 scaling are single-pass: the lanes that share a scale group
// keep their elements in registers between the amax reduction and the cast, so the
// matrix is read once (2 B/elem) and the codes written once (1 B/elem).
// The modes whose groups fit a 128 x 128 tile are single-pass as well (quant_tile128_kernel).
// TENSOR and COL scaling need every row of a group before the first cast: an amax pass that
// leaves partial maxima in the workspace, and the tile kernel, whose workgroups fold the
// partials of their columns, take scale = amax/448 and inv = 448/amax (one division each),
// cast, and write plain or transposed (the layout used for weights).
#include "common.h"

#include <type_traits>

namespace loka {

__device__ __forceinline__ float chunk_amax(const u32x4 w) {
    float a = fmaxf(fabsf(bf16_lo(w.x)), fabsf(bf16_hi(w.x)));
    a = fmaxf(a, fmaxf(fabsf(bf16_lo(w.y)), fabsf(bf16_hi(w.y))));
    a = fmaxf(a, fmaxf(fabsf(bf16_lo(w.z)), fabsf(bf16_hi(w.z))));
    return fmaxf(a, fmaxf(fabsf(bf16_lo(w.w)), fabsf(bf16_hi(w.w))));
}

// one chunk of 8 elements, past the caches or through them
template <bool STREAMED>
__device__ __forceinline__ u32x4 load_chunk(const uint16_t* p) {
    const u32x4* v = reinterpret_cast<const u32x4*>(p);
    if (STREAMED) return __builtin_nontemporal_load(v);
    return *v;
}

// Maximum over groups of GL consecutive lanes (16, 32 or 64), in all of them: moves within 16 lanes, row and half swaps.
// (lanes_max_bits is the same on the bits of magnitudes: there a NaN is the largest value, here fmaxf leaves it out.)
template <int GL>
__device__ __forceinline__ float lanes_max(float a) {
    auto moved = [&](auto ctrl) __attribute__((always_inline)) {
        return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(a), decltype(ctrl)::value, 0xF, 0xF, true));
    };
    a = fmaxf(a, moved(std::integral_constant<int, 0xB1>{}));       // lane ^ 1
    a = fmaxf(a, moved(std::integral_constant<int, 0x4E>{}));       // lane ^ 2
    a = fmaxf(a, moved(std::integral_constant<int, 0x141>{}));      // the other quad of 8
    a = fmaxf(a, moved(std::integral_constant<int, 0x140>{}));      // the other half of 16
    if (GL >= 32) {
        const u32_pair r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(a), false, false);
        a = fmaxf(__uint_as_float(r.x), __uint_as_float(r.y));
    }
    if (GL >= 64) {
        const u32_pair r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(a), false, false);
        a = fmaxf(__uint_as_float(r.x), __uint_as_float(r.y));
    }
    return a;
}

// ---------------------------------------------------------------------------------
// Single pass: TPR lanes share one row (TPR = 16, 32 or 64); each lane holds CPL
// chunks of 8 consecutive bf16 (one 16-byte load each); a wave works on RU row sets at
// once so that enough loads are in flight.  Lanes per scale group: TPR for ROW
// scaling (one group per row), 16 for 1x128 blocks (16 lanes x 8 elements).
// Bound by HBM, and where all of it is one round of workgroups by what a wave does between its loads and its stores (rows x
// columns, exchanges by LDS shuffles and divisions in every lane -> as here, us, streamed loads: 65536 x 256 11.5 -> 10.6,
// 16384 x 1024 11.6 -> 10.4; in 1 x 128 blocks 8192 x 2048 12.1 -> 10.6, 65536 x 512 20.5 -> 18.8, 2048 x 8192 16.4 -> 14.4).
template <int TPR, int CPL, int RU, bool BLOCK128>
__global__ __launch_bounds__(256) void quant_rows_kernel(const uint16_t* __restrict__ x, int64_t rows, int64_t cols,
                                                         int64_t ld, uint8_t* __restrict__ q,
                                                         float* __restrict__ scales, const int pow2, const bool streamed) {
    constexpr int ROWS_PER_WAVE = (64 / TPR) * RU;
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int lr = lane % TPR;               // lane within its row
    const int sub = lane / TPR;              // which of the wave's concurrent rows
    const int64_t chunks = cols >> 3;        // 8-element chunks per row
    const int64_t row0 = (static_cast<int64_t>(blockIdx.x) * 4 + wave) * ROWS_PER_WAVE;

    u32x4 v[RU][CPL];
    auto load = [&](auto streamed_c) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < RU; ++u) {
            const int64_t r = row0 + u * (64 / TPR) + sub;
#pragma unroll
            for (int j = 0; j < CPL; ++j) {
                const int64_t c = lr + static_cast<int64_t>(j) * TPR;
                v[u][j] = u32x4{0u, 0u, 0u, 0u};
                if (r < rows && c < chunks) v[u][j] = load_chunk<decltype(streamed_c)::value>(x + r * ld + c * 8);
            }
        }
    };
    // (each kind of read ends in a line of its own: the compiler merges the ends of the two branches otherwise, and a lane's last
    // load, an eighth to a quarter of what is to be streamed, went through the caches: training step 57472 x 896 x 1664, M x K x N, 522 -> 540 us)
    if (streamed) { load(std::true_type{}); asm volatile("; streamed"); }
    else { load(std::false_type{}); asm volatile("; through the caches"); }
    // The groups of a 16-lane row: T.  Every lane has the maxima of all of them after the exchanges (in the vector unit, no LDS
    // round trips); lane k takes group k's two divisions, and the factors go round by broadcasts: the divisions of all
    // groups in every lane were a third of the 1 x 128 form's instructions.
    constexpr int T = BLOCK128 ? RU * CPL : RU;
    float am[T];
#pragma unroll
    for (int u = 0; u < RU; ++u) {
        if (!BLOCK128) am[u] = chunk_amax(v[u][0]);
#pragma unroll
        for (int j = BLOCK128 ? 0 : 1; j < CPL; ++j) {
            if (BLOCK128) am[u * CPL + j] = chunk_amax(v[u][j]);
            else am[u] = fmaxf(am[u], chunk_amax(v[u][j]));
        }
    }
#pragma unroll
    for (int k = 0; k < T; ++k) am[k] = lanes_max<BLOCK128 ? 16 : TPR>(am[k]);
    const int k16 = lane & 15;
    float mine = am[0], scale, inv_mine;
#pragma unroll
    for (int k = 1; k < T; ++k) mine = k16 == k ? am[k] : mine;
    group_scale_any(BLOCK128 && pow2, mine, scale, inv_mine);
    if (BLOCK128) {
        const int u = k16 / CPL, j = k16 % CPL;
        const int64_t r = row0 + u * (64 / TPR) + sub, c = (lr & ~15) + static_cast<int64_t>(j) * TPR;
        if (k16 < T && r < rows && c < chunks) scales[r * (cols >> 7) + (c >> 4)] = scale;
    } else {
        const int64_t r = row0 + k16 * (64 / TPR) + sub;
        if (lr < T && r < rows) scales[r] = scale;
    }
    float inv[T];
    row_broadcasts<T>(inv_mine, inv);
#pragma unroll
    for (int u = 0; u < RU; ++u) {
        const int64_t r = row0 + u * (64 / TPR) + sub;
#pragma unroll
        for (int j = 0; j < CPL; ++j) {
            const int64_t c = lr + static_cast<int64_t>(j) * TPR;
            if (r < rows && c < chunks) {
                const u32x4 w = v[u][j];
                const float f = inv[BLOCK128 ? u * CPL + j : u];
                u32x2 o;
                o.x = e4m3x4(bf16_lo(w.x) * f, bf16_hi(w.x) * f, bf16_lo(w.y) * f, bf16_hi(w.y) * f);
                o.y = e4m3x4(bf16_lo(w.z) * f, bf16_hi(w.z) * f, bf16_lo(w.w) * f, bf16_hi(w.w) * f);
                // plain store: the GEMM that follows reads the codes from the last-level cache (measured at
                // 32768 x 4096: the GEMM runs 3 % faster than after a streaming store, this kernel no slower)
                *reinterpret_cast<u32x2*>(q + r * cols + c * 8) = o;
            }
        }
    }
}

// Rows too long for one wave (8192 < cols <= 131072): a workgroup of 16 waves holds the whole row in registers (CPL chunks
// of 8 elements per thread, 64 registers at 131072 columns: 256 KB of a CU's register file) between the amax and the
// cast, so the row is read once.  The workgroups are persistent: the register a chunk leaves at its cast takes the same
// chunk of the workgroup's next row, so the next row streams in while this one is cast and stored, and the memory never
// idles between a CU's rows.  Bound by HBM (3 B per element).  2048 x 123200: 230 us with two sweeps over the row (the
// second one misses: the rows in flight are larger than the last-level cache) -> 125 us = 6.06 TB/s; 8192 x 32768 208 -> 126,
// 2048 x 24576 37 -> 27.
template <int CPL>
__global__ __launch_bounds__(1024) void quant_wide_rows_kernel(const uint16_t* __restrict__ x, int64_t rows, int64_t cols,
                                                               int64_t ld, uint8_t* __restrict__ q, float* __restrict__ scales) {
    __shared__ float red[2][16];           // (two sets: a row's maxima are written while slow waves still read the last row's)
    const int t = static_cast<int>(threadIdx.x);
    u32x4 v[CPL];
    // buffer accesses relative to the row: one 32-bit offset per thread, chunks past the end of the row read as zeros and
    // are not stored (64-bit addresses per chunk would not fit beside the row: 114 registers spilled at CPL = 16)
    auto row_rsrc = [&](int64_t r) __attribute__((always_inline)) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(x + (r < rows ? r : 0) * ld), 0,
                                                 r < rows ? static_cast<int>(cols) * 2 : 0, 0x00020000);
    };
    auto load = [&](const __amdgpu_buffer_rsrc_t& rs, int j) __attribute__((always_inline)) {
        v[j] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, t * 16, j * 16384, 2));   // (2: streamed)
    };
    int64_t r = blockIdx.x;
    {
        const __amdgpu_buffer_rsrc_t rs = row_rsrc(r);
#pragma unroll
        for (int j = 0; j < CPL; ++j) load(rs, j);
    }
    for (int it = 0; r < rows; it ^= 1) {
        float a = chunk_amax(v[0]);
#pragma unroll
        for (int j = 1; j < CPL; ++j) a = fmaxf(a, chunk_amax(v[j]));
        a = lanes_max<64>(a);
        if ((t & 63) == 0) red[it][t >> 6] = a;
        __syncthreads();
        a = lanes_max<16>(red[it][t & 15]);
        float scale, inv;
        group_scale(a, scale, inv);
        if (t == 0) scales[r] = scale;
        const __amdgpu_buffer_rsrc_t rs = row_rsrc(r + gridDim.x);
        const __amdgpu_buffer_rsrc_t qs = __builtin_amdgcn_make_buffer_rsrc(q + r * cols, 0, static_cast<int>(cols), 0x00020000);
#pragma unroll
        for (int j = 0; j < CPL; ++j) {
            u32x4 w = v[j];
            asm volatile("; row chunk" : "+v"(w));     // (opaque: the values widened for the amax are not kept for the cast)
            u32x2 o;
            o.x = e4m3x4(bf16_lo(w.x) * inv, bf16_hi(w.x) * inv, bf16_lo(w.y) * inv, bf16_hi(w.y) * inv);
            o.y = e4m3x4(bf16_lo(w.z) * inv, bf16_hi(w.z) * inv, bf16_lo(w.w) * inv, bf16_hi(w.w) * inv);
            __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(v2i, o), qs, t * 8, j * 8192, 0);
            load(rs, j);
            __builtin_amdgcn_sched_barrier(0);     // (a chunk's cast, its store, its reload: in this order no second row's registers)
        }
        r += gridDim.x;
    }
}

// Rows longer than the register-resident kernels cover: one workgroup per row, two
// sweeps over the row (one for 1x128 groups, which need no sweep of their own).
template <bool BLOCK128>
__global__ __launch_bounds__(256) void quant_long_rows_kernel(const uint16_t* __restrict__ x, int64_t rows,
                                                              int64_t cols, int64_t ld, uint8_t* __restrict__ q,
                                                              float* __restrict__ scales, const int pow2) {
    __shared__ float red[4];
    const int64_t r = blockIdx.x;
    const int64_t chunks = cols >> 3;
    const uint16_t* xr = x + r * ld;
    float inv_row = 0.f;
    if (!BLOCK128) {
        float a = 0.f;
        for (int64_t c = threadIdx.x; c < chunks; c += 256) {
            const u32x4 w = *reinterpret_cast<const u32x4*>(xr + c * 8);
            a = fmaxf(a, fmaxf(fabsf(bf16_lo(w.x)), fabsf(bf16_hi(w.x))));
            a = fmaxf(a, fmaxf(fabsf(bf16_lo(w.y)), fabsf(bf16_hi(w.y))));
            a = fmaxf(a, fmaxf(fabsf(bf16_lo(w.z)), fabsf(bf16_hi(w.z))));
            a = fmaxf(a, fmaxf(fabsf(bf16_lo(w.w)), fabsf(bf16_hi(w.w))));
        }
        for (int m = 1; m < 64; m <<= 1) a = fmaxf(a, wave_shfl_xor(a, m));
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = a;
        __syncthreads();
        a = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
        float scale;
        group_scale(a, scale, inv_row);
        if (threadIdx.x == 0) scales[r] = scale;
    }
    // chunks is a multiple of 16 for 1x128 blocks, so the 16 lanes of a group stay together
    for (int64_t c0 = 0; c0 < chunks; c0 += 256) {
        const int64_t c = c0 + threadIdx.x;
        const bool ok = c < chunks;
        u32x4 w = u32x4{0u, 0u, 0u, 0u};
        if (ok) w = *reinterpret_cast<const u32x4*>(xr + c * 8);
        float inv = inv_row;
        if (BLOCK128) {
            float a = fmaxf(fabsf(bf16_lo(w.x)), fabsf(bf16_hi(w.x)));
            a = fmaxf(a, fmaxf(fabsf(bf16_lo(w.y)), fabsf(bf16_hi(w.y))));
            a = fmaxf(a, fmaxf(fabsf(bf16_lo(w.z)), fabsf(bf16_hi(w.z))));
            a = fmaxf(a, fmaxf(fabsf(bf16_lo(w.w)), fabsf(bf16_hi(w.w))));
            a = lanes_max<16>(a);
            float scale;
            group_scale_any(pow2, a, scale, inv);
            if (ok && (c & 15) == 0) scales[r * (cols >> 7) + (c >> 4)] = scale;
        }
        if (ok) {
            u32x2 o;
            o.x = e4m3x4(bf16_lo(w.x) * inv, bf16_hi(w.x) * inv, bf16_lo(w.y) * inv, bf16_hi(w.y) * inv);
            o.y = e4m3x4(bf16_lo(w.z) * inv, bf16_hi(w.z) * inv, bf16_lo(w.w) * inv, bf16_hi(w.w) * inv);
            *reinterpret_cast<u32x2*>(q + r * cols + c * 8) = o;
        }
    }
}

// ---------------------------------------------------------------------------------
// TENSOR and COL, first pass: partial maxima, parts[part][group] (group = column, or the one group of TENSOR).  Plain
// stores of one value per workgroup (or column) instead of atomics: nothing has to be cleared first, and the pass that
// casts folds the few partials itself, so the two passes are the whole call (with a clearing kernel, atomics and a
// kernel for the scales in between it was four, and the atomics alone took 21 - 31 us at 256 x 1024).
constexpr int kMaxParts = 64;              // row ranges of a COL pass: what every tile of the cast folds per column
constexpr int kTensorParts = 1024;         // workgroups of a TENSOR pass

__global__ __launch_bounds__(256) void amax_tensor_kernel(const uint16_t* __restrict__ x, int64_t rows, int64_t cols,
                                                          int64_t ld, float* __restrict__ parts) {
    __shared__ float red[4];
    const int64_t chunks = cols >> 3, total = rows * chunks, step = static_cast<int64_t>(gridDim.x) * 256;
    const bool flat = ld == cols;          // (no division per chunk then)
    float a = 0.f;
    for (int64_t i0 = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; i0 < total; i0 += 4 * step) {
        u32x4 w[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t i = i0 + u * step;
            w[u] = u32x4{0u, 0u, 0u, 0u};
            if (i < total) {
                const int64_t r = flat ? 0 : i / chunks, c = flat ? i : i - r * chunks;
                w[u] = *reinterpret_cast<const u32x4*>(x + r * ld + c * 8);       // (plain: the cast reads it again)
            }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) a = fmaxf(a, chunk_amax(w[u]));
    }
    a = lanes_max<64>(a);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = a;
    __syncthreads();
    if (threadIdx.x == 0) parts[blockIdx.x] = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
}

// A workgroup takes 64 columns (128-byte runs) of one row range: 8 chunk columns x 32 rows at a time.
__global__ __launch_bounds__(256) void amax_col_kernel(const uint16_t* __restrict__ x, int64_t rows, int64_t cols,
                                                       int64_t ld, int64_t rows_per_part, float* __restrict__ parts) {
    __shared__ float red[4][64];
    const int cc = threadIdx.x & 7, rr = threadIdx.x >> 3, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t c = static_cast<int64_t>(blockIdx.x) * 64 + cc * 8;
    const int64_t r0 = static_cast<int64_t>(blockIdx.y) * rows_per_part;
    const int64_t r1 = r0 + rows_per_part < rows ? r0 + rows_per_part : rows;
    float a[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int64_t r = r0 + rr; r < r1; r += 128) {
        u32x4 w[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            w[u] = u32x4{0u, 0u, 0u, 0u};
            if (c < cols && r + 32 * u < r1) w[u] = *reinterpret_cast<const u32x4*>(x + (r + 32 * u) * ld + c);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            a[0] = fmaxf(a[0], fabsf(bf16_lo(w[u].x))); a[1] = fmaxf(a[1], fabsf(bf16_hi(w[u].x)));
            a[2] = fmaxf(a[2], fabsf(bf16_lo(w[u].y))); a[3] = fmaxf(a[3], fabsf(bf16_hi(w[u].y)));
            a[4] = fmaxf(a[4], fabsf(bf16_lo(w[u].z))); a[5] = fmaxf(a[5], fabsf(bf16_hi(w[u].z)));
            a[6] = fmaxf(a[6], fabsf(bf16_lo(w[u].w))); a[7] = fmaxf(a[7], fabsf(bf16_hi(w[u].w)));
        }
    }
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
        for (int m = 8; m < 64; m <<= 1) a[j] = fmaxf(a[j], wave_shfl_xor(a[j], m));
    if (lane < 8) {
#pragma unroll
        for (int j = 0; j < 8; ++j) red[wave][cc * 8 + j] = a[j];
    }
    __syncthreads();
    const int t = static_cast<int>(threadIdx.x);
    const int64_t col = static_cast<int64_t>(blockIdx.x) * 64 + t;
    if (t < 64 && col < cols)
        parts[static_cast<int64_t>(blockIdx.y) * cols + col] = fmaxf(fmaxf(red[0][t], red[1][t]), fmaxf(red[2][t], red[3][t]));
}

// A workgroup takes a 128 x 128 tile (8 rows x 8 columns per thread: 32 registers), finds the factors of its groups,
// scales, casts and stores - every element is read once and written once (3 bytes per element).
//   G_TILE:    the whole tile is one group (BLOCK_128x128 and its power-of-two form); scales [rows/128][cols/128]
//   G_COL128:  every column of the tile is a group (BLOCK_128x1); scales [cols][rows/128]
//   G_COL:     a group is a whole column (COL), G_TENSOR: the whole matrix: the workgroup folds the partial maxima of
//              its groups that the amax pass left (parts[nparts][groups]); the first row of tiles writes the scales
//   G_COL_ALL: COL with few rows: the workgroup reads the other tiles of its columns itself (a second read from L2 in
//              place of the amax pass, whose launch costs more than the reads)
//   TRANSPOSE: codes leave as [cols, rows] through an LDS tile (128-byte runs per output row)
// rows % 128 == 0 for G_TILE and G_COL128; rows % 16 == 0 with TRANSPOSE; any rows else.  cols % 16 == 0 (% 128 for G_TILE).
// Measured (us, whole call with the amax pass; before: clearing, atomics, scales and a cast through a byte-wise LDS tile,
// four kernels): COL transposed 1024 x 1024 7.4, 4096 x 4096 44.8 -> 19.3, 123200 x 1024 423 -> 129; TENSOR
// 16384 x 512 57 -> 10.4, 65536 x 1024 95 -> 58, 32768 x 4096 136 -> 120.
enum { G_TILE, G_COL128, G_COL_ALL, G_COL, G_TENSOR };
template <int GROUPS, bool TRANSPOSE>
__global__ __launch_bounds__(256) void quant_tile128_kernel(const uint16_t* __restrict__ x, int64_t rows, int64_t cols,
                                                            int64_t ld, uint8_t* __restrict__ q, float* __restrict__ scales,
                                                            const int pow2, const bool streamed, const float* __restrict__ parts,
                                                            const int nparts) {
    constexpr bool ROW_TAIL = GROUPS == G_COL || GROUPS == G_COL_ALL || GROUPS == G_TENSOR;   // rows need not fill the last tile
    __shared__ float red[4 * 128];                      // per wave: column maxima (G_COL128) or one value
    __shared__ float inv_s[128];
    __shared__ __attribute__((aligned(16))) uint8_t tile[TRANSPOSE ? 128 * (128 + 16) : 16];   // [c][r], rows padded to 144 bytes
    const int t = static_cast<int>(threadIdx.x), lane = t & 63, wave = t >> 6;
    const int cc = t & 15, rr = t >> 4;                 // chunk column; the thread's 8 consecutive rows are rr * 8 + [0, 8)
    const unsigned tiles_c = static_cast<unsigned>((cols + 127) >> 7);
    const unsigned by = blockIdx.x / tiles_c, bx = blockIdx.x - by * tiles_c;
    const int64_t r0 = static_cast<int64_t>(by) * 128, c0 = static_cast<int64_t>(bx) * 128;
    const bool live = c0 + cc * 8 < cols;
    u32x4 w[8];
    auto load = [&](auto streamed_c) __attribute__((always_inline)) {
#pragma unroll
        for (int sw = 0; sw < 8; ++sw) {
            w[sw] = u32x4{0u, 0u, 0u, 0u};
            if (live && (!ROW_TAIL || r0 + rr * 8 + sw < rows))
                w[sw] = load_chunk<decltype(streamed_c)::value>(x + (r0 + rr * 8 + sw) * ld + c0 + cc * 8);
        }
    };
    if (streamed) { load(std::true_type{}); asm volatile("; streamed"); }         // (as in quant_rows_kernel)
    else { load(std::false_type{}); asm volatile("; through the caches"); }
    float inv8[8];
    if (GROUPS == G_COL128 || GROUPS == G_COL_ALL) {
        float a[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        auto column_maxima = [&](const u32x4 (&v)[8]) __attribute__((always_inline)) {
#pragma unroll
            for (int sw = 0; sw < 8; ++sw) {
                a[0] = fmaxf(a[0], fabsf(bf16_lo(v[sw].x))); a[1] = fmaxf(a[1], fabsf(bf16_hi(v[sw].x)));
                a[2] = fmaxf(a[2], fabsf(bf16_lo(v[sw].y))); a[3] = fmaxf(a[3], fabsf(bf16_hi(v[sw].y)));
                a[4] = fmaxf(a[4], fabsf(bf16_lo(v[sw].z))); a[5] = fmaxf(a[5], fabsf(bf16_hi(v[sw].z)));
                a[6] = fmaxf(a[6], fabsf(bf16_lo(v[sw].w))); a[7] = fmaxf(a[7], fabsf(bf16_hi(v[sw].w)));
            }
        };
        if (GROUPS == G_COL_ALL) {
            for (int64_t rb = 0; rb < rows; rb += 128) {
                if (rb == r0) continue;
                u32x4 v[8];
#pragma unroll
                for (int sw = 0; sw < 8; ++sw) {
                    v[sw] = u32x4{0u, 0u, 0u, 0u};
                    if (live && rb + rr * 8 + sw < rows)
                        v[sw] = *reinterpret_cast<const u32x4*>(x + (rb + rr * 8 + sw) * ld + c0 + cc * 8);
                }
                column_maxima(v);
            }
        }
        column_maxima(w);
        // lanes l, l ^ 16, l ^ 32, l ^ 48 of a wave hold the same columns (rows rr differ); then the 4 waves through LDS
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            a[j] = fmaxf(a[j], wave_shfl_xor(a[j], 16));
            a[j] = fmaxf(a[j], wave_shfl_xor(a[j], 32));
        }
        if (lane < 16) {
#pragma unroll
            for (int j = 0; j < 8; ++j) red[wave * 128 + cc * 8 + j] = a[j];
        }
        __syncthreads();
        if (t < 128) {
            const float am = fmaxf(fmaxf(red[t], red[128 + t]), fmaxf(red[256 + t], red[384 + t]));
            float sc, iv;
            group_scale_any(pow2 != 0, am, sc, iv);
            inv_s[t] = iv;
            if (GROUPS == G_COL_ALL) {
                if (by == 0 && c0 + t < cols) scales[c0 + t] = sc;
            } else if (c0 + t < cols) {
                scales[(c0 + t) * (rows >> 7) + by] = sc;
            }
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 8; ++j) inv8[j] = inv_s[cc * 8 + j];
    } else if (GROUPS == G_COL) {
        // two threads per column fold half of the partials each (loads of 128 consecutive floats, eight in flight)
        const int col = t & 127, half = t >> 7;
        float am = 0.f;
        if (c0 + col < cols) {
            const float* src = parts + c0 + col;
            for (int k0 = half; k0 < nparts; k0 += 16) {
                float v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = k0 + 2 * u < nparts ? src[static_cast<int64_t>(k0 + 2 * u) * cols] : 0.f;
#pragma unroll
                for (int u = 0; u < 8; ++u) am = fmaxf(am, v[u]);
            }
        }
        red[half * 128 + col] = am;
        __syncthreads();
        if (t < 128) {
            float sc, iv;
            group_scale(fmaxf(red[t], red[128 + t]), sc, iv);
            inv_s[t] = iv;
            if (by == 0 && c0 + t < cols) scales[c0 + t] = sc;
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 8; ++j) inv8[j] = inv_s[cc * 8 + j];
    } else {
        float a = 0.f;
        if (GROUPS == G_TENSOR) {
            for (int k = t; k < nparts; k += 256) a = fmaxf(a, parts[k]);
        } else {
#pragma unroll
            for (int sw = 0; sw < 8; ++sw) a = fmaxf(a, chunk_amax(w[sw]));
        }
        a = lanes_max<64>(a);
        if (lane == 0) red[wave] = a;
        __syncthreads();
        float sc, iv;
        group_scale_any(pow2 != 0, fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3])), sc, iv);
        if (GROUPS == G_TENSOR) {
            if (t == 0 && blockIdx.x == 0) scales[0] = sc;
        } else if (t == 0) {
            scales[by * static_cast<int64_t>(tiles_c) + bx] = sc;
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) inv8[j] = iv;
    }
    uint32_t lo[8], hi[8];                              // codes of row rr * 8 + sw, columns cc * 8 + [0, 4) and + [4, 8)
#pragma unroll
    for (int sw = 0; sw < 8; ++sw) {
        lo[sw] = e4m3x4(bf16_lo(w[sw].x) * inv8[0], bf16_hi(w[sw].x) * inv8[1], bf16_lo(w[sw].y) * inv8[2], bf16_hi(w[sw].y) * inv8[3]);
        hi[sw] = e4m3x4(bf16_lo(w[sw].z) * inv8[4], bf16_hi(w[sw].z) * inv8[5], bf16_lo(w[sw].w) * inv8[6], bf16_hi(w[sw].w) * inv8[7]);
        if (!TRANSPOSE && live && (!ROW_TAIL || r0 + rr * 8 + sw < rows))
            *reinterpret_cast<u32x2*>(q + (r0 + rr * 8 + sw) * cols + c0 + cc * 8) = u32x2{lo[sw], hi[sw]};
    }
    if (TRANSPOSE) {
        // the thread's 8 x 8 block of codes is transposed in registers (byte permutes on 4 x 4 sub-blocks), so that each
        // of its 8 columns becomes one 8-byte run of consecutive rows; the runs go through LDS and leave as 64-byte runs
        auto t4 = [](uint32_t a0, uint32_t a1, uint32_t a2, uint32_t a3, uint32_t (&c)[4]) __attribute__((always_inline)) {
            const uint32_t p0 = __builtin_amdgcn_perm(a1, a0, 0x05010400u), p1 = __builtin_amdgcn_perm(a1, a0, 0x07030602u);
            const uint32_t p2 = __builtin_amdgcn_perm(a3, a2, 0x05010400u), p3 = __builtin_amdgcn_perm(a3, a2, 0x07030602u);
            c[0] = __builtin_amdgcn_perm(p2, p0, 0x05040100u); c[1] = __builtin_amdgcn_perm(p2, p0, 0x07060302u);
            c[2] = __builtin_amdgcn_perm(p3, p1, 0x05040100u); c[3] = __builtin_amdgcn_perm(p3, p1, 0x07060302u);
        };
        uint32_t a[4], b[4], c[4], d[4];
        t4(lo[0], lo[1], lo[2], lo[3], a);                  // columns 0..3, rows 0..3
        t4(lo[4], lo[5], lo[6], lo[7], b);                  // columns 0..3, rows 4..7
        t4(hi[0], hi[1], hi[2], hi[3], c);                  // columns 4..7, rows 0..3
        t4(hi[4], hi[5], hi[6], hi[7], d);                  // columns 4..7, rows 4..7
        // (LDS row = output row: 16 runs of 8 codes, run rr at position rr ^ cc with cc = the row's chunk column: the 64
        // lanes of a write then spread over all banks two deep, where unswizzled they met on 16 of the 64)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            *reinterpret_cast<u32x2*>(tile + (cc * 8 + j) * 144 + ((rr ^ cc) << 3)) = u32x2{a[j], b[j]};
            *reinterpret_cast<u32x2*>(tile + (cc * 8 + 4 + j) * 144 + ((rr ^ cc) << 3)) = u32x2{c[j], d[j]};
        }
        __syncthreads();
        // output row c0 + c: 128 codes.  Eight consecutive lanes write one row's 128 bytes, a store instruction of a
        // wave eight whole rows (full cache lines per request: with a thread per half row, four stores apart, every
        // instruction scattered 16-byte pieces over 32 lines)
        const int chunk = t & 7;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int col = j * 32 + (t >> 3), key = col >> 3;           // the row's runs 2 chunk, 2 chunk + 1 sit at ^ key
            u32x4 v = *reinterpret_cast<const u32x4*>(tile + col * 144 + ((chunk ^ (key >> 1)) << 4));
            if (key & 1) v = u32x4{v.z, v.w, v.x, v.y};
            if (c0 + col < cols && (!ROW_TAIL || r0 + chunk * 16 < rows))
                *reinterpret_cast<u32x4*>(q + (c0 + col) * rows + r0 + chunk * 16) = v;
        }
    }
}

__global__ void e4m3_from_f32_kernel(const float* __restrict__ t, uint8_t* __restrict__ codes, int64_t n) {
    int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < n) codes[i] = static_cast<uint8_t>(e4m3x4(t[i], 0.f, 0.f, 0.f) & 0xFFu);
}

// ---------------------------------------------------------------------------------
// Whether X is read past the caches.  Under 64 MB a plain read is as fast or faster whatever the last-level cache holds.  A pass, us,
// streamed -> plain, on one X in every pass | on an X that no cache holds | on an X that the kernel before has written (with that
// kernel):
//   quantization alone        49152 x 512                14.9 -> 13.8 | 16.0 -> 15.9 | 33.3 -> 32.6
//                             16384 x 1024                9.1 ->  9.1 | 10.6 -> 10.8 | 24.5 -> 23.6
//                             65536 x 256                 9.1 ->  9.0 | 10.6 -> 10.5 | 24.5 -> 23.2
//   layer (M x K x N)         65536 x 256 x 768          54.5 -> 51.7 | 52.5 -> 51.1 | 65.1 -> 63.0
//                             65536 x 384 x 384          55.6 -> 52.0 | 53.6 -> 51.8 | 69.6 -> 69.2
//                             65536 x 128 x 512          32.0 -> 31.7 | 31.2 -> 31.7 | 35.4 -> 35.1
//   ... in block scales       8192 x 2048 x 2048         58.5 -> 56.5 | 55.7 -> 54.2 | 66.3 -> 66.3
//                             65536 x 256 x 256          37.3 -> 28.5 | 36.8 -> 28.8 | 42.3 -> 41.0
//   two layers                65536 x 256 x 512 x 256    66.4 -> 64.2 | 66.2 -> 65.5 | 80.1 -> 78.2
//                             65536 x 256 x 1024 x 256   93.7 -> 91.5 | 93.3 -> 92.6 | 105.4 -> 104.2 (three X in turn 91.6 -> 92.5)
//                             65536 x 128 x 512 x 128    51.7 -> 52.6 | 51.7 -> 53.0 | 60.2 -> 60.0
//   training step             16384 x 512 x 512          81.8 -> 79.0 | 81.8 -> 81.2 | 90.0 -> 88.6
//   probe                     16384 x 1024 x 1024         120 -> 118  |  115 -> 113  |  127 -> 125
// From 64 MB on X stays in that cache in the place of what the calls behind it read: a training step of 57472 x 896 x 1664 takes
// 551 us with X (103 MB) and dY (191 MB) streamed and 569 with both plain, one of 65536 x 256 x 1024 (dY 128 MB) 207 and 225.
static bool read_streamed(int64_t rows, int64_t cols) { return rows * cols >= int64_t(1) << 25; }

template <bool B128>
static void launch_rows(const uint16_t* x, int64_t rows, int64_t cols, int64_t ld, uint8_t* q, float* scales,
                        int pow2, hipStream_t s) {
    const int64_t chunks = cols / 8;
    const bool streamed = read_streamed(rows, cols);
    auto grid = [&](int rows_per_wave) {
        return dim3(static_cast<unsigned>((rows + 4 * rows_per_wave - 1) / (4 * rows_per_wave)));
    };
#define LOKA_QR(TPR, CPL, RU) \
    quant_rows_kernel<TPR, CPL, RU, B128><<<grid((64 / TPR) * RU), 256, 0, s>>>(x, rows, cols, ld, q, scales, pow2, streamed)
    // Rows per wave: enough loads in flight per lane when the launch has many waves per SIMD anyway, fewer rows
    // per wave (more waves) when the whole tensor would otherwise be a handful of waves per SIMD.
    const bool few = rows * chunks < (int64_t(1) << 21);      // under 32 MB of bf16 (measured: 16384 x 512 8.8 -> 6.7 us)
    if (chunks <= 16) LOKA_QR(16, 1, 2);
    else if (chunks <= 32) { if (few) LOKA_QR(32, 1, 1); else LOKA_QR(32, 1, 4); }
    else if (chunks <= 64) { if (few) LOKA_QR(64, 1, 2); else LOKA_QR(64, 1, 8); }
    else if (chunks <= 128) { if (few) LOKA_QR(64, 2, 1); else LOKA_QR(64, 2, 4); }
    else if (chunks <= 256) LOKA_QR(64, 4, 2);
    else if (chunks <= 512) LOKA_QR(64, 8, 1);
    else if (chunks <= 1024) LOKA_QR(64, 16, 1);
    else if (!B128 && chunks <= 16384) {
        // as many workgroups as stay resident: 2 per CU (2048 threads) while a thread's row share is small
        const int64_t slots = chunks <= 4096 ? 512 : 256;
        const dim3 g(static_cast<unsigned>(rows < slots ? rows : slots));
        if (chunks <= 2048) quant_wide_rows_kernel<2><<<g, 1024, 0, s>>>(x, rows, cols, ld, q, scales);
        else if (chunks <= 4096) quant_wide_rows_kernel<4><<<g, 1024, 0, s>>>(x, rows, cols, ld, q, scales);
        else if (chunks <= 8192) quant_wide_rows_kernel<8><<<g, 1024, 0, s>>>(x, rows, cols, ld, q, scales);
        else quant_wide_rows_kernel<16><<<g, 1024, 0, s>>>(x, rows, cols, ld, q, scales);
    } else quant_long_rows_kernel<B128><<<dim3(static_cast<unsigned>(rows)), 256, 0, s>>>(x, rows, cols, ld, q, scales, pow2);
#undef LOKA_QR
}

// COL in one kernel (G_COL_ALL) instead of two: every workgroup reads all row tiles of its columns, so the time grows with
// their number where the amax pass costs a launch.  Measured (us, two kernels -> one): 256 x 1024 7.3 -> 4.8, 256 x 65536
// 18.3 -> 11.5, 256 x 262144 60.9 -> 51.8; 512 x 1024 7.3 -> 5.9, 512 x 16384 11.2 -> 8.1, but 512 x 65536 31.6 -> 40.7 and
// 1024 x 1024 7.4 -> 8.5.
static bool col_in_one(int64_t rows, int64_t cols) { return rows <= 256 || (rows <= 512 && cols <= 16384); }

// Row ranges of a COL amax pass: 128 rows each (four rows per thread) as long as the cast has few partials to fold.
static int64_t col_rows_per_part(int64_t rows) {
    const int64_t per = (rows + kMaxParts - 1) / kMaxParts;
    return ((per < 128 ? 128 : per) + 31) / 32 * 32;
}

// Workgroups of a TENSOR amax pass: four chunks per thread as long as the cast has few partials to fold.
static int64_t tensor_parts(int64_t rows, int64_t cols) {
    const int64_t want = (rows * (cols / 8) + 1023) / 1024;
    return want < kTensorParts ? want : kTensorParts;
}

// (at least the two values per group that callers of the smallest shapes have always been asked for)
size_t quantize_workspace_bytes(loka_scale_mode mode, int64_t rows, int64_t cols) {
    const int64_t groups = mode == LOKA_SCALE_TENSOR ? 1 : cols, per = col_rows_per_part(rows);
    const int64_t parts = mode == LOKA_SCALE_TENSOR ? tensor_parts(rows, cols) : (rows + per - 1) / per;
    return static_cast<size_t>(groups) * (parts < 2 ? 2 : parts) * sizeof(float);
}

loka_status quantize_launch(const void* x_bf16, int64_t rows, int64_t cols, int64_t ld, loka_scale_mode mode,
                            int transpose_out, uint8_t* q, float* scales, void* workspace, hipStream_t s) {
    const uint16_t* x = static_cast<const uint16_t*>(x_bf16);
    // the power-of-two block modes: the plain block modes' passes with another scale rule
    const int pow2 = mode == LOKA_SCALE_BLOCK_1x128_POW2 || mode == LOKA_SCALE_BLOCK_128x128_POW2;
    if (mode == LOKA_SCALE_BLOCK_1x128_POW2) mode = LOKA_SCALE_BLOCK_1x128;
    if (mode == LOKA_SCALE_BLOCK_128x128_POW2) mode = LOKA_SCALE_BLOCK_128x128;
    if (!transpose_out && (mode == LOKA_SCALE_ROW || mode == LOKA_SCALE_BLOCK_1x128)) {
        if (mode == LOKA_SCALE_ROW) launch_rows<false>(x, rows, cols, ld, q, scales, 0, s);
        else launch_rows<true>(x, rows, cols, ld, q, scales, pow2, s);
        return hipGetLastError() == hipSuccess ? LOKA_OK : LOKA_ERR_HIP;
    }
    const bool streamed = read_streamed(rows, cols);
    const dim3 tiles(static_cast<unsigned>(((cols + 127) / 128) * ((rows + 127) / 128)));
    if (mode == LOKA_SCALE_BLOCK_128x128 || mode == LOKA_SCALE_BLOCK_128x1) {
        // groups that fit a workgroup: one pass
        if (mode == LOKA_SCALE_BLOCK_128x1) quant_tile128_kernel<G_COL128, true><<<tiles, 256, 0, s>>>(x, rows, cols, ld, q, scales, 0, streamed, nullptr, 0);
        else if (transpose_out) quant_tile128_kernel<G_TILE, true><<<tiles, 256, 0, s>>>(x, rows, cols, ld, q, scales, pow2, streamed, nullptr, 0);
        else quant_tile128_kernel<G_TILE, false><<<tiles, 256, 0, s>>>(x, rows, cols, ld, q, scales, pow2, streamed, nullptr, 0);
        return hipGetLastError() == hipSuccess ? LOKA_OK : LOKA_ERR_HIP;
    }
    float* parts = static_cast<float*>(workspace);
    if (mode == LOKA_SCALE_TENSOR) {
        const int n = static_cast<int>(tensor_parts(rows, cols));
        amax_tensor_kernel<<<dim3(static_cast<unsigned>(n)), 256, 0, s>>>(x, rows, cols, ld, parts);
        if (transpose_out) quant_tile128_kernel<G_TENSOR, true><<<tiles, 256, 0, s>>>(x, rows, cols, ld, q, scales, 0, streamed, parts, n);
        else quant_tile128_kernel<G_TENSOR, false><<<tiles, 256, 0, s>>>(x, rows, cols, ld, q, scales, 0, streamed, parts, n);
    } else if (col_in_one(rows, cols)) {
        if (transpose_out) quant_tile128_kernel<G_COL_ALL, true><<<tiles, 256, 0, s>>>(x, rows, cols, ld, q, scales, 0, streamed, nullptr, 0);
        else quant_tile128_kernel<G_COL_ALL, false><<<tiles, 256, 0, s>>>(x, rows, cols, ld, q, scales, 0, streamed, nullptr, 0);
    } else {
        const int64_t per = col_rows_per_part(rows);
        const int n = static_cast<int>((rows + per - 1) / per);
        const dim3 g(static_cast<unsigned>((cols + 63) / 64), static_cast<unsigned>(n));
        amax_col_kernel<<<g, 256, 0, s>>>(x, rows, cols, ld, per, parts);
        if (transpose_out) quant_tile128_kernel<G_COL, true><<<tiles, 256, 0, s>>>(x, rows, cols, ld, q, scales, 0, streamed, parts, n);
        else quant_tile128_kernel<G_COL, false><<<tiles, 256, 0, s>>>(x, rows, cols, ld, q, scales, 0, streamed, parts, n);
    }
    return hipGetLastError() == hipSuccess ? LOKA_OK : LOKA_ERR_HIP;
}

loka_status e4m3_from_f32_launch(const float* t, uint8_t* codes, int64_t n, hipStream_t s) {
    e4m3_from_f32_kernel<<<dim3(static_cast<unsigned>((n + 255) / 256)), 256, 0, s>>>(t, codes, n);
    return hipGetLastError() == hipSuccess ? LOKA_OK : LOKA_ERR_HIP;
}

}  // namespace loka
