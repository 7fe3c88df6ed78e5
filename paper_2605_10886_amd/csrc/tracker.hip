// Online distribution tracker of the probe (Section 3.1, "Online Distribution Learning": the batched
// Welford tracker for activations, after Chan et al.).  One batch X [B, K] (bf16) is merged into the running
// summary (n, mu [K], Sigma [K, K] = unnormalized scatter, fp32):
//   mu_b = column means,  S_b = (X - 1 mu_b^T)^T (X - 1 mu_b^T),  n' = n + B,  delta = mu_b - mu,
//   mu' = mu + (B / n') delta,   Sigma' = Sigma + S_b + (n B / n') delta delta^T.
//
// How it runs here.  S_b is computed as X^T X - B mu_b mu_b^T: the raw second moment is a dense
// contraction over the batch rows and goes to the BF16 matrix cores (products of two bf16 values are exact
// in fp32; accumulation is fp32), the column sums are accumulated in fp64 on the vector ALUs, and the
// subtraction, the delta delta^T term and the merge with the stored state are done in fp64 and rounded once.
//
//   tracker_scatter_kernel   one workgroup per (tile pair ti <= tj of 256 x 256 outputs, one of S row ranges of
//                            the batch): raw partial scatter -> workspace (fp32); workgroups on diagonal
//                            tiles also write fp64 column sums of their 256 columns, those of the first range
//                            a copy of the old mean
//   tracker_merge_kernel     folds the column sums (mu_b, delta in fp64) and the partial scatters in a fixed order,
//                            forms S_b and the rank-1 term and updates mu and Sigma in place (both triangles; the
//                            mirror image goes through an LDS transpose)
//
// The contraction runs over the rows of a row-major matrix, i.e. over the strided dimension of both MFMA
// operands: an MFMA lane needs 8 consecutive batch rows of ONE column.  Each 8 x 8 block of X is transposed
// once, in registers, on its way from global memory to LDS (byte permutes), so that an operand fragment is a
// single 16-byte LDS read.  The MFMA's k order is irrelevant here because both operands come from the same
// rows in the same order.
#include "gemm_common.h"
#include "tracker_stage.h"

#include <type_traits>

namespace loka {

typedef float v16f __attribute__((ext_vector_type(16)));

constexpr int TRK_T = 256;                      // output tile (columns i x columns j) per workgroup
constexpr int TRK_MS = 64;                      // batch rows per pipeline stage (four MFMA k steps of 16)
constexpr int TRK_TILEB = TRK_MS * TRK_T * 2;   // one operand tile of a stage (32 KB)
constexpr int TRK_STAGEB = 2 * TRK_TILEB;       // i tile, then j tile
constexpr size_t TRK_LDS = 2 * TRK_STAGEB + 2 * TRK_T * sizeof(double);
constexpr int TRK_PLAN_SLOTS = 256;             // cost model only: workgroups assumed in flight per round (the CU count of an
                                                // MI355X).  It steers the number of row splits (and with it the workspace
                                                // size, which must not depend on the device); results do not depend on it

// Work decomposition: workgroup = (tile pair ti <= tj, one of S equal row ranges of the batch).  All
// workgroups in flight walk their rows at the same pace, so the workgroups of an XCD that share a column
// tile find it in that XCD's L2.  S trades the rounding of pairs * S to whole rounds of 256 workgroups
// against the fp32 partial tile every workgroup leaves in the workspace (256 KB written and read back, 144 of a diagonal one).
struct TrackerPlan {
    int T, pairs, splits;
    int64_t rows_per_split;
    size_t off_colsum, off_mu, bytes;
};

TrackerPlan tracker_plan(int64_t B, int64_t K) {
    TrackerPlan pl{};
    pl.T = static_cast<int>((K + TRK_T - 1) / TRK_T);
    pl.pairs = pl.T * (pl.T + 1) / 2;
    const int64_t steps = (B + TRK_MS - 1) / TRK_MS;
    int64_t max_s = steps / 2 > 0 ? steps / 2 : 1;                    // at least 2 stages per workgroup
    if (max_s > 256) max_s = 256;
    // estimated time in units of one stage (about 1.2 us): rounds * (stages per workgroup + start-up) for the
    // scatter, and so much per partial tile, written and then read back by the merge: 256 KB, of a diagonal tile 144
    // (one tile: its merge is a few workgroups and takes longer with every range).  More from 8 column tiles on, where the
    // partial tiles are 100 MB and more and the plans' estimates lie close together (ranges by 0.08 and 0.05, by 0.1, us:
    // 65536 x 2560 9 473, 4 455; 8000 x 2048 7 60.4, 6 59.7; 65536 x 4096 7 1180, 250 MB, 5 1180, 178 MB).
    const double tiles_cost = pl.T == 1 ? 0.06 : pl.T >= 8 ? 0.1 * pl.pairs : 0.08 * (pl.pairs - pl.T) + 0.05 * pl.T;
    int64_t best_s = 1;
    double best = 1e300;
    for (int64_t sp = 1; sp <= max_s; ++sp) {
        const int64_t rounds = (static_cast<int64_t>(pl.pairs) * sp + TRK_PLAN_SLOTS - 1) / TRK_PLAN_SLOTS;
        const double cost = static_cast<double>(rounds) * ((steps + sp - 1) / sp + 3) + tiles_cost * static_cast<double>(sp);
        if (cost < best) { best = cost; best_s = sp; }
    }
    int64_t rows = (B + best_s - 1) / best_s;
    rows = (rows + TRK_MS - 1) / TRK_MS * TRK_MS;
    pl.rows_per_split = rows;
    pl.splits = static_cast<int>((B + rows - 1) / rows);
    const size_t slots = static_cast<size_t>(pl.splits) * pl.pairs;
    const size_t kp = static_cast<size_t>(pl.T) * TRK_T;
    pl.off_colsum = slots * TRK_T * TRK_T * sizeof(float);
    pl.off_mu = pl.off_colsum + slots * TRK_T * sizeof(double);
    pl.bytes = pl.off_mu + kp * sizeof(float);
    return pl;
}

struct TrackerParams {
    const uint16_t* x;
    int64_t B, ld, rows_per_split;
    int K, T, pairs, splits;
    float* partial;      // [splits][pairs][256][256] (of a diagonal pair the 32 x 32 blocks on and above the diagonal, live columns)
    double* colsum;      // [splits][pairs][256] (written for diagonal pairs only)
    const float* mu;     // [K]: the mean before this call, copied to
    float* mu_old;       // the workspace by the diagonal pairs of the first range
};

__device__ __forceinline__ void pair_to_tiles(int pair, int T, int& ti, int& tj) {
    int i = 0, rem = pair;
    while (rem >= T - i) { rem -= T - i; ++i; }
    ti = i; tj = i + rem;
}
__host__ __device__ __forceinline__ int diag_pair(int t, int T) { return t * T - t * (t - 1) / 2; }

// 8 waves: wave (wi, wj) of a 2 x 4 arrangement owns 4 x 2 MFMA blocks of 32 x 32 (v_mfma_f32_32x32x16_bf16).
//
// Staging.  A stage is 64 batch rows x 256 columns per operand.  Thread (c = chunk of 8 columns, g = group
// of 8 rows) fetches its 8 x 8 block (8 loads of 16 bytes, 512-byte runs per row across 32 lanes), transposes
// it in registers (32 byte permutes) and writes one 16-byte word per column: the 8 contraction values an
// MFMA lane needs, so an operand fragment is ONE ds_read_b128.  LDS layout of a tile: [row group g][position
// pos][16 bytes] with column 8 c + e at position 32 e + c: the 32 lanes that write column e of their chunks
// write 512 consecutive bytes, and MFMA block t (positions 32 t .. 32 t + 31) is the set of columns 8 m + t,
// m = 0..31 = the block's MFMA row (or column) index.  Which tile column lands on which MFMA row is free as
// long as the epilogue knows: wave (wi, wj) owns blocks 4 wi .. 4 wi + 3 on the i side, 2 wj, 2 wj + 1 on the j side.
// A diagonal pair needs only the MFMA blocks (a, b) with a <= b, block (b, a) being the transpose of (a, b): 36 of 64.  Its
// waves 0..5 own the four blocks of one pair of 2-block groups each, waves 6 and 7 the three blocks within each of two groups;
// a SIMD (waves w, w + 4) then issues 8 or 10 MFMAs per k step instead of 16.  The blocks below the diagonal are filled in from
// the same registers when the tile leaves through LDS.  (Ranges of few stages: all 64 blocks, like any other pair.)
// Waves 0..3 stage the i tile, waves 4..7 the j tile (nothing on a diagonal pair, where both operands are
// the i tile).  The loads of stage s + 1 are in flight while stage s is multiplied (registers), two LDS
// buffers, one barrier per stage.
__global__ __launch_bounds__(512) void tracker_scatter_kernel(const TrackerParams p) {
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
    double* red = reinterpret_cast<double*>(smem + 2 * TRK_STAGEB);           // [2][256]

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wi = wave >> 2, wj = wave & 3;
    const int ldB = static_cast<int>(p.ld) * 2;

    // Renumbered, an XCD's workgroups share row ranges.  Where the grid is no multiple of 8 that pays from about 1000 rows per
    // range on (launch order -> renumbered, batch x features: 53098 x 1240, ranges of 3136, 126.4 -> 115.3 us; 32768 x 1024,
    // 1728, 72.5 -> 70.5; nothing either way from 830 to 1250: 8192 x 1024, 832, 38.9 -> 39.2); short ranges are faster in
    // launch order (1593 x 1168, 320, 26.3 -> 28.6; 18786 x 456, 576, 32.3 -> 34.3).
    const bool spread = gridDim.x % 8 == 0 || p.rows_per_split >= 1024;
    const int id = spread ? xcd_contiguous(blockIdx.x, gridDim.x) : static_cast<int>(blockIdx.x);
    const int split = id / p.pairs, pair = id - split * p.pairs;
    const int64_t row_begin = static_cast<int64_t>(split) * p.rows_per_split;
    const int64_t row_end = row_begin + p.rows_per_split < p.B ? row_begin + p.rows_per_split : p.B;
    const int nst = static_cast<int>((row_end - row_begin + TRK_MS - 1) / TRK_MS);
    int ti, tj;
    pair_to_tiles(pair, p.T, ti, tj);
    const bool diag = ti == tj;

    // staging role of this thread
    const bool stager = wave < 4 || !diag;
    const int my_tile = wave < 4 ? ti : tj;
    const int sc = tid & 31, sg = (tid & 255) >> 5;                         // column chunk, row group
    // everything that decides whether a load is in range sits in the per-lane offset: rows past the end of
    // the batch fall behind the descriptor's byte count, columns past K get an offset beyond any descriptor
    const unsigned st_voff = (my_tile * TRK_T + sc * 8 < p.K) ? static_cast<unsigned>(sg * 8 * ldB + sc * 16) : 0x80000000u;
    const int st_lds = (wave < 4 ? 0 : TRK_TILEB) + sg * 4096 + sc * 16;    // + 512 e per column of the chunk
    u32x4 in[8];
    auto fetch = [&](int st) __attribute__((always_inline)) {
        if (!stager) return;
        const int64_t r0 = row_begin + static_cast<int64_t>(st) * TRK_MS;
        int64_t rows_valid = row_end - r0;
        rows_valid = rows_valid > TRK_MS ? TRK_MS : rows_valid;
        const int rec = static_cast<int>(rows_valid) * ldB - my_tile * TRK_T * 2;
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<uint16_t*>(p.x + r0 * p.ld + my_tile * TRK_T), 0, rec, 0x00020000);
#pragma unroll
        for (int r = 0; r < 8; ++r)
            in[r] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, st_voff + static_cast<unsigned>(r * ldB), 0, 0));
    };
    auto stage = [&](int buf) __attribute__((always_inline)) {
        if (!stager) return;
        uint8_t* dst = smem + buf * TRK_STAGEB + st_lds;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            u32x4 o;
            const unsigned sel = (e & 1) ? 0x07060302u : 0x05040100u;
            o.x = __builtin_amdgcn_perm(in[1][e >> 1], in[0][e >> 1], sel);
            o.y = __builtin_amdgcn_perm(in[3][e >> 1], in[2][e >> 1], sel);
            o.z = __builtin_amdgcn_perm(in[5][e >> 1], in[4][e >> 1], sel);
            o.w = __builtin_amdgcn_perm(in[7][e >> 1], in[6][e >> 1], sel);
            *reinterpret_cast<u32x4*>(dst + e * 512) = o;
        }
    };

    // fragment reads: lane (m = lane % 32, h = lane / 32) takes position 32 t + m of row group 2 kk + h
    const int fr_off = (lane >> 5) * 4096 + (lane & 31) * 16;
    const int a_off = fr_off + wi * 4 * 512, b_off = fr_off + wj * 2 * 512;
    auto read_frags = [&](const uint8_t* At, const uint8_t* Bt, int kk, v8bf (&fa)[4], v8bf (&fb)[2]) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < 4; ++t) fa[t] = __builtin_bit_cast(v8bf, *reinterpret_cast<const u32x4*>(At + a_off + t * 512 + kk * 8192));
#pragma unroll
        for (int e = 0; e < 2; ++e) fb[e] = __builtin_bit_cast(v8bf, *reinterpret_cast<const u32x4*>(Bt + b_off + e * 512 + kk * 8192));
    };
    auto run = [&](auto diag_c) __attribute__((always_inline)) {
        constexpr bool DIAG = decltype(diag_c)::value;
        v16f acc[4][2];
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int e = 0; e < 2; ++e)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[t][e][r] = 0.f;
        auto mma = [&](const v8bf (&fa)[4], const v8bf (&fb)[2]) __attribute__((always_inline)) {
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int e = 0; e < 2; ++e)
                    acc[t][e] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[t], fb[e], acc[t][e], 0, 0, 0);
        };
        // issue order of one k step: an MFMA, then one LDS read of the next step's fragments, six times over
        auto interleave = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < 6; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            }
            __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
        };
        // diagonal pairs: groups (2 blocks each) of this wave; waves 0..5 multiply the two, waves 6, 7 each with itself
        const int g0 = trk_group(wave, 0), g1 = trk_group(wave, 1);
        const bool self = trk_self(wave);
        auto read_diag = [&](const uint8_t* At, int kk, v8bf (&f)[4]) __attribute__((always_inline)) {
#pragma unroll
            for (int t = 0; t < 4; ++t)
                f[t] = __builtin_bit_cast(v8bf, *reinterpret_cast<const u32x4*>(At + fr_off + (2 * (t < 2 ? g0 : g1) + (t & 1)) * 512 + kk * 8192));
        };
        auto mma_diag = [&](const v8bf (&f)[4]) __attribute__((always_inline)) {
            if (self) {
#pragma unroll
                for (int t = 0; t < 4; ++t)
#pragma unroll
                    for (int e = t & 1; e < 2; ++e)
                        acc[t][e] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[t], f[(t & 2) + e], acc[t][e], 0, 0, 0);
            } else {
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int e = 0; e < 2; ++e)
                        acc[t][e] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[t], f[2 + e], acc[t][e], 0, 0, 0);
            }
        };
        // column sums (diagonal pairs): thread = (position tid % 256, row groups 4 (tid / 256) .. + 3), fp64
        double cs = 0.0;
        const int cs_off = (tid >> 8) * 4 * 4096 + (tid & 255) * 16;

        fetch(0);
        stage(0);
        __syncthreads();
        for (int s = 0; s < nst; ++s) {
            const uint8_t* At = smem + (s & 1) * TRK_STAGEB;
            const uint8_t* Bt = diag ? At : At + TRK_TILEB;
            // the two waves of a SIMD (w, w + 4) request their blocks of the next stage at different times: a wave
            // sits in the load issue until the memory pipeline has taken its requests, and should not do so together
            // with the wave that shares its matrix pipe.  (Measured: both groups at the start of the stage 750 us
            // at B = 32768, K = 4096; staggered 690 us; the eight loads spread over the stage, two per k step, with
            // a second register set so that they have a whole stage to land: 955 us.)
            if (s + 1 < nst && wave < 4) fetch(s + 1);
            if constexpr (!DIAG) {
                v8bf fa0[4], fb0[2], fa1[4], fb1[2];
                read_frags(At, Bt, 0, fa0, fb0);
                read_frags(At, Bt, 1, fa1, fb1);
                mma(fa0, fb0);
                interleave();
                if (s + 1 < nst && wave >= 4) fetch(s + 1);
                read_frags(At, Bt, 2, fa0, fb0);
                mma(fa1, fb1);
                interleave();
                read_frags(At, Bt, 3, fa1, fb1);
                mma(fa0, fb0);
                interleave();
                mma(fa1, fb1);
            } else {
                v8bf f0[4], f1[4];
                read_diag(At, 0, f0);
                read_diag(At, 1, f1);
                mma_diag(f0);
                read_diag(At, 2, f0);
                mma_diag(f1);
                read_diag(At, 3, f1);
                mma_diag(f0);
                mma_diag(f1);
            }
            if (diag) {
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const u32x4 v = *reinterpret_cast<const u32x4*>(At + cs_off + g * 4096);
#pragma unroll
                    for (int w = 0; w < 4; ++w) {
                        cs += static_cast<double>(bf16_lo(v[w]));
                        cs += static_cast<double>(bf16_hi(v[w]));
                    }
                }
            }
            if (s + 1 < nst) stage((s + 1) & 1);
            __syncthreads();
        }

        // raw partial scatter: element r of a lane is MFMA row R = 8 (r / 4) + 4 h + r % 4, MFMA column C = lane % 32 of its
        // block; block (ta, tb) row R is tile row 8 R + 4 wi + ta, column C is tile column 8 C + 2 wj + tb: a lane holds
        // pairs of columns 32 bytes apart.  Stored straight from registers every instruction would scatter 8-byte pieces
        // over 64 cache lines (measured: 70 us of the 780 us at B = 32768, K = 4096); the tile goes through the stage
        // buffers instead, 128 rows at a time (R < 16, then R >= 16 = elements r < 8, then r >= 8), and leaves as whole
        // 1 KB rows (tracker_stage.h: the writes of 32 lanes are 256 consecutive bytes).
        // (offsets recomputed from an opaque copy of the lane id: derived from a loop invariant, the compiler
        // would keep the addresses alive across the main loop, in registers the accumulators need)
        int lane_o = lane, tid_o = tid;
        asm volatile("" : "+v"(lane_o), "+v"(tid_o));
        float* const stg = reinterpret_cast<float*>(smem);
        // Diagonal pairs: acc[t][e] is block (a, b) = (2 ga + t % 2, 2 gb + e).
        const int h_o = lane_o >> 5, c_o = lane_o & 31;
        auto grp_a = [&](int t) __attribute__((always_inline)) { return t < 2 ? g0 : g1; };
        auto grp_b = [&](int t) __attribute__((always_inline)) { return DIAG ? (self ? grp_a(t) : g1) : wj; };
        const int q4 = tid_o & 63, cq = q4 >> 1, uq = q4 & 1;
        const int st_r = (tid_o >> 6) * 256 + (2 * uq) * 64, pos_r = (2 * cq) ^ (uq * 32);
        float* const out = p.partial + static_cast<int64_t>(id) * (TRK_T * TRK_T) + (tid_o >> 6) * TRK_T + 4 * q4;
#pragma unroll
        for (int ps = 0; ps < 2; ++ps) {
            if (ps) __syncthreads();                                        // the first half has been read out of LDS
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                if (DIAG && !self && !trk_pair_holds(t)) continue;
                const TrkAddr ad = trk_direct(DIAG, DIAG ? 2 * grp_a(t) + (t & 1) : 4 * wi + t, 2 * grp_b(t), h_o, c_o);
                float* const st = stg + ad.row;
                if (DIAG && self && !trk_self_stores(t, 0)) {
#pragma unroll
                    for (int r8 = 0; r8 < 8; ++r8) st[trk_direct_step(r8) + (ad.pos ^ trk_direct_key(DIAG, r8)) + 1] = acc[t][1][8 * ps + r8];
                } else {
#pragma unroll
                    for (int r8 = 0; r8 < 8; ++r8)
                        *reinterpret_cast<f32x2_t*>(st + trk_direct_step(r8) + (ad.pos ^ trk_direct_key(DIAG, r8))) =
                            f32x2_t{acc[t][0][8 * ps + r8], acc[t][1][8 * ps + r8]};
                }
            }
            if constexpr (DIAG) {
                if ((c_o >> 4) == ps) {
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        if (self ? !trk_self_mirrors(t, 1) : !trk_pair_holds(t)) continue;
#pragma unroll
                        for (int e = 0; e < 2; ++e) {
                            if (self && !trk_self_mirrors(t, e)) continue;         // (a, a) is its own mirror image
                            const TrkAddr ad = trk_mirror(2 * grp_a(t) + (t & 1), 2 * grp_b(t) + e, h_o, c_o);
                            float* const st = stg + ad.row;
#pragma unroll
                            for (int r = 0; r < 16; ++r) st[ad.pos ^ trk_mirror_key(r)] = acc[t][e][r];
                        }
                    }
                }
            }
            __syncthreads();
            // a diagonal tile leaves from its 32 x 32 blocks on the diagonal on, and as far as there are columns: the merge reads
            // nothing else of it
            const int last = DIAG || diag ? p.K - ti * TRK_T : TRK_T;
#pragma unroll 4
            for (int it = 0; it < 16; ++it) {
                const float* const src = stg + st_r + it * 8 * 256 + (pos_r ^ (DIAG ? 2 * it : 0));
                const f32x2_t lo = *reinterpret_cast<const f32x2_t*>(src);
                const f32x2_t hi = *reinterpret_cast<const f32x2_t*>(src + 64);
                if (!(DIAG || diag) || (4 * q4 >= 32 * (4 * ps + it / 4) && 4 * q4 < last))
                    *reinterpret_cast<v4f*>(out + (128 * ps + it * 8) * TRK_T) = v4f{lo[0], lo[1], hi[0], hi[1]};
            }
        }
        if (diag) {
            // position pos holds column 8 (pos % 32) + pos / 32
            // (from a copy of its own: the ids' parts would be kept across the main loop, in two registers that are spilled)
            int tid_e = tid;
            asm volatile("" : "+v"(tid_e));
            const int pos = tid_e & 255, col = 8 * (pos & 31) + (pos >> 5);
            red[(tid_e >> 8) * TRK_T + col] = cs;
            __syncthreads();
            if (tid_e < TRK_T) {
                p.colsum[static_cast<int64_t>(id) * TRK_T + tid_e] = red[tid_e] + red[TRK_T + tid_e];
                const int k = ti * TRK_T + tid_e;
                if (id < p.pairs && k < p.K) p.mu_old[k] = p.mu[k];          // id = range * pairs + pair
            }
        }
    };
    // Short ranges do not pay for the transposed writes (us, all blocks -> a <= b, ranges in stages: 2000 x 64, 2, 13.4 -> 14.2;
    // 4096 x 512, 4, 22.0 -> 22.4; 1593 x 1168, 5, 24.3 -> 24.3; 18786 x 456, 9, 29.9 -> 29.6; 30000 x 768, 17, 46.0 -> 44.5;
    // 32768 x 1024, 27, 61.6 -> 59.3; 65536 x 1024, 41, 98.2 -> 91.0; 32768 x 4096, 103, 620.8 -> 609.1)
    if (diag && nst >= 6) run(std::true_type{});
    else run(std::false_type{});
}

// Bound by the latency of the loads of a run's ranges and, with many tiles, by their bytes: what is never read is not
// written either (whole call, us: 32768 x 1024 63.3 -> 58.8, 65536 x 512 45.7 -> 42.9,
// 65536 x 256 35.7 -> 32.2, 16384 x 512 30.3 -> 26.9, 4000 x 1024 28.3 -> 26.8, 32768 x 4096 the same).
// grid (pairs, 64): workgroup y handles the 32 x 32 block (y / 8, y % 8) of its pair's tile, PARTS threads per run of four
// columns (each folds every PARTS-th range, their sums are added in order), and the mirrored block of the lower
// triangle (through a transposing LDS tile, so both triangles are written in full 128-byte runs); of a diagonal pair's
// blocks those below the diagonal have nothing to do.
// The workgroup folds the column sums of its 64 columns by itself (wave q takes the ranges q, q + 4 PARTS, ..., then the
// waves' sums in order: the same bits in every workgroup), with the first loads in flight together with those of the
// partial tiles.  A kernel of its own for the means ran a few workgroups for 4.7 us between the two large ones (whole
// call before and after: 65536 x 256 42.0 -> 36.8 us, 4096 x 512 23.7 -> 22.0, 32768 x 1024 64.6 -> 62.0).  The
// old mean is the scatter kernel's copy, because the workgroups of the diagonal blocks overwrite mu here.
template <int PARTS>
__global__ __launch_bounds__(256 * PARTS) void tracker_merge_kernel(const float* __restrict__ partial, const double* __restrict__ colsum,
                                                            const float* __restrict__ mu_old, int T, int pairs, int splits,
                                                            int K, int64_t B, double ratio, double coef,
                                                            float* __restrict__ mu, float* __restrict__ sigma) {
    __shared__ double tr[32][33];
    __shared__ double part[4 * PARTS][64], mub[64], delta[64];           // columns: 32 of the i block, 32 of the j block
    __shared__ double sums[PARTS > 1 ? PARTS - 1 : 1][4][256];
    const int tid = threadIdx.x, run = tid & 255, mine = tid >> 8;
    const int tq = run & 7, ty = run >> 3;                               // 8 runs of four columns x 32 rows
    const int pair = blockIdx.x, bi = blockIdx.y >> 3, bj = blockIdx.y & 7;
    int ti, tj;
    pair_to_tiles(pair, T, ti, tj);
    const bool diag = ti == tj;
    if (diag && bi > bj) return;
    const bool mirrored = !diag || bi < bj;
    const double Bd = static_cast<double>(B);
    const int64_t tile_elems = TRK_T * TRK_T, stride = static_cast<int64_t>(pairs) * tile_elems;
    const int il = bi * 32 + ty, jl = bj * 32 + 4 * tq;
    const int i = ti * TRK_T + il, j = tj * TRK_T + jl;                  // K % 8 == 0: a run is inside or outside
    const bool live = i < K && j < K;
    const int fc = tid & 63, fq = tid >> 6;                              // folding: column, first range
    const int ft = fc < 32 ? ti : tj, fl = (fc < 32 ? bi : bj) * 32 + (fc & 31), fk = ft * TRK_T + fl;
    const double* fsrc = colsum + static_cast<int64_t>(diag_pair(ft, T)) * TRK_T + fl;
    const int64_t fstride = static_cast<int64_t>(pairs) * TRK_T;
    double cv[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) cv[u] = fq + 4 * PARTS * u < splits ? fsrc[(fq + 4 * PARTS * u) * fstride] : 0.0;
    const double m0 = fk < K ? static_cast<double>(mu_old[fk]) : 0.0;
    double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
    float* dst = sigma + static_cast<int64_t>(i) * K + j;
    // mirrored block: row jl2 of the lower triangle takes column jl2 of this block
    const int jl2 = bj * 32 + ty, il2 = bi * 32 + 4 * tq;
    const int i2 = ti * TRK_T + il2, j2 = tj * TRK_T + jl2;
    const bool live2 = mirrored && mine == 0 && i2 < K && j2 < K;
    float* dst2 = sigma + static_cast<int64_t>(j2) * K + i2;
    v4f old{}, old2{};
    if (live2) old2 = *reinterpret_cast<const v4f*>(dst2);
    if (live) {
        if (mine == 0) old = *reinterpret_cast<const v4f*>(dst);
        const float* src = partial + static_cast<int64_t>(pair) * tile_elems + il * TRK_T + jl;
#pragma unroll 8
        for (int sp = mine; sp < splits; sp += PARTS) {
            const v4f v = *reinterpret_cast<const v4f*>(src + sp * stride);
            s0 += static_cast<double>(v[0]); s1 += static_cast<double>(v[1]);
            s2 += static_cast<double>(v[2]); s3 += static_cast<double>(v[3]);
        }
    }
    double cs = 0.0;
#pragma unroll
    for (int u = 0; u < 8; ++u) cs += cv[u];
#pragma unroll 4
    for (int sp = fq + 32 * PARTS; sp < splits; sp += 4 * PARTS) cs += fsrc[sp * fstride];
    part[fq][fc] = cs;
    if (PARTS > 1 && mine > 0) {
        sums[mine - 1][0][run] = s0; sums[mine - 1][1][run] = s1; sums[mine - 1][2][run] = s2; sums[mine - 1][3][run] = s3;
    }
    __syncthreads();
    if (tid < 64) {
        double t = 0.0;
#pragma unroll
        for (int u = 0; u < 4 * PARTS; ++u) t += part[u][fc];
        const double mb = t / Bd;
        mub[fc] = mb;
        delta[fc] = mb - m0;
        if (diag && bi == bj && fc < 32 && fk < K) mu[fk] = static_cast<float>(m0 + ratio * (mb - m0));
    }
    __syncthreads();
    double c[4] = {0.0, 0.0, 0.0, 0.0};
    if (live && mine == 0) {
        double sv[4] = {s0, s1, s2, s3};
        if (PARTS > 1) {
#pragma unroll
            for (int u = 0; u < PARTS - 1; ++u)
#pragma unroll
                for (int e = 0; e < 4; ++e) sv[e] += sums[u][e][run];
        }
        v4f nw;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            // products of the two columns first: (i, j) and (j, i) then give identical bits
            const double sb = sv[e] - Bd * (mub[ty] * mub[32 + 4 * tq + e]);
            c[e] = sb + coef * (delta[ty] * delta[32 + 4 * tq + e]);
            nw[e] = static_cast<float>(static_cast<double>(old[e]) + c[e]);
        }
        *reinterpret_cast<v4f*>(dst) = nw;
    }
    if (mirrored) {
        if (mine == 0) {
#pragma unroll
            for (int e = 0; e < 4; ++e) tr[ty][4 * tq + e] = c[e];
        }
        __syncthreads();
        if (live2) {
            v4f nw;
#pragma unroll
            for (int e = 0; e < 4; ++e) nw[e] = static_cast<float>(static_cast<double>(old2[e]) + tr[4 * tq + e][ty]);
            *reinterpret_cast<v4f*>(dst2) = nw;
        }
    }
}

size_t tracker_workspace_bytes(int64_t B, int64_t K) { return tracker_plan(B, K).bytes; }

loka_status tracker_update_launch(const void* x, int64_t B, int64_t K, int64_t ld, int64_t n_old, float* mu, float* sigma,
                                  void* workspace, hipStream_t s) {
    const TrackerPlan pl = tracker_plan(B, K);
    uint8_t* ws = static_cast<uint8_t*>(workspace);
    double* colsum = reinterpret_cast<double*>(ws + pl.off_colsum);
    TrackerParams p{};
    p.x = static_cast<const uint16_t*>(x); p.B = B; p.ld = ld; p.K = static_cast<int>(K);
    p.T = pl.T; p.pairs = pl.pairs; p.splits = pl.splits; p.rows_per_split = pl.rows_per_split;
    p.partial = reinterpret_cast<float*>(ws); p.colsum = colsum;
    p.mu = mu; p.mu_old = reinterpret_cast<float*>(ws + pl.off_mu);
    // set on every call (a host-side table write): no process-wide state, and correct on whichever device is current
    LOKA_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(&tracker_scatter_kernel),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(TRK_LDS)));
    tracker_scatter_kernel<<<dim3(pl.pairs * pl.splits), 512, TRK_LDS, s>>>(p);
    const double n_new = static_cast<double>(n_old) + static_cast<double>(B);
    const double ratio = static_cast<double>(B) / n_new, coef = static_cast<double>(n_old) * static_cast<double>(B) / n_new;
    auto merge = [&](auto parts) {
        tracker_merge_kernel<decltype(parts)::value><<<dim3(pl.pairs, 64), 256 * decltype(parts)::value, 0, s>>>(
            p.partial, colsum, p.mu_old, pl.T, pl.pairs, pl.splits, static_cast<int>(K), B, ratio, coef, mu, sigma);
    };
    // Four threads per run where workgroups are few and ranges many (us, one thread -> four: 65536 x 256, 128 ranges, 33.8 -> 32.5,
    // 16384 x 512, 37, 28.1 -> 27.1, 18786 x 456, 42, 28.2 -> 27.7; but 12000 x 512, 32, 28.7 -> 29.1, 8000 x 512, 25, 24.8 -> 25.2,
    // 2000 x 64, 16, 13.5 -> 14.4, and with three column tiles and more 65536 x 768, 41, 64.8 -> 66.8, 32768 x 1024, 25, 56.2 -> 61.5)
    if (pl.T <= 2 && pl.splits >= 32) merge(std::integral_constant<int, 4>{});
    else merge(std::integral_constant<int, 1>{});
    return hipGetLastError() == hipSuccess ? LOKA_OK : LOKA_ERR_HIP;
}

}  // namespace loka
