// Definitions shared by the GEMM translation units (gemm.hip, gemm_panel32.hip).
#pragma once

#include "common.h"

namespace loka {

enum { EPI_ROW_IN_TILE = 0, EPI_PARTIAL_STATS = 1, EPI_PANEL_SYNC = 2, EPI_SPLITK = 3 };

struct GemmParams {
    const uint8_t* X;      // [batch][M][KB] bytes (KB = K for FP8, 2K for BF16)
    const uint8_t* W;      // [batch][N][KB]
    int M, N, KB;
    int batch;
    int64_t strideX, strideW;   // bytes between problems
    int64_t strideO;            // elements between problems (O, Y)
    const float* sx;
    const float* sw;
    int64_t strideSx, strideSw; // scales between problems
    int x_mode, w_mode;
    const uint16_t* gamma;
    const uint16_t* beta;
    uint16_t* out;
    uint8_t* outq;         // FP8 output instead of `out`: e4m3 codes [batch][M][N] ...
    float* outs;           // ... and their row scales [batch][M]
    const uint16_t* xb;    // fused quantization (streaming kernel): bf16 X [batch][M][K] instead of X / sx ...
    float* sx_out;         // ... and, optionally, where the row scales it computes are written [batch][M]
    int qpro;              // quantize prologue (streaming kernel): xb is quantized row by row into X / sx (written, then read back)
    float* y;
    int norm;              // loka_norm
    int block_n, act;      // LOKA_NORM_BLOCKNORM group width; loka_act
    float eps;
    int tiles_m, tiles_n;
    int ksplit, k_per_split;   // EPI_SPLITK: number of K ranges, and 128-byte K steps per range; part = [ksplit][batch][M][N] fp32
    float* part;           // EPI_PARTIAL_STATS / EPI_PANEL_SYNC: [batch][M][tiles_n * 2] (mean, M2) or (0, sumsq)
                           // (gemm_panel32.hip: [batch][tiles_m][tiles_n][256] such pairs, then as many (min, max) pairs)
    // EPI_PANEL_SYNC, the exchange between the workgroups of a row panel (see panel_publish_and_wait):
    unsigned long long* flags;   // [exchanges][batch * tiles_m][tiles_n] arrival words; a tile has arrived when its word == nonce
    unsigned long long* header;  // [0] nonce of the last launch on this workspace, [1] nonce of the last launch with a wait that ran out
    unsigned long long nonce;    // launch-unique, never 0
    unsigned long long expect;   // value the waits look for: nonce (nonce + 2, which nobody writes, in the error-path test)
    unsigned spin_limit;
};

// Output column of MFMA tile ti, element i, for a lane of group q (= lane / 16), relative to the wave's
// first column: (ti / 2) * 32 + q * 8 + (ti % 2) * 4 + i.  A lane owns 8 consecutive columns per tile pair,
// and the four lane groups of a row together cover 32 consecutive columns: one 16-byte bf16 store per
// lane writes full 64-byte runs per row.
__host__ __device__ constexpr int coff_of(int ti) { return (ti >> 1) * 32 + (ti & 1) * 4; }

// Workgroups are dealt to the 8 XCDs round-robin (block b runs on XCD b % 8), and each XCD has an L2 of its own.  This
// renumbers G blocks so that every XCD works on one contiguous range of logical ids (any G: the first G % 8 XCDs have one
// more): neighbours in the id order, which share operands, then find them in the same L2.
__host__ __device__ constexpr int xcd_contiguous(int b, int G) {
    const int x = b & 7, r = G & 7;
    return x * (G >> 3) + (x < r ? x : r) + (b >> 3);
}

// Whether a persistent launch of G workgroups whose tiles_n neighbours wait for one another may be renumbered so.
// An XCD starts its share of a launch in order, on 32 CUs.  Of a launch that it has not started in full it holds at most
// tiles_n - 1 workgroups of an unfinished panel, so while L such launches share the chip and L (tiles_n - 1) < 32, XCD 0 gets
// through its share, then XCD 1, whose first panel may begin on XCD 0, and so on: nobody's wait can fill an XCD.
// That covers four launches up to 8 tiles and two up to 16 (there only without a panel on two XCDs: its workgroups would
// start first on one and last on the other).  Wider rows keep launch order, which gives every XCD a few workgroups of each
// panel and is the faster one there as well: 8192 x 8192 x 2048 (M x N x K) 167 -> 150 us, 4096 x 5120 x 2048 72.8 -> 67.9,
// 8192 x 16384 x 512 193 -> 185; slowest the other way 3000 x 5120 x 512 22.3 -> 23.2, 3000 x 4096 x 512 19.8 -> 20.4.
__host__ __device__ constexpr bool panels_may_spread(int G, int tiles_n) {
    return tiles_n <= 8 || (tiles_n <= 16 && G % 8 == 0 && (G / 8) % tiles_n == 0);
}

// The numbering of the panel schedule's tiles below 256 x 256 (up to two workgroups per CU; rows of up to 8 tiles): a panel's
// workgroups one behind the other on one XCD, the panels dealt to the XCDs in turn; fewer than 8 panels may be left, whose
// workgroups follow in equal shares.  Of one launch an XCD then holds at most 7 workgroups that wait for others still to be
// started: of a panel that it has begun, or, after the last whole panel, its share of those left (7 panels / 8).  So four
// launches side by side (28 of at least 32 slots) always start in full; in launch order, where a panel lies on tiles_n
// XCDs, two launches that two XCDs begin in different order can fill both with workgroups that wait for each other.
// (A share of consecutive panels per XCD puts a last round that is partly full on a few XCDs: 3000 x 2048 x 512 on 32 x 256
// tiles 22.0 -> 26.6 us.  Dealt in turn, geometric mean over 81 shapes against launch order: 32 x 256 0.995, 64 x 256 1.013,
// 128 x 128 0.980.)
__host__ __device__ constexpr int panel_per_xcd(int b, int G, int tiles_n) {
    const int whole = G / (8 * tiles_n) * (8 * tiles_n);
    if (b >= whole) return whole + xcd_contiguous(b - whole, G - whole);
    const int i = b >> 3;
    return ((i / tiles_n) * 8 + (b & 7)) * tiles_n + i % tiles_n;
}

// Loads of block scales that a wave of the large-tile kernel requests at the start of K step k, for step k + 1: W's scale and
// X's four, or (quad: a lane holds four K blocks' scales of X) W's alone in three steps of four.  What may stay in flight
// where the step needs X(k + 1) and W(k + 1) is these and the 4 loads of X(k + 2), the only ones requested behind W(k + 1).
__host__ __device__ constexpr int panel32_scale_loads(bool quad, int k) { return quad && ((k + 1) & 3) != 0 ? 1 : 5; }

// Tile t of a tiles_m x tiles_n grid in bands of 8 tile rows, walked column by column inside a band: 64 neighbours in the
// order cover an 8 x 8 block of tiles and read 8 + 8 operand strips, where plain row order would read 1 + 64.
__device__ __forceinline__ void banded_tile(int t, int tiles_m, int tiles_n, int& tm, int& tn) {
    const int band = t / (8 * tiles_n), r = t - band * 8 * tiles_n;
    const int rows = tiles_m - band * 8 < 8 ? tiles_m - band * 8 : 8;
    tn = r / rows;
    tm = band * 8 + r - tn * rows;
}

// Workgroup barrier that orders LDS traffic only: LDS reads/writes issued before it are complete, but
// global loads (including the loads that stream the next stage into LDS) stay in flight across it.
// Completion of those is awaited explicitly (s_waitcnt vmcnt) where a stage is about to be read.
// Written as an instruction sequence: a fence builtin on the LDS address space makes the compiler wait for
// vmcnt(0) as well whenever loads-to-LDS are outstanding, which would expose their full latency each phase.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

// Waits until at most N_ of this wave's vector-memory operations are outstanding (6-bit count, split
// over two fields of the instruction's immediate); the LDS and scalar counters are left alone.
template <int N_>
__device__ __forceinline__ void wait_vmcnt() {
    __builtin_amdgcn_s_waitcnt(0x0F70 | (N_ & 15) | ((N_ >> 4) << 14));
}

// Sums over lanes l, l ^ 32 and over l, l ^ 16, l ^ 32, l ^ 48 (identical bits on all of them), by the half and row swaps of the
// vector unit: no LDS round trip, which a shuffle is.
__device__ __forceinline__ float half_lanes_sum(float v) {
    const u32_pair r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(r.x) + __uint_as_float(r.y);
}
__device__ __forceinline__ float half_lanes_max(float v) {
    const u32_pair r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __builtin_fmaxf(__uint_as_float(r.x), __uint_as_float(r.y));
}
__device__ __forceinline__ float row_lanes_sum(float v) {
    const u32_pair r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return half_lanes_sum(__uint_as_float(r.x) + __uint_as_float(r.y));
}

// Chan's pairwise merge of (count, mean, M2).
__device__ __forceinline__ void merge_stats(float& n, float& mean, float& m2, float nb, float mb, float m2b) {
    const float nn = n + nb;
    if (nb > 0.f) {
        const float d = mb - mean;
        const float f = nb * __builtin_amdgcn_rcpf(nn);   // nn > 0 here; 1-ulp reciprocal (an IEEE divide costs ~300 cycles)
        mean = mean + d * f;
        m2 = m2 + m2b + d * d * n * f;
        n = nn;
    }
}

// The lane's number, made where it is asked for: neither the thread id is kept in a register for it nor what is derived from it.
__device__ __forceinline__ int lane_id() {
    int l;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
    return l;
}

// The exchange between the tiles_n workgroups that share a row panel (Section 3.2, Case 2: a row wider than a
// workgroup's tile).  Called by every thread of the workgroup after its per-row records have been STORED with
// device-coherent (agent-scope atomic, write-through) stores:
//   1. every wave waits until its own stores have been acknowledged (s_waitcnt vmcnt(0): a store is acknowledged once
//      it is visible at the scope it was issued with, here the device), then the workgroup barrier: all records of
//      this tile are visible device-wide;
//   2. wave 0 stores the tile's arrival word (= the launch's nonce; device-coherent) - program order after 1 - and polls
//      the panel's tiles_n arrival words (lanes = tiles; device-coherent loads that bypass this XCD's caches) until all
//      equal `expect`, sleeping between polls, for at most spin_limit polls;
//   3. barrier; the caller's threads then read the other tiles' records with device-coherent loads, issued after the
//      poll that saw every arrival word (loads are not issued early on this hardware, and they bypass the non-coherent
//      caches), so they return what was stored before step 2 of the publishing workgroup.
// No L2-wide write-back or invalidate is involved: the records and words are the only data that cross workgroups.
// Arrival words are compared with a nonce instead of counted, so nothing has to be zeroed between launches: a stale
// or uninitialised word never equals a fresh 64-bit nonce.
// Returns false when the wait ran out (never when all tiles_n workgroups are resident, which the launch arranges):
// the launch's nonce is then recorded in header[1] and the caller poisons the rows of its tile.
// `lds_word` is one LDS word the workgroup does not otherwise use during the call; first_wave: this is wave 0.
__device__ __forceinline__ bool panel_publish_and_wait(const GemmParams& p, unsigned long long* words, int tn, int tiles_n,
                                                       int* lds_word, bool first_wave) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // (with the clobber the record stores stay in front of it)
    __syncthreads();
    if (first_wave) {
        const int lane = lane_id();                       // (opaque: addresses derived from it are not hoisted out of the tile loop)
        // (the two 64-bit values restart from the scalar registers here: taken from the parameter block directly, the
        // compiler moves them into vector registers once, before the tile loop, and spills them through the main loop)
        unsigned n_lo = static_cast<unsigned>(p.nonce), n_hi = static_cast<unsigned>(p.nonce >> 32);
        unsigned e_lo = static_cast<unsigned>(p.expect), e_hi = static_cast<unsigned>(p.expect >> 32);
        asm volatile("; arrival values" : "+s"(n_lo), "+s"(n_hi), "+s"(e_lo), "+s"(e_hi));
        const unsigned long long nonce = (static_cast<unsigned long long>(n_hi) << 32) | n_lo;
        const unsigned long long expect = (static_cast<unsigned long long>(e_hi) << 32) | e_lo;
        if (lane == 0) __hip_atomic_store(words + tn, nonce, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        unsigned spins = 0;
        bool failed = false;
        for (;;) {
            bool here = true;
            for (int t = lane; t < tiles_n; t += 64)
                here = here && __hip_atomic_load(words + t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == expect;
            if (__builtin_amdgcn_ballot_w64(!here) == 0) break;
            if (++spins > p.spin_limit) { failed = true; break; }
            __builtin_amdgcn_s_sleep(2);      // (measured at 32768 x 4096 x 4096: 16 costs 2 % of the kernel, 0 gains nothing more)
        }
        if (lane == 0) {
            if (failed) __hip_atomic_store(p.header + 1, nonce, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            *lds_word = failed ? 1 : 0;
        }
    }
    __syncthreads();
    return *lds_word == 0;
}

}  // namespace loka
