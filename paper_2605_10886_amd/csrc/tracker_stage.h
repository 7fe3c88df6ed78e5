// Where the elements of a tracker tile lie in LDS on their way out, and which wave stores which: the index arithmetic of
// tracker_scatter_kernel's epilogue (host and device, so that it can be enumerated without a GPU).
//
// A tile of 256 x 256 outputs is 8 x 8 MFMA blocks of 32 x 32; block (a, b) element (R, C) is tile row 8 R + a, tile column
// 8 C + b; two blocks with neighbouring b are a group.  Element r of a lane is R = 8 (r / 4) + 4 h + r % 4, C = c, with
// h = lane / 32 and c = lane % 32.  The tile leaves in two halves of 128 rows (R < 16: r < 8, then R >= 16).
//
// LDS word of (R, C): row 8 (R % 16) + a of 256 words, the four groups side by side in it, position (2 C + b % 2) of the group's
// 64, the upper two groups with their halves exchanged (the two 8-byte reads of the 32 lanes that share a row half then fall
// on different banks).  On diagonal pairs rows 8 R .. 8 R + 7 are rotated by an XOR of 2 R as well, so that the transposed
// writes (lanes = rows 8 C + b) spread over the banks.
#pragma once
#include <hip/hip_runtime.h>

namespace loka {

// A lane's share of the address: element r8 of the half (mirrored: r) is word row + step + (pos ^ key), with step and key
// compile-time constants.  (Kept apart for the kernel: added up in here, the address takes registers that it does not have.)
struct TrkAddr { int row, pos; };

// block (a, b), b even; that of block (a, b + 1) is the word behind it
__host__ __device__ constexpr TrkAddr trk_direct(bool diag, int a, int b, int h, int c) {
    return {(32 * h + a) * 256 + (b >> 1) * 64, (2 * c) ^ ((b >> 2) * 32) ^ (diag ? 8 * h : 0)};
}
__host__ __device__ constexpr int trk_direct_step(int r8) { return (64 * (r8 >> 2) + 8 * (r8 & 3)) * 256; }
__host__ __device__ constexpr int trk_direct_key(bool diag, int r8) { return diag ? 16 * (r8 >> 2) + 2 * (r8 & 3) : 0; }
// the transpose of block (a, b) (diagonal pairs), i.e. block (b, a): elements of the lanes with c / 16 = half, no step
__host__ __device__ constexpr TrkAddr trk_mirror(int a, int b, int h, int c) {
    return {(8 * (c & 15) + b) * 256 + (a >> 1) * 64, (a & 1) ^ ((a >> 2) * 32) ^ (8 * h) ^ (2 * (c & 15))};
}
__host__ __device__ constexpr int trk_mirror_key(int r) { return 16 * (r >> 2) + 2 * (r & 3); }

// Diagonal pairs: the two groups of a wave.  Waves 0..5 multiply the one with the other (acc[t][e], t < 2, is block
// (2 group 0 + t, 2 group 1 + e)), waves 6 and 7 each with itself (acc[t][e] is block (2 g + t % 2, 2 g + e), g = group t / 2).
__host__ __device__ constexpr int trk_group(int wave, int which) { return ((which ? 0x31223331u : 0x20102100u) >> (4 * wave)) & 3; }
__host__ __device__ constexpr bool trk_self(int wave) { return wave >= 6; }
// Whether acc[t][e] is stored, and whether its transpose is: of the waves with two groups both where t < 2, of the others by these
// two.  Every word has one writer: a block below the diagonal is nothing but the transpose of its mirror image (acc[t][0] of odd
// t in waves 6 and 7 is such a block and holds nothing).
__host__ __device__ constexpr bool trk_pair_holds(int t) { return t < 2; }
__host__ __device__ constexpr bool trk_self_stores(int t, int e) { return (t & 1) <= e; }
__host__ __device__ constexpr bool trk_self_mirrors(int t, int e) { return (t & 1) < e; }

}  // namespace loka
