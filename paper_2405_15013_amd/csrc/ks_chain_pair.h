// Two-factor chains of Monarch type in one persistent kernel
// (ks_chain_pair.hip): K_1 = (1, b, b, q), K_2 = (q, b, b, 1), b = 16*BT with
// BT in 1 .. 4, q = 8*NBW with NBW in {1, 2, 4, 8} (paper Section 1 and
// Appendix B.1).  Shared by the kernel, the host planner (ks_host.cpp) and the
// host replay (ks_verify.hip).
//
// K_2, applied first, multiplies each run of b consecutive rows by its own
// block i; K_1 multiplies the rows l*q + j (l < b) by block j.  A workgroup of
// eight wavefronts keeps both factors' values in registers for its whole life
// (wavefront w holds blocks w*NBW .. w*NBW + NBW - 1 of each) and walks over
// batch tiles: the first factor's X operands come straight from global memory
// into registers (those of the next tile while this one is finished), the
// intermediate goes through LDS, and X is read and Y written once.
#pragma once
#include <hip/hip_runtime.h>
#include <cstdint>

namespace ks {

constexpr int kPairWaves = 8;
constexpr int kPairMaxLds = 160 * 1024;

struct PairChain {
  const void* x;
  void* y;
  const void* k1;  // values of K_1 (applied second)
  const void* k2;  // values of K_2 (applied first)
  int batch, tiles;
  int layout, bt, nbw;  // launch only
};

// Batch columns of a tile.  Batch-size-last: one 128-byte line per row.
__host__ __device__ constexpr int pair_cols(int layout, int esize) { return layout == 0 ? 16 : 128 / esize; }
// LDS bytes: the intermediate (batch-size-first: fp32, 16 columns per row;
// batch-size-last: the storage type, 128 bytes per row), and batch-size-first
// the output tile, which takes the intermediate's place when both do not fit.
__host__ __device__ constexpr int pair_t_bytes(int layout, int N) { return N * (layout == 0 ? 64 : 128); }
__host__ __device__ constexpr int pair_y_pitch(int esize, int N) { return N + 16 / esize; }  // elements
__host__ __device__ constexpr int pair_y_bytes(int esize, int N) { return 16 * pair_y_pitch(esize, N) * esize; }
__host__ __device__ constexpr bool pair_y_separate(int esize, int N) {
  return pair_t_bytes(0, N) + pair_y_bytes(esize, N) <= kPairMaxLds;
}
__host__ __device__ constexpr int pair_lds(int layout, int esize, int N) {
  return layout != 0 ? pair_t_bytes(layout, N)
                     : (pair_y_separate(esize, N) ? pair_t_bytes(0, N) + pair_y_bytes(esize, N)
                                                  : (pair_t_bytes(0, N) > pair_y_bytes(esize, N) ? pair_t_bytes(0, N)
                                                                                                 : pair_y_bytes(esize, N)));
}

// Instances: where the values of both factors (2*NBW*BT*BT runs of 4 per lane)
// and a tile's X fit the registers, or miss them by so few that the kernel is
// faster than ks_chain_mfma.hip's all the same: (b, q) = (32, 64) batch-size-first
// in 16 bits spills 17 registers (bf16 at batch 4096, 16384, 24592 23.5 -> 21.7,
// 86.4 -> 51.7, 141.9 -> 81.6 us), (48, 16) in fp32 one (15.6 -> 14.6, 55.4 ->
// 36.5, 83.2 -> 51.7 us).  Batch-size-last only 16-bit types: an fp32
// tile of whole lines ran 0-20 % slower than ks_chain_mfma.hip's.
__host__ __device__ constexpr bool pair_instance(int layout, int esize, int bt, int nbw) {
  return bt >= 1 && bt <= 4 && (nbw == 1 || nbw == 2 || nbw == 4 || nbw == 8) &&
         (layout == 0 ? nbw * bt * bt <= (esize == 4 ? 18 : 32) : esize == 2 && nbw * bt * bt <= 18) &&
         pair_lds(layout, esize, 128 * bt * nbw) <= kPairMaxLds;
}

// Factor values on their way to the registers: a wavefront's blocks of one
// factor are one run of rows of U = b*esize/16 units of 16 bytes, moved to its
// part of LDS by DMA, lane by lane in order, and read from there in the MFMA's
// lane order (16 rows at once, the same unit of each).  Unit u of row r sits at
// position r*U + (u + pair_k_rot(U, r)) % U, which spreads the 16 rows over the
// banks.
__host__ __device__ constexpr int pair_k_shift(int U) {
  return U % 16 == 0 ? 0 : (U % 8 == 0 ? 1 : (U % 4 == 0 ? 2 : (U % 2 == 0 ? 3 : 4)));
}
__host__ __device__ __forceinline__ int pair_k_rot(int U, int r) { return (r & 15) >> pair_k_shift(U); }
__host__ __device__ __forceinline__ int pair_k_pos(int U, int r, int u) {
  const int v = u + pair_k_rot(U, r);
  return r * U + (v >= U ? v - U : v);
}
// Unit (of the run) that belongs at position p.
__host__ __device__ __forceinline__ int pair_k_unit(int U, int p) {
  const int r = p / U, v = p - r * U - pair_k_rot(U, r);
  return r * U + (v < 0 ? v + U : v);
}
// A wavefront's part of LDS (bytes, whole DMA instructions) and the row tiles
// (16 rows) of its run that it holds at a time.
__host__ __device__ constexpr int pair_k_area(int lds) { return lds / kPairWaves / 1024 * 1024; }
__host__ __device__ constexpr int pair_k_tiles(int lds, int U, int total) {
  int g = 0;
  while (g < total && ((g + 1) * 256 * U + 1023) / 1024 * 1024 <= pair_k_area(lds)) ++g;
  return g;
}

// LDS row of intermediate row m.  The second factor reads rows
// (4*LP*c + LP*g + t) * q + j, g = 0 .. 3 at once; the first writes rows
// (multiple of 16) + 4 g + r.  A row is a quarter (batch-size-first) or half of
// the 64 banks: the low two bits of the LDS row, which pick the part, are mixed
// with bits 2, 3 and sh, sh + 1 of m, 2^sh = q * LP, so that both accesses
// touch all parts.
__host__ __device__ __forceinline__ int pair_row(int m, int sh) {
  return (m & ~3) | ((m ^ (m >> 2) ^ (m >> sh)) & 3);
}
// The same for the two accesses, as the kernel computes it in bytes of rows of
// `rb` bytes: a per-lane part and a wave-uniform part.
//   write of row m0 + 4g + r (m0 a multiple of 16)
__host__ __device__ __forceinline__ int pair_write_lane(int rb, int g, int r) { return rb * (4 * g + (r ^ g)); }
__host__ __device__ __forceinline__ int pair_write_mix(int rb, int m0, int sh) { return rb * ((m0 >> sh) & 3); }
//   read of row m0 + LP*g*q (m0 = (4*LP*c + t) * q + j)
__host__ __device__ __forceinline__ int pair_read_lane(int rb, int LP, int q, int g) { return rb * (LP * q * g + g); }
__host__ __device__ __forceinline__ int pair_read_mix(int rb, int m0) { return rb * ((m0 ^ (m0 >> 2)) & 3); }
// LDS byte of the row: rb * (m0 without its low bits for the read) + (lane ^ mix).

}  // namespace ks
