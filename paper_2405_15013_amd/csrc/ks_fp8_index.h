// Index arithmetic of the FP8 kernel for long batch rows (ks_fp8.hip,
// ks_fp8_rows_kernel), shared by the kernel and by the host-side plan verifier.
//
// An item is a wavefront's walk: the 16 * mt output rows k0 .. of block row i
// for all 8 values of j, over the batch tiles (16 rows) bt0, bt0 + nseg, ...
#pragma once
#include "ks_masked_index.h"

namespace ks {

struct Fp8Rows {
  int mt;       // 16-row output tiles per wavefront (1 or 2)
  int kgroups;  // b / (16 * mt)
  int nbt;      // batch tiles
  int nseg;     // walks over the batch tiles
  int items;    // a * nseg * kgroups
};

struct Fp8Walk {
  int i, k0, bt0;
};

// Wavefronts per SIMD that each instance is compiled for: as many as hold its
// K operands, two tiles of X and the accumulators of 16 rows without spilling.
constexpr int fp8_rows_waves(int mt, int nch, bool half) {
  return mt * nch == 4 ? 2 : (mt * nch == 2 && !(mt == 2 && half) ? 3 : 4);
}

// True when the call takes the long-row kernel: d = 8, whole 16-row tiles of b,
// 16-byte pieces of X and Y, 8-byte K operands that fit the registers
// (c <= 64).  All walks are equally long but for one tile, and are no more
// than the chip holds at a time.  Left to ks_fp8_kernel: calls of one batch tile
// per walk with the most K operands (two tiles of b, c of 64), which a walk of
// one tile does not earn back (34 calls of batch 1 to 4096: 1.02 of its time
// in the mean, up to 1.13; c of 56 and less 0.76-0.98, longer walks 0.42-0.91).
// d other than 8 and c above 64 have not been tried in this form.
inline bool fp8_rows(const Problem& p, Fp8Rows* t) {
  if (p.dtype != FP8 || p.layout != BSF || p.d != 8 || p.b % 16 || p.c % 8 || p.c > 64 || p.align < 16) return false;
  if (reinterpret_cast<uintptr_t>(p.kv) % 8) return false;
  t->mt = p.b % 32 == 0 ? 2 : 1;
  t->kgroups = p.b / (16 * t->mt);
  t->nbt = (p.batch + 15) / 16;
  const int64_t walks = (int64_t)p.a * t->kgroups;
  const int nch = (p.c + 31) / 32;
  const int64_t resident = 256 * 4 * fp8_rows_waves(t->mt, nch, p.c - 32 * (nch - 1) <= 16);  // 256 CUs of 4 SIMDs
  const int64_t most = walks < resident ? resident / walks : 1;
  const int64_t tiles = (t->nbt + most - 1) / most;  // of a walk
  if (tiles == 1 && t->mt == 2 && p.c > 56) return false;
  t->nseg = (int)((t->nbt + tiles - 1) / tiles);
  if (walks * t->nseg > 0x7fffffff - 3) return false;
  t->items = (int)(walks * t->nseg);
  return true;
}

// k-group fastest (the wavefronts of a workgroup read the same rows of X), then
// walk, then i.
KS_MHD Fp8Walk fp8_rows_item(const Fp8Rows& t, int mt, int item) {
  Fp8Walk it;
  int rest = item;
  it.k0 = 16 * mt * (rest % t.kgroups);
  rest /= t.kgroups;
  it.bt0 = rest % t.nseg;
  it.i = rest / t.nseg;
  return it;
}

// Batch row of lane column n of tile bt (the last row beyond the batch).
KS_MHD int fp8_rows_row(const Problem& p, int bt, int n) {
  const int row = 16 * bt + n;
  return row < p.batch ? row : p.batch - 1;
}

// Byte offset in a row of X of piece g of the 64-byte run of values 8q .. 8q + 7
// (values beyond c: those of the block's first run).
KS_MHD int fp8_rows_x_piece(const Problem& p, int i, int q, int g) {
  return (i * p.c + (8 * q < p.c ? 8 * q : 0)) * 8 + 16 * g;
}

// Bytes of a row of the output tile in LDS (16 of padding: the 16 lanes of a
// row column write all banks once).
KS_MHD constexpr int fp8_rows_pitch(int mt) { return 256 * mt + 16; }

// Store q of a lane: 16-byte unit u (8 outputs of row k0 + u) of batch row
// `row` of the tile (the last row of the batch instead of those beyond it).
KS_MHD int fp8_rows_unit(int mt, int q, int lane) { return (64 * q + lane) & (16 * mt - 1); }
KS_MHD int fp8_rows_unit_row(const Problem& p, int mt, int bt, int q, int lane) {
  const int row = (64 * q + lane) / (16 * mt), last = p.batch - 1 - 16 * bt;
  return row < last ? row : last;
}

}  // namespace ks
