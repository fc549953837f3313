// Index arithmetic of the masked kernels for blocks, batches and buffers of any
// size and alignment (ks_ragged.h), shared with the host-side plan verifier.
//
// Both work on 16 x 16 MFMA tiles (lane (n, g) = (lane % 16, lane / 16), LP
// values of l per lane and chunk, paper Section 4.1, Algorithm 2) of which the
// last ones of b, c and the batch may be cut short: rows k >= b repeat row b - 1
// and are not stored, values l >= c are zero on both sides.  Memory is accessed
// in vectors whatever the alignment (the hardware takes element-aligned
// vectors); where a vector would cross an end it is moved back or taken apart.
//
//  * batch-size-last: one wavefront per item, a batch group of 16*V entries of
//    one (i, j) and 16*MT rows k.  Lane column n covers V consecutive entries;
//    the last one of the batch is moved back to end there (its first `shift`
//    entries belong to the column before and are not stored).
//  * batch-size-first: a workgroup of four wavefronts takes 16*RG batch rows of
//    one i and KB rows k.  The runs X[beta, i*c*d .. (i+1)*c*d) go to LDS, the
//    wavefronts take (j, 16*MT rows) items in turn, the outputs leave through
//    an LDS tile as runs Y[beta, (i*b + k0)*d .. ).
#pragma once
#include <hip/hip_runtime.h>
#include <cstdint>

#include "ks_divide.h"
#include "ks_internal.h"

#define KS_RHD __host__ __device__ __forceinline__

namespace ks {

struct RaggedTile {
  int items;             // batch-size-last: wavefront items; batch-size-first: workgroups
  int kgroups;           // batch-size-last: ceil(b / 16 MT); batch-size-first: splits of b
  int nbt;               // batch groups
  int kb;                // batch-size-first: rows k per workgroup (a multiple of 16; the last item of 16 MT rows may be cut short)
  int upr;               // batch-size-first: 16-byte units per run of X
  int xpitch, ypitch;    // batch-size-first: LDS row pitches in bytes
  int lds;
  uint32_t mkg, mnbt, md, mupr;
  int skg, snbt, sd, supr;
};

KS_RHD constexpr int ragged_lp(int esize) { return esize == 4 ? 4 : 8; }

// LDS row pitch for `bytes`: whole 16-byte units, an odd number of them, so that
// the same element of 16 rows lies in 16 different banks.
KS_RHD int ragged_pitch(int bytes) {
  const int u = (bytes + 15) / 16;
  return 16 * (u | 1);
}

inline RaggedTile ragged_bsl_tile(const Problem& p, int V, int MT) {
  RaggedTile t{};
  t.kgroups = (p.b + 16 * MT - 1) / (16 * MT);
  t.nbt = (p.batch + 16 * V - 1) / (16 * V);
  t.items = (int)((int64_t)t.nbt * p.a * p.d * t.kgroups);
  div_magic((uint32_t)t.kgroups, &t.mkg, &t.skg);
  div_magic((uint32_t)t.nbt, &t.mnbt, &t.snbt);
  div_magic((uint32_t)p.d, &t.md, &t.sd);
  return t;
}
inline RaggedTile ragged_bsf_tile(const Problem& p, int RG, int MT, int kb) {
  RaggedTile t{};
  const int S = p.dtype == F32 ? 4 : 2;
  t.kb = kb;
  t.kgroups = (p.b + kb - 1) / kb;
  t.nbt = (p.batch + 16 * RG - 1) / (16 * RG);
  t.items = (int)((int64_t)t.nbt * p.a * t.kgroups);
  t.upr = (p.c * p.d * S + 15) / 16;
  t.xpitch = ragged_pitch(p.c * p.d * S);
  t.ypitch = ragged_pitch(kb * p.d * S);
  t.lds = 16 * RG * (t.xpitch + t.ypitch);
  div_magic((uint32_t)t.kgroups, &t.mkg, &t.skg);
  div_magic((uint32_t)t.nbt, &t.mnbt, &t.snbt);
  div_magic((uint32_t)p.d, &t.md, &t.sd);
  div_magic((uint32_t)t.upr, &t.mupr, &t.supr);
  return t;
}

struct RItem {
  int i, j, k0, bt;
};
// k-group fastest (neighbours share X), then the batch group, then (BSL) j, then i.
KS_RHD RItem ragged_item(const Problem& p, const RaggedTile& t, int item, int rows) {
  RItem it;
  const uint32_t q1 = div_fast((uint32_t)item, t.mkg, t.skg);
  it.k0 = (int)((uint32_t)item - q1 * (uint32_t)t.kgroups) * rows;
  const uint32_t q2 = div_fast(q1, t.mnbt, t.snbt);
  it.bt = (int)(q1 - q2 * (uint32_t)t.nbt);
  if (p.layout == BSL) {
    const uint32_t q3 = div_fast(q2, t.md, t.sd);
    it.j = (int)(q2 - q3 * (uint32_t)p.d);
    it.i = (int)q3;
  } else {
    it.j = 0;
    it.i = (int)q2;
  }
  return it;
}

// Batch-size-last: first batch entry of lane column n as loaded (the vector
// lies inside the batch), and how many of its entries another column stores
// (V or more: all of them).  Needs batch >= V.
KS_RHD int ragged_col(const Problem& p, const RItem& it, int V, int n) {
  const int col = it.bt * 16 * V + V * n, last = p.batch - V;
  return col < last ? col : last;
}
KS_RHD int ragged_shift(const Problem& p, const RItem& it, int V, int n) {
  return it.bt * 16 * V + V * n - ragged_col(p, it, V, n);
}
// First element of K row `row` of block (i, j), rows beyond b repeating the last.
KS_RHD int64_t ragged_k_row(const Problem& p, int i, int j, int row) {
  return ((int64_t)(i * p.d + j) * p.b + (row < p.b ? row : p.b - 1)) * p.c;
}

}  // namespace ks
