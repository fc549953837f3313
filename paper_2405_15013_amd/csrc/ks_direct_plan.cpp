// Planner and launcher of the register-direct MFMA kernels (ks_direct.h).
//
// A plan fixes the vector width V (along the batch in BSL: 8 elements for
// 16-bit storage when the batch allows it, else 4; the j-run min(d, 4) in
// BSF), the number MT of 16-row M-tiles per wavefront,
// and the wavefronts per workgroup.  MT trades X re-reads (b / (16*MT)
// wavefronts read the same X tile) against registers and parallelism.
#include "ks_direct_index.h"
#include "ks_internal.h"
#include "ks_masked_index.h"
#include "ks_ragged_index.h"

namespace ks {

hipError_t launch_direct_f32(const Problem& p, const DirectTile& t, int V, bool strided, int mt, unsigned grid,
                             hipStream_t s);
hipError_t launch_direct_bf16(const Problem& p, const DirectTile& t, int V, bool strided, int mt, unsigned grid,
                              hipStream_t s);
hipError_t launch_direct_f16(const Problem& p, const DirectTile& t, int V, bool strided, int mt, unsigned grid,
                             hipStream_t s);
hipError_t launch_direct_f32_epi(const Problem& p, const DirectTile& t, int V, bool strided, int mt, unsigned grid,
                                 hipStream_t s);
hipError_t launch_direct_bf16_epi(const Problem& p, const DirectTile& t, int V, bool strided, int mt, unsigned grid,
                                  hipStream_t s);
hipError_t launch_direct_f16_epi(const Problem& p, const DirectTile& t, int V, bool strided, int mt, unsigned grid,
                                 hipStream_t s);
hipError_t launch_ragged_f32(const Problem& p, const RaggedTile& t, int V, int MT, hipStream_t s);
hipError_t launch_ragged_bf16(const Problem& p, const RaggedTile& t, int V, int MT, hipStream_t s);
hipError_t launch_ragged_f16(const Problem& p, const RaggedTile& t, int V, int MT, hipStream_t s);
hipError_t launch_masked_f32(const Problem& p, const MaskedTile& t, int V, unsigned grid, hipStream_t s);
hipError_t launch_masked_bf16(const Problem& p, const MaskedTile& t, int V, unsigned grid, hipStream_t s);
hipError_t launch_masked_f16(const Problem& p, const MaskedTile& t, int V, unsigned grid, hipStream_t s);

// Largest MT instantiated for (storage size, layout, V); keep in sync with
// direct_mt_max() in ks_direct.h.
static int mt_max(int esize, int layout, int V) {
  return esize == 4 ? ((layout == BSL || V <= 2) ? 4 : 2) : ((layout == BSL || V <= 2) ? 4 : 2);
}

DirectTile direct_tile(const Problem& p, const Plan& pl) {
  DirectTile t;
  const int V = pl.vec, MT = pl.waves_m;
  t.kgroups = p.b / (16 * MT);
  t.jgroups = p.layout == BSL ? p.d : p.d / V;
  const int span = p.layout == BSL ? 16 * V : 16;
  t.nbt = (p.batch + span - 1) / span;
  t.items = t.nbt * p.a * t.jgroups * t.kgroups;
  t.waves = (int)pl.block / 64;
  div_magic((uint32_t)t.kgroups, &t.mkg, &t.skg);
  div_magic((uint32_t)t.nbt, &t.mnbt, &t.snbt);
  div_magic((uint32_t)t.jgroups, &t.mjg, &t.sjg);
  return t;
}

bool plan_direct(const Problem& p, bool al16, Plan* pl) {
  if (!al16 || p.b % 16 || p.c % 16) return false;
  const int s = p.dtype == F32 ? 4 : 2;
  const int vec = 4;  // kDirectVec in ks_direct.h
  int V;
  bool strided = false;
  if (p.layout == BSL) {
    // 16-bit storage: 8 batch entries per lane (16-byte loads and stores)
    // when the batch allows it (kDirectVecBsl16 in ks_direct.h).
    V = (s == 2 && p.batch % 8 == 0) ? 8 : vec;
    if (p.batch % V) return false;
  } else {
    V = p.d < vec ? p.d : vec;
    if (V != 1 && V != 2 && V != 4) return false;
    if (p.d % V) return false;
    strided = V < p.d;
  }
  const int kt = p.b / 16;  // M-tiles per block
  const int span = p.layout == BSL ? 16 * V : 16;
  const int64_t nbt = (p.batch + span - 1) / span;
  const int64_t per_k = nbt * p.a * (p.layout == BSL ? p.d : p.d / V);
  // Largest MT that still leaves >= 768 wavefronts (three per CU); otherwise
  // the MT giving the most wavefronts.  Fewer k-groups mean fewer re-reads of
  // each X tile, which measured worth more than extra wavefronts down to
  // about three per CU.
  int best = 0;
  for (int mt = mt_max(s, p.layout, V); mt >= 1; --mt) {
    if (kt % mt) continue;
    best = mt;
    if (per_k * (kt / mt) >= 768) break;
  }
  const int64_t items = per_k * (kt / best);
  // Four wavefronts per workgroup at every size: consecutive items (the
  // k-groups of one X tile first) share a CU's caches, and spreading small
  // problems over more, smaller workgroups measured slower.
  const int waves = 4;
  const int64_t grid = (items + waves - 1) / waves;
  if (items > 0x7fffffff || grid > 0x7fffffff) return false;
  pl->variant = V_DIRECT;
  pl->vec = V;
  pl->unroll = strided ? 1 : 0;
  pl->waves_m = best;
  pl->waves_n = kt / best;
  pl->bt = span;
  pl->jg = p.layout == BSL ? 1 : V;
  pl->lds_bytes = 0;
  pl->block = 64u * waves;
  pl->grid = (unsigned)grid;
  pl->xcd_remap = 0;
  return true;
}

// Masked kernels: blocks that the other MFMA kernels cannot run and that are not
// small enough for the VALU kernels (valu_pays in ks_host.cpp).  Batch-size-last,
// and batch-size-first rows that fit LDS and are enough to pay there: the kernels
// of ks_ragged.h (plan field unroll = 1).  Other batch-size-first rows: the
// register kernel of ks_masked.h, with the access width V that d and the
// buffers' alignment allow.
int masked_vec(const Problem& p) {
  const int s = p.dtype == F32 ? 4 : 2;
  int V = 4;
  for (; V > 1; V /= 2) {
    if (p.d % V) continue;
    if (V * s >= 8 && p.align % (V * s)) continue;  // vector accesses need their alignment
    // 8-byte pieces measured slower than element pieces (fp32 (6,64,16,8) at
    // batch 25088: 2.0 ms with 8-byte pieces, 0.68 ms with 4-byte ones)
    if (V * s == 8) continue;
    break;
  }
  return V;
}

// Row tiles per wavefront: the most of mtmax, .., 1 that pad b's 16-row tiles
// by at most a quarter and leave `least` items.
template <typename F>
int ragged_mt(int KT, int mtmax, int64_t least, F items) {
  for (int mt = mtmax; mt > 1; mt /= 2) {
    const int kg = (KT + mt - 1) / mt;
    if (4 * (kg * mt - KT) <= KT && items(kg) >= least) return mt;
  }
  return 1;
}

bool plan_ragged_bsl(const Problem& p, Plan* pl) {
  const int S = p.dtype == F32 ? 4 : 2, vmax = 16 / S, KT = (p.b + 15) / 16;
  // 16-byte vectors along the batch, narrower where 16 columns of them would hold
  // the whole batch more than once, and where they leave fewer than 512 wavefronts
  // of one row tile (two per CU): the call is then one wavefront's latency, which
  // narrower vectors shorten.  Of 1500 calls (batch 1 to 3000) vectors of half and
  // a quarter of 16 bytes took 0.83 and 0.71-0.81 of the time below 256
  // wavefronts, 0.84-0.9 and 0.81-0.94 below 512, 0.96-1.03 and 0.97-1.11 from
  // there on.
  auto groups_of = [&](int v) { return (int64_t)((p.batch + 16 * v - 1) / (16 * v)) * p.a * p.d; };
  int V = 1;
  while (V < vmax && 16 * V < p.batch) V *= 2;
  while (V > 1 && groups_of(V) * KT < 512) V /= 2;
  const int64_t groups = groups_of(V);
  const int MT = ragged_mt(KT, V == 8 ? 2 : 4, 1024, [&](int kg) { return groups * kg; });
  if ((groups * ((KT + MT - 1) / MT) + 3) / 4 > kMaxGrid256) return false;
  const RaggedTile t = ragged_bsl_tile(p, V, MT);
  pl->variant = V_MASKED;
  pl->unroll = 1;
  pl->vec = V;
  pl->waves_m = MT;
  pl->waves_n = t.kgroups;
  pl->bt = 16 * V;
  pl->jg = 1;
  pl->lds_bytes = 0;
  pl->block = 256;
  pl->grid = (unsigned)((t.items + 3) / 4);
  pl->xcd_remap = 0;
  return true;
}

// Batch-size-first: two row groups where that leaves a workgroup per CU and
// LDS for two of them per CU, and b split until there are enough workgroups
// (each split reads the X rows again, from L2).  Rows of Y that do not fit as a
// whole keep the register kernel, also where a split of b would fit (not timed).
constexpr int kRaggedMaxLds = 160 * 1024;  // ks_ragged.h
bool plan_ragged_bsf(const Problem& p, Plan* pl) {
  const int S = p.dtype == F32 ? 4 : 2, KT = (p.b + 15) / 16;
  if ((int64_t)p.d * (p.b > p.c ? p.b : p.c) * S > kRaggedMaxLds) return false;
  int best_rg = 0, best_kt = 0;
  int64_t best_score = -1;
  for (int rg = 2; rg >= 1; --rg)
    for (int ks = 1; ks <= KT; ++ks) {
      const int kt = (KT + ks - 1) / ks;
      const RaggedTile t = ragged_bsf_tile(p, rg, 1, 16 * kt);
      if (t.lds > kRaggedMaxLds) continue;
      const int64_t wgs = (int64_t)t.nbt * p.a * t.kgroups;
      if (wgs > kMaxGrid256) continue;
      // enough workgroups, then room for two per CU, then fewer reads of K, then of X
      const int64_t score = ((wgs < 512 ? wgs : 512) << 20) + (t.lds <= kRaggedMaxLds / 2 ? 1 << 16 : 0) + (rg << 12) + kt;
      if (score > best_score) {
        best_score = score;
        best_rg = rg;
        best_kt = kt;
      }
    }
  if (best_rg == 0) return false;
  const int MT = ragged_mt(best_kt, 4, 4, [&](int kg) { return (int64_t)kg * p.d; });
  const RaggedTile t = ragged_bsf_tile(p, best_rg, MT, 16 * best_kt);
  pl->variant = V_MASKED;
  pl->unroll = 1;
  pl->vec = best_rg;
  pl->waves_m = MT;
  pl->waves_n = t.kgroups;
  pl->kgw = best_kt;
  pl->bt = 16 * best_rg;
  pl->jg = 1;
  pl->lds_bytes = t.lds;
  pl->block = 256;
  pl->grid = (unsigned)t.items;
  pl->xcd_remap = 0;
  return true;
}

RaggedTile ragged_tile_of(const Problem& p, const Plan& pl) {
  return p.layout == BSL ? ragged_bsl_tile(p, pl.vec, pl.waves_m)
                         : ragged_bsf_tile(p, pl.vec, pl.waves_m, 16 * pl.kgw);
}

// Batch-size-first, register kernel: one wavefront per (batch tile, j-group, 16
// rows), however few batch rows there are.
bool plan_masked_reg(const Problem& p, Plan* pl) {
  if (p.layout != BSF) return false;
  const int V = masked_vec(p);
  const MaskedTile t = masked_tile(p, V);
  const int64_t items = (int64_t)t.nbt * p.a * t.jgroups * t.kgroups;
  if ((items + 3) / 4 > kMaxGrid256) return false;
  pl->variant = V_MASKED;
  pl->vec = V;
  pl->unroll = 0;
  pl->waves_m = 1;
  pl->waves_n = t.kgroups;
  pl->bt = 16;
  pl->jg = V;
  pl->lds_bytes = 0;
  pl->block = 256;
  pl->grid = (unsigned)((items + 3) / 4);
  pl->xcd_remap = 0;
  return true;
}

// Where rows through LDS are the faster batch-size-first form.  Its workgroup
// takes the d * b / (16 MT) products of a tile one after the other on four
// wavefronts, which the register kernel has a wavefront each for: with few
// workgroups that chain is the call's time ((2,3,34,37) fp32 at batch 104 4.5 us
// in registers, 13.5 us through LDS; (3,29,2,228) bf16 at batch 1 3.8, 41.9 us),
// with many the shared X rows and whole-line stores win (down to 0.17 of the
// register kernel's time).  Timed both ways on 2500 calls with b or c above 16
// (batch 1 to 4000, fp32, bf16, f16, with and without the epilogue): below 16
// batch rows the LDS form is slower unless a wavefront has one product of a long
// sum.  Above, with at least 6 KB of rows to share, it pays where the register
// kernel has 2500 wavefronts and more, so that its gathers and not their latency
// are what it waits for, from eight workgroups per product of the chain; with
// fewer wavefronts, from 32 per product and sums of 36.  This leaves 17 of those
// calls more than 5 % behind the register kernel, one more than 1.2 times
// (eight workgroups per product alone: 88, 33), and the mean at 0.72 of its time.
bool ragged_bsf_pays(const Problem& p, const Plan& pl) {
  const int kgroups = (pl.kgw + pl.waves_m - 1) / pl.waves_m;
  const int64_t chain = ((int64_t)kgroups * p.d + 3) / 4;  // products per wavefront
  if (p.batch < 16) return chain == 1 && p.c >= 64;
  if (pl.lds_bytes < 6000) return false;
  if (pl.grid >= 32 * chain && p.c >= 36) return true;
  const MaskedTile t = masked_tile(p, masked_vec(p));
  return pl.grid >= 8 * chain && (int64_t)t.nbt * p.a * t.jgroups * t.kgroups >= 2500;
}

// The masked kernel when it is asked for: ks_ragged.h's wherever it can run.
bool plan_masked(const Problem& p, Plan* pl) {
  if (p.layout == BSL) return plan_ragged_bsl(p, pl);
  return plan_ragged_bsf(p, pl) || plan_masked_reg(p, pl);
}

// Batch-size-first: the faster masked kernel is the one with rows in LDS.
bool masked_rows_in_lds(const Problem& p) {
  Plan lds;
  return plan_ragged_bsf(p, &lds) && ragged_bsf_pays(p, lds);
}

// The faster masked kernel.
bool plan_masked_auto(const Problem& p, Plan* pl) {
  if (p.layout == BSL) return plan_ragged_bsl(p, pl);
  Plan lds;
  const bool fits = plan_ragged_bsf(p, &lds);
  if (!(fits && ragged_bsf_pays(p, lds)) && plan_masked_reg(p, pl)) return true;
  if (fits) *pl = lds;
  return fits;
}

hipError_t launch_masked(const Problem& p, const Plan& pl, hipStream_t s) {
  if (pl.unroll) {
    const RaggedTile t = ragged_tile_of(p, pl);
    switch (p.dtype) {
      case F32: return launch_ragged_f32(p, t, pl.vec, pl.waves_m, s);
      case BF16: return launch_ragged_bf16(p, t, pl.vec, pl.waves_m, s);
      case F16: return launch_ragged_f16(p, t, pl.vec, pl.waves_m, s);
      default: return hipErrorInvalidValue;
    }
  }
  const MaskedTile t = masked_tile(p, pl.vec);
  switch (p.dtype) {
    case F32: return launch_masked_f32(p, t, pl.vec, pl.grid, s);
    case BF16: return launch_masked_bf16(p, t, pl.vec, pl.grid, s);
    case F16: return launch_masked_f16(p, t, pl.vec, pl.grid, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_direct(const Problem& p, const Plan& pl, hipStream_t s) {
  const DirectTile t = direct_tile(p, pl);
  const bool strided = pl.unroll != 0;
  if (has_epilogue(p)) {
    switch (p.dtype) {
      case F32: return launch_direct_f32_epi(p, t, pl.vec, strided, pl.waves_m, pl.grid, s);
      case BF16: return launch_direct_bf16_epi(p, t, pl.vec, strided, pl.waves_m, pl.grid, s);
      case F16: return launch_direct_f16_epi(p, t, pl.vec, strided, pl.waves_m, pl.grid, s);
      default: return hipErrorInvalidValue;
    }
  }
  switch (p.dtype) {
    case F32: return launch_direct_f32(p, t, pl.vec, strided, pl.waves_m, pl.grid, s);
    case BF16: return launch_direct_bf16(p, t, pl.vec, strided, pl.waves_m, pl.grid, s);
    case F16: return launch_direct_f16(p, t, pl.vec, strided, pl.waves_m, pl.grid, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace ks
