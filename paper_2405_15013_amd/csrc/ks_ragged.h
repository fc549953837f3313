// Masked MFMA kernels for blocks, batches and buffers of any size and alignment
// (decomposition and index arithmetic in ks_ragged_index.h): b or c not a
// multiple of 16, batch-size-last batches that are not whole vectors, buffers
// that are not 16-byte aligned.
//
// The kernel before them moved X and K in pieces as wide as the batch, d and
// the buffers' alignment allowed (single elements for an odd batch or d), one
// chunk of l at a time with nothing in flight meanwhile, one 16-row tile per
// wavefront, and batch-size-first every lane gathered its own row: it was bound
// by its load instructions and by one memory latency per chunk.  Here every
// load of X is a 16-byte vector, the next chunks are loaded while one is
// multiplied, and batch-size-first the rows go through LDS as runs.  Measured
// (before, now; rate of X + K + Y): fp32 batch-size-last (4,40,24,6) at batch
// 10007 31.5, 16.8 us (3.7 TB/s); (8,64,96,4) at 14637 225, 111 us (2.7 TB/s);
// f16 (6,96,96,4) at 2630 39.0, 12.5 us; bf16 batch-size-first (6,110,80,3) at
// 5504 129, 44 us; (4,29,89,5) at 3327 44, 13 us; 70 calls of all sizes 1.66x in
// the mean.  What bounds it now: batch-size-last the misaligned vectors (two
// lines each) and K operands in lane order, batch-size-first K per 16 or 32 rows
// and the single-element LDS reads; small calls one latency per stage.
#pragma once
#include <type_traits>

#include "ks_direct.h"
#include "ks_ragged_index.h"

namespace ks {

// N elements at an element-aligned address, as one access.
template <typename T, int N>
__device__ __forceinline__ void ragged_load(const T* p, T (&v)[N]) { __builtin_memcpy(v, p, N * sizeof(T)); }
template <typename T, int N>
__device__ __forceinline__ void ragged_store(T* p, const T (&v)[N]) { __builtin_memcpy(p, v, N * sizeof(T)); }

// A K operand: LP values from l of a row (its first element at kr), zero from
// c on.  FULL: the whole chunk lies inside c.  Otherwise the 16-byte vector is
// moved back to end with the row and shifted into place (c >= LP), or its
// elements are loaded one by one.
template <typename T, int LP, bool FULL>
__device__ __forceinline__ void ragged_k(const T* __restrict__ kr, int l, int c, uint32_t (&w)[LP * sizeof(T) / 4]) {
  static_assert(LP * sizeof(T) == 16, "an operand is one 16-byte vector");
  T v[LP];
  if constexpr (FULL) {
    ragged_load<T, LP>(kr + l, v);
    __builtin_memcpy(w, v, sizeof w);
  } else if (c >= LP) {  // wave-uniform
    const int base = l < c - LP ? l : c - LP, shift = (l - base) * 8 * (int)sizeof(T);
    ragged_load<T, LP>(kr + base, v);
    uint64_t q[2];
    __builtin_memcpy(q, v, 16);
    const uint64_t hi = shift < 64 ? q[1] >> shift : 0;
    const uint64_t far = shift < 128 ? q[1] >> (shift & 63) : 0;
    const uint64_t lo = shift == 0 ? q[0] : ((q[0] >> (shift & 63)) | (q[1] << (64 - (shift & 63) & 63)));
    q[0] = shift < 64 ? lo : far;
    q[1] = hi;
    __builtin_memcpy(w, q, 16);
  } else {
#pragma unroll
    for (int q = 0; q < LP; ++q) {
      const int lq = l + q < c ? l + q : c - 1;
      const T x = kr[lq];
      v[q] = l + q < c ? x : T(0);
    }
    __builtin_memcpy(w, v, sizeof w);
  }
}

// Bias and activation of MT row tiles (rows k0 + 16 mt + 4 g + r of block
// (i, j)), NC accumulator columns each.
template <typename T, int MT, int NC>
__device__ __forceinline__ void ragged_epilogue(const Problem& p, int i, int j, int k0, int g, f32x4 (&acc)[MT][NC]) {
  if (p.bias != nullptr) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int k = k0 + 16 * mt + 4 * g + r;
        const float bv = bias_value<T>(p, ((int64_t)i * p.b + (k < p.b ? k : p.b - 1)) * p.d + j);
#pragma unroll
        for (int e = 0; e < NC; ++e) acc[mt][e][r] += bv;
      }
  }
  if (epilogue_gelu(p)) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int e = 0; e < NC; ++e)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[mt][e][r] = gelu_f32<T>(acc[mt][e][r]);
  }
}

// Batch-size-last: the next chunk of l is loaded while one is multiplied.
// (Register hint: accumulators, two chunks, and about 56 for addresses.)
template <typename T, int V, int MT> constexpr int ragged_bsl_waves() {
  constexpr int S = sizeof(T), LP = ragged_lp(S);
  constexpr int regs = 4 * MT * V + 2 * (LP * V * S / 4 + MT * LP * S / 4) + 56, w = 512 / regs;
  return w > 5 ? 5 : w;
}
template <typename T, int V, int MT, bool EPI>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(ragged_bsl_waves<T, V, MT>())))
void ks_masked_bsl_kernel(Problem p, RaggedTile t) {
  constexpr int S = sizeof(T), LP = ragged_lp(S), CH = 4 * LP, XW = LP * V * S / 4;
  const int lane = threadIdx.x & 63, n = lane & 15, g = lane >> 4;
  const int item0 = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool live = item0 < t.items;  // wave-uniform; spare waves work on the last item and store nothing
  const RItem it = ragged_item(p, t, live ? item0 : t.items - 1, 16 * MT);
  const int c = p.c, nfull = c / CH;
  const int64_t ls = (int64_t)p.d * p.batch;  // between rows l
  const T* __restrict__ x = static_cast<const T*>(p.x) + ((int64_t)it.i * c * p.d + it.j) * p.batch;
  const int col = ragged_col(p, it, V, n), lo = (int)((uint32_t)ls * (uint32_t)(LP * g)) + col;
  const T* __restrict__ kr[MT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
    kr[mt] = static_cast<const T*>(p.kv) + ragged_k_row(p, it.i, it.j, it.k0 + 16 * mt + n);

  struct Chunk {
    uint32_t xw[XW], kw[MT][1][LP * S / 4];
  };
  auto load = [&](int ch, Chunk& k) {
    T xs[LP][V];
#pragma unroll
    for (int q = 0; q < LP; ++q) ragged_load<T, V>(x + (int64_t)(ch * CH + q) * ls + lo, xs[q]);
    __builtin_memcpy(k.xw, xs, sizeof k.xw);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) ragged_k<T, LP, true>(kr[mt], ch * CH + LP * g, c, k.kw[mt][0]);
  };
  f32x4 acc[MT][V];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int e = 0; e < V; ++e) acc[mt][e] = f32x4{0.f, 0.f, 0.f, 0.f};
  Chunk ka, kb;
  if (nfull > 0) load(0, ka);
  // The chunk that c cuts short first, behind the loads of the first whole one.
  if (nfull * CH < c) {
    Chunk k;
    T xs[LP][V];
#pragma unroll
    for (int q = 0; q < LP; ++q) {
      const int l = nfull * CH + LP * g + q;
      ragged_load<T, V>(x + (int64_t)(l < c ? l : c - 1) * ls + col, xs[q]);
    }
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) ragged_k<T, LP, false>(kr[mt], nfull * CH + LP * g, c, k.kw[mt][0]);
#pragma unroll
    for (int q = 0; q < LP; ++q)
#pragma unroll
      for (int e = 0; e < V; ++e) xs[q][e] = nfull * CH + LP * g + q < c ? xs[q][e] : T(0);
    __builtin_memcpy(k.xw, xs, sizeof k.xw);
    direct_mma<T, BSL, V, MT, LP>(k.xw, k.kw, acc);
    mfma_results_settle();  // before the paths join
  }
  __builtin_amdgcn_sched_barrier(0);
  int ch = 0;
  for (; ch + 2 < nfull; ch += 2) {
    load(ch + 1, kb);
    __builtin_amdgcn_sched_barrier(0);
    direct_mma<T, BSL, V, MT, LP>(ka.xw, ka.kw, acc);
    load(ch + 2, ka);
    __builtin_amdgcn_sched_barrier(0);
    direct_mma<T, BSL, V, MT, LP>(kb.xw, kb.kw, acc);
    mfma_results_settle();  // the paths' join copies the accumulators, here and below
  }
  if (ch + 1 < nfull) {
    load(ch + 1, kb);
    __builtin_amdgcn_sched_barrier(0);
    direct_mma<T, BSL, V, MT, LP>(ka.xw, ka.kw, acc);
    direct_mma<T, BSL, V, MT, LP>(kb.xw, kb.kw, acc);
    mfma_results_settle();
  } else if (ch < nfull) {
    direct_mma<T, BSL, V, MT, LP>(ka.xw, ka.kw, acc);
    mfma_results_settle();
  }
  if (!live) return;
  if constexpr (EPI) ragged_epilogue<T, MT, V>(p, it.i, it.j, it.k0, g, acc);
  const int shift = ragged_shift(p, it, V, n);
  if (shift >= V) return;
  T* __restrict__ y = static_cast<T*>(p.y) + ((int64_t)it.i * p.b * p.d + it.j) * p.batch + col;
  // Rows of aligned vectors are streamed; others share lines with their
  // neighbours' stores, which meet in L2.
  const bool stream = V * S == 16 && p.batch % V == 0 && p.align >= 16;
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int k = it.k0 + 16 * mt + 4 * g + r;
      if (k >= p.b) continue;
      T v[V];
#pragma unroll
      for (int e = 0; e < V; ++e) v[e] = from_f32<T>(acc[mt][e][r]);
      T* yk = y + (int64_t)k * ls;
      if (V * S == 16 && stream) {
        u32x4 w;
        __builtin_memcpy(&w, v, V * S == 16 ? 16 : V * S);
        __builtin_nontemporal_store(w, reinterpret_cast<u32x4*>(yk));
      } else if (shift == 0) {
        ragged_store<T, V>(yk, v);
      } else {
#pragma unroll
        for (int e = 1; e < V; ++e)
          if (e >= shift) yk[e] = v[e];
      }
    }
}

// Batch-size-first.
template <typename T, int RG, int MT, bool EPI>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(MT * RG >= 8 ? 2 : (MT * RG * (int)sizeof(T) >= 16 ? 3 : (sizeof(T) == 4 ? 4 : (MT * RG >= 4 ? 2 : (MT * RG >= 2 ? 3 : 4)))))))
void ks_masked_bsf_kernel(Problem p, RaggedTile t) {
  constexpr int S = sizeof(T), LP = ragged_lp(S), CH = 4 * LP, E = 16 / S, KW = LP * S / 4, ROWS = 16 * RG, LB = 8;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  char* yl = smem + ROWS * t.xpitch;
  const int tid = threadIdx.x, lane = tid & 63, n = lane & 15, g = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const RItem it = ragged_item(p, t, (int)blockIdx.x, t.kb);
  const int c = p.c, d = p.d, nfull = c / CH;
  const int kend = it.k0 + t.kb < p.b ? it.k0 + t.kb : p.b;  // rows k0 .. kend
  const int row0 = it.bt * ROWS;
  const T* __restrict__ kv = static_cast<const T*>(p.kv);

  // Items of this wavefront: s = w, w + 4, ... < items, j = s % d, group s / d.
  const int items = (kend - it.k0 + 16 * MT - 1) / (16 * MT) * d;
  struct KOps {
    uint32_t w[MT][KW];
  };
  const T* kr[MT];
  auto item_rows = [&](int s) {
    const int kg = (int)div_fast((uint32_t)s, t.md, t.sd), j = s - kg * d;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) kr[mt] = kv + ragged_k_row(p, it.i, j, it.k0 + kg * 16 * MT + 16 * mt + n);
  };
  auto kload = [&](int ch, KOps& k) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) ragged_k<T, LP, true>(kr[mt], ch * CH + LP * g, c, k.w[mt]);
  };
  // An item's first operands: chunk 0, or where c ends inside it, that.
  auto kfirst = [&](KOps& k) {
    if (nfull > 0) {
      kload(0, k);
    } else {
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) ragged_k<T, LP, false>(kr[mt], LP * g, c, k.w[mt]);
    }
  };
  KOps ka, kb;
  if (w < items) {
    item_rows(w);
    kfirst(ka);
  }

  // X runs to LDS, 16 bytes a time (a unit past the run's end reads what
  // follows it, which no operand uses; past the buffer's end, nothing).
  {
    const T* __restrict__ x = static_cast<const T*>(p.x);
    const int64_t total = (int64_t)p.batch * p.N;
    const int units = ROWS * t.upr;
    for (int u0 = tid; u0 < units; u0 += 256 * LB) {
      u32x4 v[LB];
#pragma unroll
      for (int q = 0; q < LB; ++q) {
        const int u = u0 + 256 * q < units ? u0 + 256 * q : units - 1;
        const int row = (int)div_fast((uint32_t)u, t.mupr, t.supr);
        const int beta = row0 + row < p.batch ? row0 + row : p.batch - 1;
        const int64_t off = (int64_t)beta * p.N + (int64_t)it.i * c * d + (u - row * t.upr) * E;
        T e[E];
        if (off + E <= total) {
          ragged_load<T, E>(x + off, e);
        } else {
#pragma unroll
          for (int z = 0; z < E; ++z) e[z] = off + z < total ? x[off + z] : T(0);
        }
        __builtin_memcpy(&v[q], e, 16);
      }
#pragma unroll
      for (int q = 0; q < LB; ++q) {
        const int u = u0 + 256 * q;
        if (u >= units) break;
        const int row = (int)div_fast((uint32_t)u, t.mupr, t.supr);
        *reinterpret_cast<u32x4*>(smem + row * t.xpitch + (u - row * t.upr) * 16) = v[q];
      }
    }
  }
  __syncthreads();

  for (int s = w; s < items; s += 4) {
    const int kg = (int)div_fast((uint32_t)s, t.md, t.sd), j = s - kg * d;
    f32x4 acc[MT][RG];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int u = 0; u < RG; ++u) acc[mt][u] = f32x4{0.f, 0.f, 0.f, 0.f};
    const T* xl = reinterpret_cast<const T*>(smem + n * t.xpitch) + j;
    auto mma = [&](auto full, int ch, const KOps& k) {
      const int l0 = ch * CH + LP * g, ustep = 16 * t.xpitch / S;
      T xs[RG][LP];
      if constexpr (!decltype(full)::value) {
#pragma unroll
        for (int u = 0; u < RG; ++u)
#pragma unroll
          for (int q = 0; q < LP; ++q) {
            const T v = xl[u * ustep + (l0 + q < c ? l0 + q : c - 1) * d];
            xs[u][q] = l0 + q < c ? v : T(0);
          }
      } else if (d == 1) {
#pragma unroll
        for (int u = 0; u < RG; ++u) __builtin_memcpy(xs[u], __builtin_assume_aligned(xl + u * ustep + l0, 16), sizeof xs[u]);
      } else {
#pragma unroll
        for (int u = 0; u < RG; ++u)
#pragma unroll
          for (int q = 0; q < LP; ++q) xs[u][q] = xl[u * ustep + (l0 + q) * d];
      }
#pragma unroll
      for (int u = 0; u < RG; ++u) {
        uint32_t xw[KW];
        __builtin_memcpy(xw, xs[u], sizeof xw);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
          if constexpr (S == 4) {
#pragma unroll
            for (int q = 0; q < 4; ++q) DMma<T, 4>::run(k.w[mt], __uint_as_float(xw[q]), q, acc[mt][u]);
          } else {
            DMma<T, LP>::run(k.w[mt], xw, acc[mt][u]);
          }
        }
      }
      // (Where the accumulators move to other registers from chunk to chunk,
      // the old ones are not reused before the MFMAs have read them.)
      if constexpr (MT * RG >= 8) mfma_results_settle();
    };
    int ch = 0;
    for (; ch + 2 < nfull; ch += 2) {
      kload(ch + 1, kb);
      __builtin_amdgcn_sched_barrier(0);
      mma(std::true_type(), ch, ka);
      kload(ch + 2, ka);
      __builtin_amdgcn_sched_barrier(0);
      mma(std::true_type(), ch + 1, kb);
      mfma_results_settle();  // the paths' join copies the accumulators, here and below
    }
    if (ch + 1 < nfull) {
      kload(ch + 1, kb);
      __builtin_amdgcn_sched_barrier(0);
      mma(std::true_type(), ch, ka);
      mma(std::true_type(), ch + 1, kb);
      mfma_results_settle();
    } else if (ch < nfull) {
      mma(std::true_type(), ch, ka);
      mfma_results_settle();
    }
    if (nfull * CH < c) {
      if (nfull > 0) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) ragged_k<T, LP, false>(kr[mt], nfull * CH + LP * g, c, ka.w[mt]);
      }
      mma(std::false_type(), nfull, ka);
      mfma_results_settle();
    }
    if (s + 4 < items) {  // the next item's first operands, behind this one's output
      item_rows(s + 4);
      kfirst(ka);
    }
    const int k0 = it.k0 + kg * 16 * MT;
    if constexpr (EPI) ragged_epilogue<T, MT, RG>(p, it.i, j, k0, g, acc);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int k = k0 + 16 * mt + 4 * g + r;
        if (k >= kend) continue;
#pragma unroll
        for (int u = 0; u < RG; ++u)
          reinterpret_cast<T*>(yl + (16 * u + n) * t.ypitch)[(k - it.k0) * d + j] = from_f32<T>(acc[mt][u][r]);
      }
  }
  __syncthreads();

  // Y runs from LDS.
  {
    const int run = (kend - it.k0) * d, upr = (run + E - 1) / E;
    T* __restrict__ y = static_cast<T*>(p.y) + ((int64_t)it.i * p.b + it.k0) * d;
    const int valid = p.batch - row0 < ROWS ? p.batch - row0 : ROWS;
    // 16 lanes per row
    for (int row = tid >> 4; row < valid; row += 16)
      for (int v = tid & 15; v < upr; v += 16) {
        const u32x4 val = *reinterpret_cast<const u32x4*>(yl + row * t.ypitch + v * 16);
        T* dst = y + (int64_t)(row0 + row) * p.M + v * E;
        T e[E];
        __builtin_memcpy(e, &val, 16);
        if (v * E + E <= run) {
          ragged_store<T, E>(dst, e);
        } else {
#pragma unroll
          for (int z = 0; z < E; ++z)
            if (v * E + z < run) dst[z] = e[z];
        }
      }
  }
}

constexpr int kRaggedMaxLds = 160 * 1024;

template <typename T>
hipError_t launch_ragged_type(const Problem& p, const RaggedTile& t, int V, int MT, hipStream_t s) {
  const bool epi = has_epilogue(p);
#define KS_RAGGED_BSL(VV, M)                                                                                  \
  if (V == VV && MT == M) {                                                                                   \
    const dim3 grid((t.items + 3) / 4);                                                                       \
    if (epi) hipLaunchKernelGGL((ks_masked_bsl_kernel<T, VV, M, true>), grid, dim3(256), 0, s, p, t);          \
    else hipLaunchKernelGGL((ks_masked_bsl_kernel<T, VV, M, false>), grid, dim3(256), 0, s, p, t);             \
    return hipGetLastError();                                                                                 \
  }
#define KS_RAGGED_BSF_EPI(R, M, EP)                                                                           \
  {                                                                                                           \
    if (t.lds > 64 * 1024) {                                                                                  \
      static const hipError_t raised = hipFuncSetAttribute(reinterpret_cast<const void*>(&ks_masked_bsf_kernel<T, R, M, EP>), \
                                                           hipFuncAttributeMaxDynamicSharedMemorySize, kRaggedMaxLds); \
      if (raised != hipSuccess) return raised;                                                                \
    }                                                                                                         \
    hipLaunchKernelGGL((ks_masked_bsf_kernel<T, R, M, EP>), dim3(t.items), dim3(256), t.lds, s, p, t);        \
    return hipGetLastError();                                                                                 \
  }
#define KS_RAGGED_BSF(R, M)                                                                                   \
  if (V == R && MT == M) {                                                                                    \
    if (epi) KS_RAGGED_BSF_EPI(R, M, true) else KS_RAGGED_BSF_EPI(R, M, false)                                \
  }
  if (p.layout == BSL) {
    KS_RAGGED_BSL(1, 1) KS_RAGGED_BSL(1, 2) KS_RAGGED_BSL(1, 4)
    KS_RAGGED_BSL(2, 1) KS_RAGGED_BSL(2, 2) KS_RAGGED_BSL(2, 4)
    KS_RAGGED_BSL(4, 1) KS_RAGGED_BSL(4, 2) KS_RAGGED_BSL(4, 4)
    if constexpr (sizeof(T) == 2) {
      KS_RAGGED_BSL(8, 1) KS_RAGGED_BSL(8, 2)
    }
  } else {
    KS_RAGGED_BSF(1, 1) KS_RAGGED_BSF(1, 2) KS_RAGGED_BSF(1, 4)
    KS_RAGGED_BSF(2, 1) KS_RAGGED_BSF(2, 2) KS_RAGGED_BSF(2, 4)
  }
#undef KS_RAGGED_BSL
#undef KS_RAGGED_BSF
#undef KS_RAGGED_BSF_EPI
  return hipErrorInvalidValue;
}

}  // namespace ks
