// LDS-DMA MFMA kernels for batch-size-first KS patterns.
//
// Same output-stationary tiles and products as the LDS-staged kernels (paper
// Section 4.1, Algorithm 2; tile and item mapping in ks_staged_index.h), with
// the X stages moved from HBM to LDS by the memory unit itself
// (global_load_lds_dwordx4: every lane's 16 bytes land at M0 + 16 * lane), so
// the bytes in flight occupy no registers.  Three stage buffers per
// workgroup: while stage s is multiplied, stages s+1 and s+2 are in flight.
// The paper's weak batch-size-first case (Section 4.2) again becomes
// contiguous row runs: each stage row is X[beta, i*c*d + ls*d .. (ls+LCH)*d).
//
// Synchronisation, per stage s:
//   1. wait until at most UD vector-memory operations are outstanding (the
//      DMAs of stage s+1), so this wavefront's DMAs of stage s and its K loads
//      of stage s have completed;
//   2. s_barrier: every wavefront's DMAs of stage s are in LDS, and every
//      wavefront has finished reading stage s-1, whose buffer is refilled next;
//   3. load K of stage s+1 (registers), then DMA stage s+2;
//   4. read the operands of stage s from LDS and run the MFMAs.
// The vector-memory issue order of step 3 (K loads, then DMAs) is pinned with
// scheduling barriers, which is what makes the count of step 1 exact.  The
// operand reads are issued as inline assembly with their own wait: the
// compiler cannot tell which LDS bytes a DMA writes and would otherwise wait
// for every DMA in flight before using any LDS value.
//
// Outputs leave through the structured epilogue of the staged kernel (LDS
// copy of the output tile, coalesced 16-byte stores; Appendix D.3).
#pragma once
#include <type_traits>

#include "ks_direct.h"
#include "ks_staged_index.h"

namespace ks {

typedef __attribute__((address_space(3))) void lds_void_t;
constexpr int kDmaMaxLds = 160 * 1024;

// vmcnt(N) on gfx9: vmcnt in bits 3:0 and 15:14, expcnt (bits 6:4) and
// lgkmcnt (bits 11:8) left at their maxima (no wait).
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt is six bits");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

// The problem's and the tile description's fields in scalar registers at
// kernel entry, in one statement so that they arrive in one round of
// kernel-argument loads (as kernarg_fetch(Problem) in ks_direct.h).
__device__ __forceinline__ void kernarg_fetch(const Problem& p, const StagedTile& t) {
  asm volatile("" ::KS_PROBLEM_FIELDS(p), "s"(t.tiles), "s"(t.remap), "s"(t.kgt), "s"(t.nbt), "s"(t.mkgt),
               "s"(t.skgt), "s"(t.mnbt), "s"(t.snbt), "s"(t.RS), "s"(t.lRS), "s"(t.JG), "s"(t.lJG), "s"(t.KGW),
               "s"(t.UR), "s"(t.lUR), "s"(t.stage));
}

// Workgroup barrier without a memory fence (a fence would wait for every DMA
// in flight); the empty asm statements keep the compiler from moving memory
// accesses across it, the scheduling barriers keep the scheduler from doing so.
__device__ __forceinline__ void dma_barrier() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// One LDS read of NB bytes at LDS byte address addr, outside the compiler's
// tracking (the caller waits with lds_wait before using the value).
template <int NB> struct LdsVec;
template <> struct LdsVec<16> {
  typedef u32x4 type;
  __device__ static __forceinline__ type read(uint32_t addr) {
    type v;
    asm volatile("ds_read_b128 %0, %1" : "=v"(v) : "v"(addr));
    return v;
  }
};
template <> struct LdsVec<8> {
  typedef u32x2 type;
  __device__ static __forceinline__ type read(uint32_t addr) {
    type v;
    asm volatile("ds_read_b64 %0, %1" : "=v"(v) : "v"(addr));
    return v;
  }
};

// The K operands of one chunk (one stage): MT x V blocks of LP values of l
// (load: straight into registers; see KLDS below for the other way).
template <typename T, int V, int MT, int LP>
struct DmaK {
  static constexpr int KW = LP * (int)sizeof(T) / 4;
  uint32_t kw[MT][V][KW];
  __device__ __forceinline__ void load(const T* __restrict__ kl, int64_t kmstride, int64_t kestride, int l) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int e = 0; e < V; ++e) load_piece<KW * 4, false>(kl + mt * kmstride + e * kestride + l, kw[mt][e]);
  }
};

// KLDS: the K operands of a stage go to LDS by DMA as well, into a buffer of
// the wavefront's own, and are read from there in the MFMA's lane order.  A
// register load in that order gives every group of four lanes four rows of K
// and takes the address unit 64 cycles per operand instead of 16; with b and c
// large that bound the kernel ((8,128,128,8) bf16 at batch 25088: 12544 tiles of
// 128 operands and 96 other 1 KB accesses are 476 K cycles per CU of the 616 K
// the call took, the unit's busy counter 465 K).  Measured: that call 265 ->
// 211 us, (2,64,64,16) fp32 140 -> 132 us, (8,128,64,8) bf16 171 -> 131 us.
// Taking the operands out of coalesced register loads with ds_bpermute instead
// (four per operand) measured 214 us, 146 us and 3 % slower elsewhere.
// V j values per lane (V = min(d, 4)): STRIDED when d > V (pieces of V
// elements at stride d), otherwise the lane's LP x V block is contiguous.
// The body of the two kernels below (KLDS false: K operands straight into
// registers, true: through LDS) is a file of its own, included in each: as a
// function that both call, the compiler orders its instructions another way, and
// single calls took up to 10 % more or less time ((6,64,16,8) bf16 with bias and
// GELU at batch 25088 51.1 -> 53.7 us, (6,48,32,16) fp32 at 13020 138 -> 145).
// Register budget per instance: the smallest tiles (MT = NT = 1) are fitted
// to four waves per SIMD (four workgroups per CU), NT = 2 to three, the rest
// to two (the accumulators then live in VGPRs instead of AGPRs).
constexpr int dma_waves(int MT, int NT) { return MT * NT == 1 ? 4 : ((MT == 1 && NT == 2) ? 3 : 2); }
template <typename T, int V, bool STRIDED, int MT, int LP, int UD, int NT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(dma_waves(MT, NT))))
void ks_dma_kernel(Problem p, StagedTile t) {
  constexpr bool KLDS = false;
#include "ks_dma_body.h"
}
template <typename T, int V, bool STRIDED, int MT, int LP, int UD, int NT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(dma_waves(MT, NT))))
void ks_dma_klds_kernel(Problem p, StagedTile t) {
  constexpr bool KLDS = true;
#include "ks_dma_body.h"
}

template <typename T, int V, bool STRIDED, int MT, int LP, int UD, int NT, bool KLDS>
hipError_t launch_dma_inst(const Problem& p, const StagedTile& t, hipStream_t s) {
  void (*kernel)(Problem, StagedTile);
  if constexpr (KLDS) kernel = ks_dma_klds_kernel<T, V, STRIDED, MT, LP, UD, NT>;
  else kernel = ks_dma_kernel<T, V, STRIDED, MT, LP, UD, NT>;
  if (t.lds > 64 * 1024) {
    // Opt in to more than 64 KB of dynamic LDS once per instance (a function-
    // local static: initialised exactly once even with concurrent callers).
    static const hipError_t raised = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                                         hipFuncAttributeMaxDynamicSharedMemorySize, kDmaMaxLds);
    if (raised != hipSuccess) return raised;
  }
  hipLaunchKernelGGL(kernel, dim3(t.tiles), dim3(256), t.lds, s, p, t);
  return hipGetLastError();
}

// (MT, NT) pairs instantiated: MT * NT <= 4.
template <typename T, int V, bool STRIDED, int LP, int UD>
hipError_t launch_dma_mt(const Problem& p, const StagedTile& t, int mt, hipStream_t s) {
  const int nt = t.NT;
#define KS_DMA_INST(M, N)                                                                              \
  if (mt == M && nt == N) {                                                                           \
    if constexpr (V == 4 && LP * sizeof(T) == 16)                                                     \
      if (t.klds) return launch_dma_inst<T, V, STRIDED, M, LP, UD, N, true>(p, t, s);                  \
    return t.klds ? hipErrorInvalidValue : launch_dma_inst<T, V, STRIDED, M, LP, UD, N, false>(p, t, s); \
  }
  KS_DMA_INST(1, 1) KS_DMA_INST(2, 1) KS_DMA_INST(1, 2) KS_DMA_INST(2, 2) KS_DMA_INST(1, 4)
#undef KS_DMA_INST
  return hipErrorInvalidValue;
}

// Instances of one storage type and j-vector mode (V, STRIDED): (MT, NT) with
// MT * NT <= 4, LP (4 for fp32; 8, or 4, for 16-bit types), 2, 4 or 8 DMA
// instructions per wavefront per stage.  One source file per storage type
// and mode, so the instances compile in parallel.
template <typename T, int V, bool STRIDED>
hipError_t launch_dma_mode(const Problem& p, const StagedTile& t, int mt, int lp, hipStream_t s) {
  if (t.W != 4) return hipErrorInvalidValue;
  if constexpr (sizeof(T) == 4) {
    if (lp != 4) return hipErrorInvalidValue;
  }
#define KS_DMA_UD(LPV)                                                              \
  switch (t.UD) {                                                                   \
    case 2: return launch_dma_mt<T, V, STRIDED, LPV, 2>(p, t, mt, s);               \
    case 4: return launch_dma_mt<T, V, STRIDED, LPV, 4>(p, t, mt, s);               \
    case 8: return launch_dma_mt<T, V, STRIDED, LPV, 8>(p, t, mt, s);               \
    default: return hipErrorInvalidValue;                                           \
  }
  if (lp == 4) { KS_DMA_UD(4) }
  if constexpr (sizeof(T) == 2) {
    if (lp == 8) { KS_DMA_UD(8) }
  }
#undef KS_DMA_UD
  return hipErrorInvalidValue;
}

}  // namespace ks
