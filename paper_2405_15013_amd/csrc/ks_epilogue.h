// Output epilogue shared by every kernel: Y = act(X K^T + bias), for the
// KS layers of a Transformer MLP (paper appendix, ViT-S/16 submodule table:
// "Linear + bias" rows, and the feed-forward block Linear + GELU).  bias holds
// one value per output feature m (the column of Y in BSF, its row in BSL) in
// the storage type; act is KS_ACT_NONE or KS_ACT_GELU (the exact form
// x * Phi(x) = 0.5 x (1 + erf(x / sqrt 2))).  Both are wave-uniform launch
// arguments.  The kernels test them once per tile, not per output: the bias
// of all of a lane's outputs is loaded in one batch, then added, then the
// activation runs over the whole register tile, so a plain ks_matmul pays two
// untaken scalar branches.
#pragma once
#include "ks_common.h"
#include "ks_internal.h"

namespace ks {

constexpr int kActGelu = 1;  // KS_ACT_GELU

__device__ __forceinline__ bool epilogue_on(const Problem& p) { return p.bias != nullptr || p.act != 0; }
__device__ __forceinline__ bool epilogue_gelu(const Problem& p) { return p.act == kActGelu; }

template <typename T>
__device__ __forceinline__ float bias_value(const Problem& p, int64_t m) {
  return to_f32(static_cast<const T*>(p.bias)[m]);
}

// Monomial coefficients of R(u), written by gelu_fit.py (Chebyshev fit of
// degree 9; |R_fit - R| <= 1.3e-7 in log2 units, i.e. a relative error of
// 9e-8 in the normal tail below, for |x| <= 16).
constexpr float kGeluR0 = -1.82569253f;
constexpr float kGeluR1 = 2.88297439f;
constexpr float kGeluR2 = 2.20453787f;
constexpr float kGeluR3 = 0.657676935f;
constexpr float kGeluR4 = -1.50583696f;
constexpr float kGeluR5 = 2.12293911f;
constexpr float kGeluR6 = -78.4830017f;
constexpr float kGeluR7 = 235.065887f;
constexpr float kGeluR8 = -269.774841f;
constexpr float kGeluR9 = 113.810883f;

// Degree 5 (gelu_fit.py, same fit): |R_fit - R| <= 1.2e-5 in log2 units, a
// relative error of 8e-6 in the tail, far below the precision of 16-bit
// outputs (bf16 2^-8, fp16 2^-11); used when the result is stored in 16 bits.
constexpr float kGeluS0 = -1.82723665f;
constexpr float kGeluS1 = 2.93737769f;
constexpr float kGeluS2 = 1.46866286f;
constexpr float kGeluS3 = 5.47383213f;
constexpr float kGeluS4 = -16.3639202f;
constexpr float kGeluS5 = 10.5570784f;

// Exact GELU without branches.  With z = |x| / sqrt 2 and u = 1 / (2 + z),
// the normal tail is Phi(-|x|) = erfc(z) / 2 = u * 2^(-log2(e) x^2 / 2 + R(u))
// where R(u) = log2(exp(z^2) erfc(z) / (2u)) is smooth on (0, 1/2] (fitted
// above).  Since Phi(x) = 1 - Phi(-x), both signs reduce to
// GELU(x) = max(x, 0) - |x| Phi(-|x|).  The tail keeps its relative accuracy
// (no 1 + erf cancellation).  |x| > 16 needs no clamp: the power of two is 0
// there and R stays finite (u goes to 0); the product |x| u alone would be
// infinity times 0 (gelu_mul0).  NaN gives NaN.
// Cost: 15 VALU operations, one v_rcp_f32 and one v_exp_f32 (11 VALU with
// the degree-5 R for 16-bit outputs, OUT the type the result is stored in), each
// of the two four times as long as a VALU operation: with short sums the
// epilogue bounds the call.  The form with a clamp of x (med3), fmaxf (whose
// operand the compiler canonicalizes first) and the polynomial's first constant
// moved for each output took three operations more.  (6,64,16,8) with bias and
// GELU at batch 25088: FP8 batch-size-first 54.4 -> 47.6 us, batch-size-last bf16
// 53.7 -> 50.0, f16 56.9 -> 53.4, FP8 63.0 -> 57.2 us; fp32 1 to 4 % faster; bf16
// batch-size-first the same (54 us, 51 since its operands are packed by
// v_perm_b32: a tile of the DMA kernel runs these operations with none of its
// own loads in flight and two workgroups per CU, so they add to the X stream
// instead of running under it).  Of 700 batch-size-first DMA calls with bias and
// GELU, batch 500 to 25088, the mean is 0.97 of the longer form's time; 28, most
// in fp32, are 1.03 to 1.17 times slower ((6,48,32,16) fp32 at batch 13020 128 ->
// 138 us, (8,64,32,16) f16 at 14208 94 -> 99), although they issue fewer
// operations.  Putting the next reciprocal and the last power of two under each
// polynomial by hand gave 137 and 99 us there, 0.99 of the time in 16 bits in the
// mean and 97 -> 102 us in (6,64,16,8) fp32, other single calls 3 to 10 % slower:
// not kept.
// A constant in a vector register, for operands that take no literal.
__device__ __forceinline__ float gelu_reg(float c) {
  asm("" : "+v"(c));
  return c;
}

// |x| * u, 0 when u is 0 (u = 0 is the reciprocal of |x| infinite).  r, which
// is computed from u, is an operand only to keep the instruction away from the
// v_rcp_f32 that made u (a transcendental's result must not be read by the very
// next instruction, and the compiler does not look into the statement).
__device__ __forceinline__ float gelu_mul0(float x, float u, float r) {
  float v;
  asm("v_mul_legacy_f32 %0, |%1|, %2" : "=v"(v) : "v"(x), "v"(u), "v"(r));
  return v;
}

template <typename OUT = float>
__device__ __forceinline__ float gelu_f32(float x) {
  const float u = __builtin_amdgcn_rcpf(__builtin_fmaf(__builtin_fabsf(x), 0.70710678118654752f, 2.0f));
  float r;
  if constexpr (sizeof(OUT) == 4) {
    r = __builtin_fmaf(gelu_reg(kGeluR9), u, kGeluR8);
    r = __builtin_fmaf(r, u, kGeluR7);
    r = __builtin_fmaf(r, u, kGeluR6);
    r = __builtin_fmaf(r, u, kGeluR5);
    r = __builtin_fmaf(r, u, kGeluR4);
    r = __builtin_fmaf(r, u, kGeluR3);
    r = __builtin_fmaf(r, u, kGeluR2);
    r = __builtin_fmaf(r, u, kGeluR1);
    r = __builtin_fmaf(r, u, kGeluR0);
  } else {
    r = __builtin_fmaf(gelu_reg(kGeluS5), u, kGeluS4);
    r = __builtin_fmaf(r, u, kGeluS3);
    r = __builtin_fmaf(r, u, kGeluS2);
    r = __builtin_fmaf(r, u, kGeluS1);
    r = __builtin_fmaf(r, u, kGeluS0);
  }
  const float e = __builtin_amdgcn_exp2f(__builtin_fmaf(x * -0.72134752044448170f, x, r));  // 2^(R(u) - log2(e)/2 x^2)
  const float relu = __builtin_amdgcn_fmed3f(x, 0.0f, gelu_reg(__builtin_inff()));
  return __builtin_fmaf(-gelu_mul0(x, u, r), e, relu);
}

// Single-output form (bias index m), for kernels with one output per thread.
template <typename T>
__device__ __forceinline__ float epilogue_apply(const Problem& p, float v, int64_t m) {
  if (p.bias != nullptr) v += bias_value<T>(p, m);
  if (epilogue_gelu(p)) v = gelu_f32<T>(v);
  return v;
}

}  // namespace ks
