// Shared by the backward pass's kernels: valid rows, the transposing LDS fragment read.
#pragma once
#include "../../include/longer.h"
#include "device.h"

namespace longer {
namespace bw {

constexpr int kComputeUnits = 256;

// Every row carries a descriptor of its token: -1 invalid, a for global token a, kSeq + t for the sequence token
// with merged index t (a learnable query token stands after the newest one).
constexpr int kSeq = 1 << 24;

// Padded token rows (row r = u L + pos with pos >= the user's length) carry no gradient.  With the
// batch's geometry at hand a kernel leaves them out: row GEMMs skip tiles without a valid row, the
// gradient GEMMs read them as zeros and pass over steps that hold nothing else, the LayerNorm kernels
// write zeros for them.  L = 0: every row counts (the reduced stack's rows).  A row stands for `unit` tokens (a group's sums: K).
struct RowsValid { const int32_t* lens; int L; };
__device__ __forceinline__ bool row_valid(const RowsValid& v, int r, int unit = 1) {
  if (v.L == 0 || v.lens == nullptr) return true;
  const int u = r / v.L;
  return (r - u * v.L) * unit < v.lens[u];
}
// any valid row in [r0, r1)?
__device__ __forceinline__ bool rows_any_valid(const RowsValid& v, int r0, int r1, int unit = 1) {
  if (v.L == 0 || v.lens == nullptr) return true;
  for (int u = r0 / v.L; u * v.L < r1; ++u) {
    const int first = max(r0, u * v.L) - u * v.L;
    if (first * unit < v.lens[u]) return true;
  }
  return false;
}

// v, or zeros.  (Requests go out unconditionally, for a row that exists, and what is not wanted is dropped afterwards: under a
// condition each request of a workgroup's start came to wait for the one before: training step of the headline batch 4333 against
// 4306 us, of a small one 312 against 309, both sides timed in turn.)
__device__ __forceinline__ bf16x8 keep_if(bf16x8 v, bool wanted) {
  const u32x4 b = __builtin_bit_cast(u32x4, v);
  u32x4 w;
#pragma unroll
  for (int e = 0; e < 4; ++e) { const uint32_t one = b[e]; w[e] = wanted ? one : 0u; }
  return __builtin_bit_cast(bf16x8, w);
}

// Phi(v) = (1 + erf(v / sqrt 2)) / 2 and exp(-v^2 / 2) from one exponential: for z >= 0,
// erf(z) = 1 - (a1 t + a2 t^2 + a3 t^3 + a4 t^4 + a5 t^5) exp(-z^2), t = 1 / (1 + p z), absolute error
// below 1.5e-7 (the classic five-term approximation; odd extension for z < 0).
// (the reciprocal: hardware estimate and one Newton step, within an ulp of the rounded one at a third of its instructions)
__device__ __forceinline__ void gauss_cdf(float v, float* cdf, float* ex) {
  const float u = v * v;
  const float e = __builtin_amdgcn_exp2f(u * -0.72134752044448170f);       // exp(-v^2 / 2)
  const float q = fmaf(0.23164189f, fabsf(v), 1.f);                        // 1 + p z, z = |v| / sqrt 2
  const float r = __builtin_amdgcn_rcpf(q);
  const float t = r * fmaf(-q, r, 2.f);
  float poly = fmaf(t, 0.5307027145f, -0.7265760135f);                     // (half the coefficients: (1 - erf(z)) / 2)
  poly = fmaf(t, poly, 0.7107068705f);
  poly = fmaf(t, poly, -0.142248368f);
  poly = fmaf(t, poly, 0.127414796f);
  const float half_erfc = poly * t * e;
  *cdf = v >= 0.f ? 1.f - half_erfc : half_erfc;
  *ex = e;
}

// The activation and its derivative at once, for the launch that rounds both to bf16 right away.
// GELU: Phi(v) - 1/2 as v times an even polynomial of degree 8 (minimax fit on [-3.5, 3.5] that reaches 1/2
// at the interval's end, clamped to [0, 1] beyond it; absolute error below 1.3e-3, under the bf16
// rounding step of the values it produces) and the density from one exponential.
__device__ __forceinline__ void act_both(float v, int act, float* a, float* da) {
  if (act == LONGER_ACT_RELU) { *a = v > 0.f ? v : 0.f; *da = v > 0.f ? 1.f : 0.f; return; }
  const float u = v * v;
  float pl = 9.366767568843253e-06f;
  pl = fmaf(pl, u, -0.0003847714538096606f);
  pl = fmaf(pl, u, 0.0064495445928312006f);
  pl = fmaf(pl, u, -0.05893596715178192f);
  pl = fmaf(pl, u, 0.3934098519357524f);
  const float c = __builtin_amdgcn_fmed3f(fmaf(v, pl, 0.5f), 0.f, 1.f);
  const float density = __builtin_amdgcn_exp2f(fmaf(u, -0.72134752044448170f, -1.3257480647361592f));      // exp(-u / 2) / sqrt(2 pi)
  *a = v * c;
  *da = fmaf(v, density, c);
}
// the activation, and a gradient g times its derivative
__device__ __forceinline__ void act_both(float v, int act, float* a, float* dg, float g) {
  float da;
  act_both(v, act, a, &da);
  *dg = g * da;
}

// Matrix-core operand fragment of a row-major LDS tile whose rows are the contraction index: lane (x = l % 32,
// hi = l / 32) gets rows 8 hi .. 8 hi + 7 of column x.  The transposing read works on groups of 16 lanes: lane i
// of a group points at four consecutive columns (4 (i % 4) ..) of row i / 4 and receives column i of the
// group's four rows.
typedef short s16x4 __attribute__((ext_vector_type(4)));
template <int PITCH>
__device__ __forceinline__ int frag_t_offset(int lane) {
  return (8 * (lane >> 5) + ((lane & 15) >> 2)) * PITCH + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
}
// s: the tile's element (first row, first column) plus frag_t_offset
template <int PITCH>
__device__ __forceinline__ bf16x8 frag_t(const __bf16* s) {
  typedef __attribute__((address_space(3))) s16x4 lds4;
  typedef short s16x8 __attribute__((ext_vector_type(8)));
  const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4*)s);
  const s16x4 up = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4*)(s + 4 * PITCH));
  const s16x8 v = __builtin_shufflevector(lo, up, 0, 1, 2, 3, 4, 5, 6, 7);
  return __builtin_bit_cast(bf16x8, v);
}

}  // namespace bw
}  // namespace longer
