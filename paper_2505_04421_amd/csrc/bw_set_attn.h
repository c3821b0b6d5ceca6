// Attention of the reduced stack (Section 3.5) for the backward pass: forward with the log-sum-exp kept, query
// side and key side of the gradient, over a user's own rows under the mask of Eq. 8, on the matrix cores.
//
// A wave owns 32 query rows (key rows on the key side) of one (user, head); a workgroup of four waves takes 128 of
// them and stages the other side's rows in LDS, kAttnChunk at a time.  With lane = query the scores come out of
// S^T = K Q^T as registers = keys, so softmax statistics are in-lane sums plus one exchange between the lane
// halves, and the probabilities (bf16) are the right operand of O^T = V^T P^T and of dQ^T = K^T dS^T as they stand;
// with lane = key the same holds for dV^T = dO^T P and dK^T = Q^T dS.  The transposed left operands are read from the
// row-major LDS tiles by the transposing LDS read.
//
// What bounds it: the exponentials and the score arithmetic around them (about 60 vector instructions per
// 32 x 32 scores against 4-6 matrix instructions, half empty at head width 16).  Row-per-thread loops over LDS rows, the
// kernels before these, were chains of dependent LDS reads: forward / query side / key side at the headline batch
// (256 users, 108 queries, 258 keys in the cross layer and 108 in three self layers) 276 / 322 / 336 us, now 89 / 166 / 121.
#pragma once
#include "bw_common.h"

namespace longer {
namespace bw {

// Every row carries a descriptor of its token: -1 invalid, a for global token a, kSeq + t for the sequence token
// with merged index t (a learnable query token stands after the newest one).
constexpr int kSeq = 1 << 24;
constexpr int kAttnRows = 128;      // rows of a workgroup
constexpr int kAttnChunk = 288;     // staged rows of the other side: m + T = 258 at the headline batch in one go

struct SetAttn {
  const __bf16* q; int qpitch;          // [B nq][..]
  const __bf16* k; const __bf16* v; int kvpitch;   // [B nk][..]
  const int* qdesc; const int* kdesc;
  int nq, nk, B, heads, gmask;
};

// Eq. 8 on descriptors, as one comparison: a key with order `ks` is visible to a query with limits (smax, gmax) iff
// ks <= (ks > 0 ? smax : gmax).  Sequence keys have their descriptor as order (> 0), global key a has -a,
// an invalid key stands above every limit.  A sequence query sees the sequence keys up to its own token and no
// global; a global query sees every sequence key and the globals of its set (causal: those with index >= its own).
constexpr int kNever = 0x7fffffff, kNothing = -0x7fffffff;
__device__ __forceinline__ int key_order(int kd) { return kd >= kSeq ? kd : (kd >= 0 ? -kd : kNever); }
__device__ __forceinline__ int query_smax(int qd) { return qd >= kSeq ? qd : (qd >= 0 ? kNever - 1 : kNothing); }
__device__ __forceinline__ int query_gmax(int qd, int gmask) {
  return (qd < 0 || qd >= kSeq) ? kNothing : (gmask == LONGER_GMASK_FULL ? 0 : -qd);
}

// Workgroup -> (user, head, 128 rows).  Workgroups go to the 8 accelerator dies round-robin, each with its own L2; a head's
// slice of a row is 32 or 64 bytes of a 128-byte line, so all heads of a user go to one die: with consecutive workgroups on
// different heads every die fetched every line (self layer of the headline batch, forward / query side / key side:
// 28 / 43 / 35 us, with a user on one die 18 / 34 / 23).
__device__ __forceinline__ bool attn_task(const SetAttn& a, int rounds, int* u, int* h, int* rd) {
  const int slot = blockIdx.x >> 3, per = a.heads * rounds, in = slot % per;
  *u = (slot / per) * 8 + (blockIdx.x & 7);
  *h = in / rounds; *rd = in - *h * rounds;
  return *u < a.B;
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
// the matrix-core operand of a row (lane = row, 8 features per lane half), straight from memory
template <int DH>
struct RowFrag {
  bf16x8 f[DH / 16];
  __device__ __forceinline__ void keep(bool wanted) {
#pragma unroll
    for (int g = 0; g < DH / 16; ++g) f[g] = keep_if(f[g], wanted);
  }
};
template <int DH>
__device__ __forceinline__ RowFrag<DH> row_frag(const __bf16* p, bool live, int hi) {
  RowFrag<DH> r;
#pragma unroll
  for (int g = 0; g < DH / 16; ++g) r.f[g] = keep_if(*(const bf16x8*)(p + 16 * g + 8 * hi), live);
  return r;
}
// rows [r0, r0 + 32) of an LDS tile (pitch DH) as the left operand, times a row operand: [rows] x [lanes]
template <int DH>
__device__ __forceinline__ f32x16 rows_times(const __bf16* s, int r0, const RowFrag<DH>& b, int l32, int hi) {
  f32x16 c;
#pragma unroll
  for (int r = 0; r < 16; ++r) c[r] = 0.f;
#pragma unroll
  for (int g = 0; g < DH / 16; ++g)
    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*(const bf16x8*)(s + (r0 + l32) * DH + 16 * g + 8 * hi), b.f[g], c, 0, 0, 0);
  return c;
}
// acc [features] x [lanes] += (rows [r0, r0 + 32) of the LDS tile)^T p, p = [rows] x [lanes] in accumulator layout: p's
// registers 8 g .. 8 g + 7 hold rows 16 g + 4 hi + (0..3) and 16 g + 8 + 4 hi + (0..3), and the left operand reads its rows
// in that order (head width 16: the upper half of its rows repeats the lower and is never looked at)
template <int DH>
__device__ __forceinline__ void add_transposed(f32x16& acc, const __bf16* s, int r0, const f32x16& p, int lane) {
  typedef __attribute__((address_space(3))) s16x4 lds4;
  typedef short s16x8 __attribute__((ext_vector_type(8)));
  const int hi = lane >> 5;
  const int off = (r0 + 4 * hi + ((lane & 15) >> 2)) * DH + (DH == 32 ? 16 * ((lane >> 4) & 1) : 0) + 4 * (lane & 3);
#pragma unroll
  for (int g = 0; g < 2; ++g) {
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4*)(s + off + 16 * g * DH));
    const s16x4 up = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4*)(s + off + (16 * g + 8) * DH));
    const s16x8 a = __builtin_shufflevector(lo, up, 0, 1, 2, 3, 4, 5, 6, 7);
    bf16x8 b;
#pragma unroll
    for (int e = 0; e < 8; ++e) b[e] = (__bf16)p[8 * g + e];
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), b, acc, 0, 0, 0);
  }
}
// acc holds [features] x [rows = lanes]: the lane's row, scaled
template <int DH>
__device__ __forceinline__ void store_row(__bf16* p, const f32x16& acc, float w, int hi) {
#pragma unroll
  for (int q = 0; q < DH / 8; ++q) {
    bf16x4 t;
#pragma unroll
    for (int e = 0; e < 4; ++e) t[e] = (__bf16)(acc[4 * q + e] * w);
    *(bf16x4*)(p + 8 * q + 4 * hi) = t;
  }
}
// n rows of a head on their way to LDS (at most N, n > 0), zeros up to the next multiple of 32
template <int DH, int N>
struct StagedRows {
  static constexpr int CP = DH / 8, NI = (N * CP + 255) / 256;
  bf16x8 v[NI];
  __device__ __forceinline__ void request(const __bf16* src, size_t pitch, int n) {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int c = threadIdx.x + 256 * i;
      v[i] = *(const bf16x8*)(src + (size_t)min(c / CP, n - 1) * pitch + 8 * (c % CP));
    }
  }
  __device__ __forceinline__ void put(__bf16* dst, int n) const {
    const int padded = (n + 31) / 32 * 32;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int c = threadIdx.x + 256 * i;
      if (c < padded * CP) *(bf16x8*)(dst + 8 * c) = keep_if(v[i], c / CP < n);
    }
  }
};

// Keys of a workgroup's (user, head) staged in LDS with their orders and each 32-key tile's smallest and largest order.
template <int DH>
struct KeyTiles {
  __bf16 k[kAttnChunk * DH], v[kAttnChunk * DH];
  int order[kAttnChunk], least[kAttnChunk / 32], most[kAttnChunk / 32];
};
template <int DH>
__device__ __forceinline__ void stage_keys(KeyTiles<DH>& t, const SetAttn& a, int u, int h, int c0, int n) {
  const size_t row0 = (size_t)u * a.nk + c0;
  constexpr int NT = (kAttnChunk / 32 + 3) / 4;      // key tiles of a wave
  StagedRows<DH, kAttnChunk> k, v;
  k.request(a.k + row0 * a.kvpitch + h * DH, a.kvpitch, n);
  v.request(a.v + row0 * a.kvpitch + h * DH, a.kvpitch, n);
  const int lane = threadIdx.x & 63, l32 = lane & 31, wave = threadIdx.x >> 6;
  int desc[NT];
#pragma unroll
  for (int i = 0; i < NT; ++i) desc[i] = a.kdesc[row0 + min((wave + 4 * i) * 32 + l32, n - 1)];
  k.put(t.k, n);
  v.put(t.v, n);
#pragma unroll
  for (int i = 0; i < NT; ++i) {
    const int kt = wave + 4 * i, j = kt * 32 + l32, ks = j < n ? key_order(desc[i]) : kNever;
    if (kt * 32 >= n) continue;
    int lo = ks, up = ks;
#pragma unroll
    for (int o = 16; o > 0; o >>= 1) { lo = min(lo, __shfl_xor(lo, o, 64)); up = max(up, __shfl_xor(up, o, 64)); }
    if (lane < 32) t.order[j] = ks;
    if (lane == 0) { t.least[kt] = lo; t.most[kt] = up; }
  }
}
// Does any lane's query see a key of tile kt (`none` otherwise), and must single keys be tested?  (A lane without a
// query sees nothing and wants nothing tested: what it computes is dropped.)
template <int DH>
__device__ __forceinline__ void tile_visibility(const KeyTiles<DH>& t, int kt, bool live, int smax, bool* none, bool* test) {
  const int lo = t.least[kt], up = t.most[kt];
  *none = lo > 0 && __builtin_amdgcn_ballot_w64(live && lo <= smax) == 0;
  *test = lo <= 0 || __builtin_amdgcn_ballot_w64(live && up > smax) != 0;
}
// scores of keys the lane's query does not see become -infinity
template <int DH>
__device__ __forceinline__ void mask_scores(f32x16& s, const KeyTiles<DH>& t, int kt, int smax, int gmax, int hi) {
  typedef int i32x4 __attribute__((ext_vector_type(4)));
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const i32x4 ks = *(const i32x4*)(t.order + 32 * kt + 8 * q + 4 * hi);
#pragma unroll
    for (int e = 0; e < 4; ++e) s[4 * q + e] = ks[e] <= (ks[e] > 0 ? smax : gmax) ? s[4 * q + e] : -__builtin_inff();
  }
}

// o[row][h] = softmax over the visible keys (q . k / sqrt(DH)) v, zeros for a row without one; stat[row][h].x = the
// log-sum-exp of its scores in units of log 2 (+infinity without a key: every probability taken from it is zero).
template <int DH>
__global__ __launch_bounds__(256) void bw_set_attn_fwd_kernel(SetAttn a, __bf16* __restrict__ o, int d, float2* __restrict__ stat) {
  __shared__ __attribute__((aligned(16))) KeyTiles<DH> t;
  const int rounds = (a.nq + kAttnRows - 1) / kAttnRows;
  int u, h, rd;
  if (!attn_task(a, rounds, &u, &h, &rd)) return;
  const int lane = threadIdx.x & 63, l32 = lane & 31, hi = lane >> 5;
  const int i0 = rd * kAttnRows + 32 * (threadIdx.x >> 6), i = i0 + l32;
  const size_t row = (size_t)u * a.nq + (i < a.nq ? i : 0);
  int qd = a.qdesc[row];
  RowFrag<DH> q = row_frag<DH>(a.q + row * a.qpitch + h * DH, true, hi);
  if (i >= a.nq) qd = -1;
  const bool live = qd >= 0;
  q.keep(live);
  const int smax = query_smax(qd), gmax = query_gmax(qd, a.gmask);
  const float c = 1.4426950408889634f * rsqrtf((float)DH);
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  float m = kNegBig, l = 0.f;
  for (int c0 = 0; c0 < a.nk; c0 += kAttnChunk) {
    const int n = min(kAttnChunk, a.nk - c0);
    if (c0) __syncthreads();
    stage_keys<DH>(t, a, u, h, c0, n);
    __syncthreads();
    if (i0 >= a.nq) continue;
    for (int kt = 0; kt * 32 < n; ++kt) {
      bool none, test;
      tile_visibility<DH>(t, kt, live, smax, &none, &test);
      if (none) continue;
      f32x16 s = rows_times<DH>(t.k, 32 * kt, q, l32, hi);
      if (test) mask_scores<DH>(s, t, kt, smax, gmax, hi);
      float mt = s[0];
#pragma unroll
      for (int r = 1; r < 16; ++r) mt = fmaxf(mt, s[r]);
      const float mn = fmaxf(m, max_halves(mt) * c), alpha = __builtin_amdgcn_exp2f(m - mn);
      m = mn;
      acc *= alpha;
      float lt = 0.f;
#pragma unroll
      for (int r = 0; r < 16; ++r) { s[r] = __builtin_amdgcn_exp2f(fmaf(s[r], c, -mn)); lt += s[r]; }
      l = fmaf(l, alpha, lt);
      add_transposed<DH>(acc, t.v, 32 * kt, s, lane);
    }
  }
  l = sum_halves(l);
  if (i >= a.nq) return;
  const bool any = live && l > 0.f;
  store_row<DH>(o + row * d + h * DH, acc, any ? 1.f / l : 0.f, hi);
  if (hi == 0) stat[row * a.heads + h] = make_float2(any ? m + __builtin_amdgcn_logf(l) : __builtin_inff(), 0.f);
}

// Query side of the gradient: P_ij = exp2(c s_ij - lse_i), dP_ij = do_i . v_j, D_i = sum_j P_ij dP_ij (to stat[].y),
// dq_i = sum_j P_ij (dP_ij - D_i) k_j / sqrt(DH).  Two passes over the keys: D first.
template <int DH>
__global__ __launch_bounds__(256) void bw_set_attn_bwd_q_kernel(SetAttn a, const __bf16* __restrict__ dob, int d,
                                                                __bf16* __restrict__ dq, int dqpitch, float2* __restrict__ stat) {
  __shared__ __attribute__((aligned(16))) KeyTiles<DH> t;
  const int rounds = (a.nq + kAttnRows - 1) / kAttnRows;
  int u, h, rd;
  if (!attn_task(a, rounds, &u, &h, &rd)) return;
  const int lane = threadIdx.x & 63, l32 = lane & 31, hi = lane >> 5;
  const int i0 = rd * kAttnRows + 32 * (threadIdx.x >> 6), i = i0 + l32;
  const size_t row = (size_t)u * a.nq + (i < a.nq ? i : 0);
  int qd = a.qdesc[row];
  float lse = stat[row * a.heads + h].x;
  RowFrag<DH> q = row_frag<DH>(a.q + row * a.qpitch + h * DH, true, hi), g = row_frag<DH>(dob + row * d + h * DH, true, hi);
  if (i >= a.nq) { qd = -1; lse = __builtin_inff(); }
  const bool live = qd >= 0;
  q.keep(live); g.keep(live);
  const int smax = query_smax(qd), gmax = query_gmax(qd, a.gmask);
  const float scale = rsqrtf((float)DH), c = 1.4426950408889634f * scale;
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  float D = 0.f;
  for (int pass = 0; pass < 2; ++pass) {
    for (int c0 = 0; c0 < a.nk; c0 += kAttnChunk) {
      const int n = min(kAttnChunk, a.nk - c0);
      if (pass == 0 || a.nk > kAttnChunk) {       // (a single chunk stays for the second pass)
        if (pass || c0) __syncthreads();
        stage_keys<DH>(t, a, u, h, c0, n);
        __syncthreads();
      }
      if (i0 >= a.nq) continue;
      for (int kt = 0; kt * 32 < n; ++kt) {
        bool none, test;
        tile_visibility<DH>(t, kt, live, smax, &none, &test);
        if (none) continue;
        f32x16 s = rows_times<DH>(t.k, 32 * kt, q, l32, hi);
        const f32x16 dp = rows_times<DH>(t.v, 32 * kt, g, l32, hi);
        if (test) mask_scores<DH>(s, t, kt, smax, gmax, hi);
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = __builtin_amdgcn_exp2f(fmaf(s[r], c, -lse));
        if (pass == 0) {
#pragma unroll
          for (int r = 0; r < 16; ++r) D = fmaf(s[r], dp[r], D);
        } else {
#pragma unroll
          for (int r = 0; r < 16; ++r) s[r] *= dp[r] - D;
          add_transposed<DH>(acc, t.k, 32 * kt, s, lane);
        }
      }
    }
    if (pass == 0) D = sum_halves(D);
  }
  if (i >= a.nq) return;
  store_row<DH>(dq + row * dqpitch + h * DH, acc, live ? scale : 0.f, hi);
  if (hi == 0) stat[row * a.heads + h].y = live ? D : 0.f;
}

// Key side: dv_j = sum_i P_ij do_i, dk_j = sum_i P_ij (dP_ij - D_i) q_i / sqrt(DH), over the user's query rows.
template <int DH>
__global__ __launch_bounds__(256) void bw_set_attn_bwd_kv_kernel(SetAttn a, const __bf16* __restrict__ dob, int d,
                                                                 __bf16* __restrict__ dk, __bf16* __restrict__ dv, int dkvpitch,
                                                                 const float2* __restrict__ stat) {
  constexpr int CH = 128;       // staged query rows
  __shared__ __attribute__((aligned(16))) struct {
    __bf16 q[CH * DH], g[CH * DH];
    float lse[CH], D[CH];
    int smax[CH], gmax[CH];
    int least[CH / 32], most[CH / 32], gmost[CH / 32];      // per 32-row tile: limits of its queries
  } t;
  typedef int i32x4 __attribute__((ext_vector_type(4)));
  const int rounds = (a.nk + kAttnRows - 1) / kAttnRows;
  int u, h, rd;
  if (!attn_task(a, rounds, &u, &h, &rd)) return;
  const int lane = threadIdx.x & 63, l32 = lane & 31, hi = lane >> 5;
  const int j0 = rd * kAttnRows + 32 * (threadIdx.x >> 6), j = j0 + l32;
  const size_t row = (size_t)u * a.nk + (j < a.nk ? j : 0);
  const int kd = a.kdesc[row];
  RowFrag<DH> kf = row_frag<DH>(a.k + row * a.kvpitch + h * DH, true, hi), vf = row_frag<DH>(a.v + row * a.kvpitch + h * DH, true, hi);
  const int ks = j < a.nk ? key_order(kd) : kNever;
  const bool live = ks != kNever;
  kf.keep(live); vf.keep(live);
  const float scale = rsqrtf((float)DH), c = 1.4426950408889634f * scale;
  f32x16 gk, gv;
#pragma unroll
  for (int r = 0; r < 16; ++r) { gk[r] = 0.f; gv[r] = 0.f; }
  for (int c0 = 0; c0 < a.nq; c0 += CH) {
    const int n = min(CH, a.nq - c0);
    const size_t q0 = (size_t)u * a.nq + c0;
    if (c0) __syncthreads();
    StagedRows<DH, CH> sq, sg;
    sq.request(a.q + q0 * a.qpitch + h * DH, a.qpitch, n);
    sg.request(dob + q0 * d + h * DH, d, n);
    static_assert(CH == 128, "a query tile a wave");
    const int qt = threadIdx.x >> 6, i = qt * 32 + l32, ic = min(i, n - 1);
    int qd = a.qdesc[q0 + ic];
    float2 st = stat[(q0 + ic) * a.heads + h];
    sq.put(t.q, n);
    sg.put(t.g, n);
    if (qt * 32 < n) {
      if (i >= n) qd = -1;
      // a row without a query: log-sum-exp +infinity, so that its probabilities are exact zeros untested
      if (qd < 0) st = make_float2(__builtin_inff(), 0.f);
      const int sm = query_smax(qd), gm = query_gmax(qd, a.gmask);
      int lo = qd >= 0 ? sm : kNever, up = sm, gu = gm;
#pragma unroll
      for (int o = 16; o > 0; o >>= 1) {
        lo = min(lo, __shfl_xor(lo, o, 64)); up = max(up, __shfl_xor(up, o, 64)); gu = max(gu, __shfl_xor(gu, o, 64));
      }
      if (lane < 32) { t.lse[i] = st.x; t.D[i] = st.y; t.smax[i] = sm; t.gmax[i] = gm; }
      if (lane == 0) { t.least[qt] = lo; t.most[qt] = up; t.gmost[qt] = gu; }
    }
    __syncthreads();
    if (j0 >= a.nk) continue;
    for (int qt = 0; qt * 32 < n; ++qt) {
      if (__builtin_amdgcn_ballot_w64(live && ks <= (ks > 0 ? t.most[qt] : t.gmost[qt])) == 0) continue;     // seen by no query
      const bool test = __builtin_amdgcn_ballot_w64(live && (ks <= 0 || ks > t.least[qt])) != 0;
      f32x16 p = rows_times<DH>(t.q, 32 * qt, kf, l32, hi);
      f32x16 ds = rows_times<DH>(t.g, 32 * qt, vf, l32, hi);
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        const f32x4 lse = *(const f32x4*)(t.lse + 32 * qt + 8 * q4 + 4 * hi), D = *(const f32x4*)(t.D + 32 * qt + 8 * q4 + 4 * hi);
        if (test) {
          const i32x4 sm = *(const i32x4*)(t.smax + 32 * qt + 8 * q4 + 4 * hi), gm = *(const i32x4*)(t.gmax + 32 * qt + 8 * q4 + 4 * hi);
#pragma unroll
          for (int e = 0; e < 4; ++e) p[4 * q4 + e] = ks <= (ks > 0 ? sm[e] : gm[e]) ? p[4 * q4 + e] : -__builtin_inff();
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          p[4 * q4 + e] = __builtin_amdgcn_exp2f(fmaf(p[4 * q4 + e], c, -lse[e]));
          ds[4 * q4 + e] = p[4 * q4 + e] * (ds[4 * q4 + e] - D[e]);
        }
      }
      add_transposed<DH>(gv, t.g, 32 * qt, p, lane);
      add_transposed<DH>(gk, t.q, 32 * qt, ds, lane);
    }
  }
  if (j >= a.nk) return;
  store_row<DH>(dk + row * dkvpitch + h * DH, gk, live ? scale : 0.f, hi);
  store_row<DH>(dv + row * dkvpitch + h * DH, gv, live ? 1.f : 0.f, hi);
}

// which: 0 forward (o), 1 query side (dq), 2 key side (dk, dv)
template <int DH>
static void set_attn_launch(hipStream_t st, int which, const SetAttn& a, const __bf16* dob, int d, __bf16* o_or_dq, int pitch,
                            __bf16* dk, __bf16* dv, float2* stat) {
  const unsigned uh = (unsigned)((a.B + 7) / 8 * 8 * a.heads);      // (see attn_task)
  const unsigned gq = uh * ((a.nq + kAttnRows - 1) / kAttnRows), gk = uh * ((a.nk + kAttnRows - 1) / kAttnRows);
  if (which == 0) bw_set_attn_fwd_kernel<DH><<<gq, 256, 0, st>>>(a, o_or_dq, d, stat);
  else if (which == 1) bw_set_attn_bwd_q_kernel<DH><<<gq, 256, 0, st>>>(a, dob, d, o_or_dq, pitch, stat);
  else bw_set_attn_bwd_kv_kernel<DH><<<gk, 256, 0, st>>>(a, dob, d, dk, dv, pitch, stat);
}

}  // namespace bw
}  // namespace longer
