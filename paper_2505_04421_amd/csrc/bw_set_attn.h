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
// 32 x 32 scores against 4-6 matrix instructions, half empty at head width 16), and, with two to nine of these squares a wave, what a workgroup does
// before its first: requests, addresses, the tiles' ranges.  Row-per-thread loops over LDS rows, the
// kernels before these, were chains of dependent LDS reads: forward / query side / key side at the headline batch
// (256 users, 108 queries, 258 keys in the cross layer and 108 in three self layers) 276 / 322 / 336 us, these 86 / 125 / 111 as kernels of their
// own; both sides in one 195, with their start made cheaper (ranges without LDS, all requests ahead of the first use, 32-bit addresses, no zeros behind the last row)
// and a self layer's probabilities alone held, 167 and the forward 80.
#pragma once
#include "bw_common.h"

namespace longer {
namespace bw {

using longer::settle;

constexpr int kAttnRows = 128;      // rows of a workgroup
constexpr int kAttnChunk = 288;     // staged rows of the other side: m + T = 258 at the headline batch in one go

struct SetAttn {
  const __bf16* q; int qpitch;          // [B qrows][..]
  const __bf16* k; const __bf16* v; int kvpitch;   // [B nk][..]
  const int* qdesc; const int* kdesc;
  int nq, nk, B, heads, gmask;
  int qrows;                            // a user's rows in q, qdesc and what goes with them (outputs, statistics, gradients): the first nq are queries
};

// Eq. 8 on descriptors: a key stands at a position (global token a at a - kSeq, sequence token t at t, an invalid one behind
// everything) and a query sees one interval of them, so that a key is tested by a subtraction and an unsigned comparison.  (A second form without the
// subtraction, for tiles without a global query, cost the forward and query sides 5 to 10 % where it was not taken, and gave nothing where it was.)  A sequence query sees the sequence keys up to its own
// token and no global; a global query sees every sequence key and the globals of its set (causal: those with index >= its own).
constexpr int kNone = 0x7fffffff - kSeq;
__device__ __forceinline__ int key_position(int kd) { return kd >= 0 ? kd - kSeq : kNone; }
struct Seen { int lo, end; };              // positions lo .. end - 1 (no query: none)
__device__ __forceinline__ Seen query_sees(int qd, int gmask) {
  if (qd < 0) return {0, 0};
  if (qd >= kSeq) return {0, qd - kSeq + 1};
  return {gmask == LONGER_GMASK_FULL ? -kSeq : qd - kSeq, kNone};
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

__device__ __forceinline__ void settle(f32x16& a, f32x16& b) { asm volatile("s_nop 10" : "+v"(a), "+v"(b)); }      // (device.h, for two)

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
// acc holds [features] x [rows = lanes]: the lane's row, scaled; w = 0: zeros, whatever the lane holds (a key row without a token has infinite
// probabilities where a query's log-sum-exp lies below -128)
template <int DH>
__device__ __forceinline__ void store_row(__bf16* p, const f32x16& acc, float w, int hi) {
#pragma unroll
  for (int q = 0; q < DH / 8; ++q) {
    bf16x4 t;
#pragma unroll
    for (int e = 0; e < 4; ++e) t[e] = (__bf16)(w != 0.f ? acc[4 * q + e] * w : 0.f);
    *(bf16x4*)(p + 8 * q + 4 * hi) = t;
  }
}
// n rows of a head on their way to LDS (at most N, n > 0); behind them the last one again, whose weights there are exact zeros
template <int DH, int N>
struct StagedRows {
  static constexpr int CP = DH / 8, NI = (N * CP + 255) / 256;
  bf16x8 v[NI];
  __device__ __forceinline__ void request(const __bf16* src, int pitch, int n) {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int c = threadIdx.x + 256 * i;
      v[i] = *(const bf16x8*)((const char*)src + (uint32_t)(2 * (min(c / CP, n - 1) * pitch + 8 * (c % CP))));
    }
  }
  __device__ __forceinline__ void put(__bf16* dst) const {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int c = threadIdx.x + 256 * i;
      if (256 * (i + 1) <= N * CP || c < N * CP) *(bf16x8*)(dst + 8 * c) = v[i];
    }
  }
};

// The smallest a and the largest b of 32 lanes (both lane halves hold the same): the lower half looks for the one and the upper for the
// smallest ~b, within rows of 16 lanes by data-parallel moves, and a lane of each row is read out.  (Shuffles go through LDS: ten in a row,
// a tenth of a workgroup's life.)
struct Range { int least, most; };
template <int CTRL> __device__ __forceinline__ int min_with(int v) { return min(v, __builtin_amdgcn_update_dpp(v, v, CTRL, 0xf, 0xf, false)); }
__device__ __forceinline__ Range range_of(int a, int b) {
  int v = threadIdx.x & 32 ? ~b : a;
  v = min_with<0x140>(min_with<0x141>(min_with<0x4e>(min_with<0xb1>(v))));      // lane ^ 1, ^ 2, mirrored in 8, in 16
  return {min(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)), ~min(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48))};
}
// all that was requested is on its way before any of it is used (what is used under a condition came to be requested under it)
__device__ __forceinline__ void all_requested() { asm volatile("" ::: "memory"); }

// Keys of a workgroup's (user, head) staged in LDS with their positions and each 32-key tile's smallest and largest one.
template <int DH, int N>
struct KeyTiles {
  __bf16 k[N * DH], v[N * DH];
  int pos[N], least[N / 32], most[N / 32];
};
// n of them (at most N) on their way there
template <int DH, int N>
struct StagedKeys {
  static constexpr int NT = (N / 32 + 3) / 4;      // key tiles of a wave
  StagedRows<DH, N> k, v;
  int desc[NT];
  __device__ __forceinline__ void request(const SetAttn& a, int u, int h, int c0, int n) {
    const size_t row0 = (size_t)u * a.nk + c0;
    k.request(a.k + row0 * a.kvpitch + h * DH, a.kvpitch, n);
    v.request(a.v + row0 * a.kvpitch + h * DH, a.kvpitch, n);
#pragma unroll
    for (int i = 0; i < NT; ++i) desc[i] = a.kdesc[row0 + min(((int)(threadIdx.x >> 6) + 4 * i) * 32 + (int)(threadIdx.x & 31), n - 1)];
  }
  __device__ __forceinline__ void put(KeyTiles<DH, N>& t, int n) const {
    const int lane = threadIdx.x & 63, l32 = lane & 31, wave = threadIdx.x >> 6;
    k.put(t.k);
    v.put(t.v);
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      const int kt = wave + 4 * i, j = kt * 32 + l32, ks = j < n ? key_position(desc[i]) : kNone;
      if (kt * 32 >= n) continue;
      const Range range = range_of(ks, ks);
      if (lane < 32) t.pos[j] = ks;
      if (lane == 0) { t.least[kt] = range.least; t.most[kt] = range.most; }
    }
  }
};
template <int DH, int N>
__device__ __forceinline__ void stage_keys(KeyTiles<DH, N>& t, const SetAttn& a, int u, int h, int c0, int n) {
  StagedKeys<DH, N> s;
  s.request(a, u, h, c0, n);
  all_requested();
  s.put(t, n);
}
// What the 32 queries of a tile see: the positions that some of them sees (least .. most - 1), and those that all see (start .. end - 1).  A lane
// without a query sees nothing and wants nothing tested: what it computes is dropped.
struct Span { int least, most, start, end; };
__device__ __forceinline__ Span span_of(bool live, const Seen& see) {
  const Range some = range_of(live ? see.lo : kNone, live ? see.end : -kSeq), all = range_of(live ? see.end : kNone, live ? see.lo : -kSeq);
  return {some.least, some.most, all.most, all.least};
}
// bit kt of `some`: a key of tile kt may be seen; of `test`: single keys must be tested
struct Tiles { uint32_t some, test; };
template <int DH, int N>
__device__ __forceinline__ Tiles key_tiles(const KeyTiles<DH, N>& t, int n, const Span& q) {
  const int lane = threadIdx.x & 63, kt = min(lane, N / 32 - 1), lo = t.least[kt], up = t.most[kt];
  const bool in = lane * 32 < n;
  return {(uint32_t)__builtin_amdgcn_ballot_w64(in && lo < q.most && up >= q.least), (uint32_t)__builtin_amdgcn_ballot_w64(in && (lo < q.start || up >= q.end))};
}
// scores of keys the lane's query does not see become -infinity
template <int DH, int N>
__device__ __forceinline__ void mask_scores(f32x16& s, const KeyTiles<DH, N>& t, int kt, const Seen& see, int hi) {
  typedef int i32x4 __attribute__((ext_vector_type(4)));
  const unsigned width = (unsigned)(see.end - see.lo);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const i32x4 ks = *(const i32x4*)(t.pos + 32 * kt + 8 * q + 4 * hi);
#pragma unroll
    for (int e = 0; e < 4; ++e) s[4 * q + e] = (unsigned)(ks[e] - see.lo) < width ? s[4 * q + e] : -__builtin_inff();
  }
}

// o[row][h] = softmax over the visible keys (q . k / sqrt(DH)) v, zeros for a row without one; stat[row][h].x = the
// log-sum-exp of its scores in units of log 2 (+infinity without a key: every probability taken from it is zero).
template <int DH>
__global__ __launch_bounds__(256) void bw_set_attn_fwd_kernel(SetAttn a, __bf16* __restrict__ o, int d, float2* __restrict__ stat) {
  __shared__ __attribute__((aligned(16))) KeyTiles<DH, kAttnChunk> t;
  const int rounds = (a.nq + kAttnRows - 1) / kAttnRows;
  int u, h, rd;
  if (!attn_task(a, rounds, &u, &h, &rd)) return;
  const int lane = threadIdx.x & 63, l32 = lane & 31, hi = lane >> 5;
  const int i0 = rd * kAttnRows + 32 * (threadIdx.x >> 6), i = i0 + l32;
  const size_t row = (size_t)u * a.qrows + (i < a.nq ? i : 0);
  int qd = a.qdesc[row];
  RowFrag<DH> q = row_frag<DH>(a.q + row * a.qpitch + h * DH, true, hi);
  if (i >= a.nq) qd = -1;
  const bool live = qd >= 0;
  q.keep(live);
  const Seen see = query_sees(qd, a.gmask);
  const Span span = span_of(live, see);
  const float c = 1.4426950408889634f * rsqrtf((float)DH);
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  float m = kNegBig, l = 0.f;
  for (int c0 = 0; c0 < a.nk; c0 += kAttnChunk) {
    const int n = min(kAttnChunk, a.nk - c0);
    if (c0) __syncthreads();
    stage_keys(t, a, u, h, c0, n);
    __syncthreads();
    if (i0 >= a.nq) continue;
    const Tiles tiles = key_tiles(t, n, span);
    for (uint32_t left = tiles.some; left; left &= left - 1) {
      const int kt = __builtin_ctz(left);
      f32x16 s = rows_times<DH>(t.k, 32 * kt, q, l32, hi);
      settle(s);                                       // (a branch follows: device.h)
      if (tiles.test >> kt & 1) mask_scores(s, t, kt, see, hi);
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
  settle(acc);
  if (i >= a.nq) return;
  const bool any = live && l > 0.f;
  store_row<DH>(o + row * d + h * DH, acc, any ? 1.f / l : 0.f, hi);
  if (hi == 0) stat[row * a.heads + h] = make_float2(any ? m + __builtin_amdgcn_logf(l) : __builtin_inff(), 0.f);
}

// Query side of the gradient: P_ij = exp2(c s_ij - lse_i), dP_ij = do_i . v_j, D_i = sum_j P_ij dP_ij,
// dq_i = sum_j P_ij (dP_ij - D_i) k_j / sqrt(DH).  Two passes over the keys: D first.
// At most kHeldTiles key tiles (a self layer's): their P stay in registers for the second pass, 64 of them, so that four waves still share a
// SIMD; dP is formed again, a matrix product of a few cycles.  (With dP held as well, three waves a SIMD: three self layers of the headline batch 116 us, so 96.
// Beyond four tiles, the first four held and the others formed again: ten registers spilled, and no faster.)
constexpr int kHeldTiles = 4;
template <int DH, int N>
__device__ __forceinline__ void query_side_held(const KeyTiles<DH, N>& t, int nk, const RowFrag<DH>& q, const RowFrag<DH>& g, const Span& span, const Seen& see,
                                                float lse, float c, float& D, f32x16& acc, int lane) {
  const int l32 = lane & 31, hi = lane >> 5;
  f32x16 P[kHeldTiles];
  const Tiles tiles = key_tiles(t, nk, span);
#pragma unroll
  for (int kt = 0; kt < kHeldTiles; ++kt) {
    if (!(tiles.some >> kt & 1)) continue;
    P[kt] = rows_times<DH>(t.k, 32 * kt, q, l32, hi);
    f32x16 dp = rows_times<DH>(t.v, 32 * kt, g, l32, hi);
    settle(P[kt], dp);
    if (tiles.test >> kt & 1) mask_scores(P[kt], t, kt, see, hi);
#pragma unroll
    for (int r = 0; r < 16; ++r) { P[kt][r] = __builtin_amdgcn_exp2f(fmaf(P[kt][r], c, -lse)); D = fmaf(P[kt][r], dp[r], D); }
  }
  D = sum_halves(D);
#pragma unroll
  for (int kt = 0; kt < kHeldTiles; ++kt) {
    if (!(tiles.some >> kt & 1)) continue;
    f32x16 dp = rows_times<DH>(t.v, 32 * kt, g, l32, hi);
    settle(dp);
#pragma unroll
    for (int r = 0; r < 16; ++r) P[kt][r] *= dp[r] - D;
    add_transposed<DH>(acc, t.k, 32 * kt, P[kt], lane);
  }
}
// one pass over n staged keys: D (SECOND: dq, D known)
template <bool SECOND, int DH, int N>
__device__ __forceinline__ void query_side_pass(const KeyTiles<DH, N>& t, int n, const RowFrag<DH>& q, const RowFrag<DH>& g, const Span& span, const Seen& see,
                                                float lse, float c, float& D, f32x16& acc, int lane) {
  const int l32 = lane & 31, hi = lane >> 5;
  const Tiles tiles = key_tiles(t, n, span);
  for (uint32_t left = tiles.some; left; left &= left - 1) {
    const int kt = __builtin_ctz(left);
    f32x16 s = rows_times<DH>(t.k, 32 * kt, q, l32, hi);
    f32x16 dp = rows_times<DH>(t.v, 32 * kt, g, l32, hi);
    settle(s, dp);
    if (tiles.test >> kt & 1) mask_scores(s, t, kt, see, hi);
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = __builtin_amdgcn_exp2f(fmaf(s[r], c, -lse));
    if constexpr (!SECOND) {
#pragma unroll
      for (int r = 0; r < 16; ++r) D = fmaf(s[r], dp[r], D);
    } else {
#pragma unroll
      for (int r = 0; r < 16; ++r) s[r] *= dp[r] - D;
      add_transposed<DH>(acc, t.k, 32 * kt, s, lane);
    }
  }
}

// Query rows of a workgroup's (user, head) staged in LDS, a tile a wave, with the upstream gradient of their output, their
// statistics and what they see.
constexpr int kQueryRows = 128;
template <int DH>
struct QueryTiles {
  __bf16 q[kQueryRows * DH], g[kQueryRows * DH];
  float lse[kQueryRows], D[kQueryRows];
  int lo[kQueryRows], width[kQueryRows];
  Span span[kQueryRows / 32];
};
template <int DH>
struct StagedQueries {
  StagedRows<DH, kQueryRows> q, g;
  int qd;
  float2 st;
  __device__ __forceinline__ void request(const SetAttn& a, const __bf16* dob, int d, const float2* stat, int u, int h, int c0, int n) {
    const size_t q0 = (size_t)u * a.qrows + c0;
    q.request(a.q + q0 * a.qpitch + h * DH, a.qpitch, n);
    g.request(dob + q0 * d + h * DH, d, n);
    const int ic = min((int)(threadIdx.x >> 6) * 32 + (int)(threadIdx.x & 31), n - 1);
    qd = a.qdesc[q0 + ic];
    st = stat[(q0 + ic) * a.heads + h];
  }
  __device__ __forceinline__ void put(QueryTiles<DH>& t, int gmask, int n) {
    const int lane = threadIdx.x & 63, qt = threadIdx.x >> 6, i = qt * 32 + (lane & 31);
    q.put(t.q);
    g.put(t.g);
    if (qt * 32 >= n) return;
    if (i >= n) qd = -1;
    // a row without a query: log-sum-exp +infinity, so that its probabilities are exact zeros untested
    if (qd < 0) st = make_float2(__builtin_inff(), 0.f);
    const Seen see = query_sees(qd, gmask);
    const Span span = span_of(qd >= 0, see);
    if (lane < 32) { t.lse[i] = st.x; t.D[i] = st.y; t.lo[i] = see.lo; t.width[i] = see.end - see.lo; }
    if (lane == 0) t.span[qt] = span;
  }
};
// Key side: dv_j = sum_i P_ij do_i, dk_j = sum_i P_ij (dP_ij - D_i) q_i / sqrt(DH), over n staged query rows; the lane's key stands at ks.
template <int DH>
__device__ __forceinline__ void key_side(const QueryTiles<DH>& t, int n, const RowFrag<DH>& kf, const RowFrag<DH>& vf, int ks, float c,
                                         f32x16& gk, f32x16& gv, int lane) {
  typedef int i32x4 __attribute__((ext_vector_type(4)));
  const int l32 = lane & 31, hi = lane >> 5;
  const Range keys = range_of(ks, ks != kNone ? ks : -kSeq - 1);
  const Span span = t.span[min(lane, kQueryRows / 32 - 1)];
  const uint32_t some = (uint32_t)__builtin_amdgcn_ballot_w64(lane * 32 < n && keys.least < span.most && keys.most >= span.least);      // (bit qt: may be seen by a query of the tile)
  const uint32_t tested = (uint32_t)__builtin_amdgcn_ballot_w64(lane * 32 < n && (keys.least < span.start || keys.most >= span.end));
  for (uint32_t left = some; left; left &= left - 1) {
    const int qt = __builtin_ctz(left);
    f32x16 p = rows_times<DH>(t.q, 32 * qt, kf, l32, hi);
    f32x16 ds = rows_times<DH>(t.g, 32 * qt, vf, l32, hi);
    settle(p, ds);
    if (tested >> qt & 1) {
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        const i32x4 width = *(const i32x4*)(t.width + 32 * qt + 8 * q4 + 4 * hi), lo = *(const i32x4*)(t.lo + 32 * qt + 8 * q4 + 4 * hi);
#pragma unroll
        for (int e = 0; e < 4; ++e) p[4 * q4 + e] = (unsigned)(ks - lo[e]) < (unsigned)width[e] ? p[4 * q4 + e] : -__builtin_inff();
      }
    }
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      const f32x4 lse = *(const f32x4*)(t.lse + 32 * qt + 8 * q4 + 4 * hi), D = *(const f32x4*)(t.D + 32 * qt + 8 * q4 + 4 * hi);
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

// Both sides of a (user, head) whose queries fit one workgroup and whose keys fit LDS: every row is fetched once and D stays here.  (A launch a side,
// as beyond these sizes: three self layers and the cross layer of the headline batch 137 + 99 us, so 96 + 71.)
template <int DH, bool HELD>
__global__ __launch_bounds__(256, 4) void bw_set_attn_bwd_kernel(SetAttn a, const __bf16* __restrict__ dob, int d, __bf16* __restrict__ dq, int dqpitch,
                                                                            __bf16* __restrict__ dk, __bf16* __restrict__ dv, int dkvpitch,
                                                                            const float2* stat) {
  constexpr int N = HELD ? 32 * kHeldTiles : kAttnChunk;
  __shared__ __attribute__((aligned(16))) KeyTiles<DH, N> t;
  __shared__ __attribute__((aligned(16))) QueryTiles<DH> s;
  int u, h, rd;
  if (!attn_task(a, 1, &u, &h, &rd)) return;
  const int lane = threadIdx.x & 63, l32 = lane & 31, hi = lane >> 5, wave = threadIdx.x >> 6;
  {
    StagedKeys<DH, N> keys;
    StagedQueries<DH> queries;
    queries.request(a, dob, d, stat, u, h, 0, a.nq);
    keys.request(a, u, h, 0, a.nk);
    all_requested();
    queries.put(s, a.gmask, a.nq);
    keys.put(t, a.nk);
  }
  __syncthreads();
  const float scale = rsqrtf((float)DH), c = 1.4426950408889634f * scale;
  if (32 * wave < a.nq) {
    const int i = 32 * wave + l32, lo = s.lo[i], width = s.width[i];
    const bool live = width != 0;      // (a query sees an interval of some length, no query one of none)
    const Seen see = {lo, lo + width};
    const Span span = s.span[wave];
    RowFrag<DH> q = row_frag<DH>(s.q + i * DH, live, hi), g = row_frag<DH>(s.g + i * DH, live, hi);
    const float lse = s.lse[i];
    f32x16 acc = splat16(0.f);
    float D = 0.f;
    if constexpr (HELD) query_side_held(t, a.nk, q, g, span, see, lse, c, D, acc, lane);
    else {
      query_side_pass<false>(t, a.nk, q, g, span, see, lse, c, D, acc, lane);
      D = sum_halves(D);
      query_side_pass<true>(t, a.nk, q, g, span, see, lse, c, D, acc, lane);
    }
    settle(acc);
    if (hi == 0) s.D[i] = live ? D : 0.f;
    if (i < a.nq) store_row<DH>(dq + ((size_t)u * a.qrows + i) * dqpitch + h * DH, acc, live ? scale : 0.f, hi);
  }
  __syncthreads();
  for (int kt = wave; kt * 32 < a.nk; kt += 4) {
    const int j = 32 * kt + l32, ks = t.pos[j];
    const bool live = ks != kNone;
    const RowFrag<DH> kf = row_frag<DH>(t.k + j * DH, live, hi), vf = row_frag<DH>(t.v + j * DH, live, hi);
    f32x16 gk = splat16(0.f), gv = splat16(0.f);
    key_side(s, a.nq, kf, vf, ks, c, gk, gv, lane);
    settle(gk, gv);
    if (j >= a.nk) continue;
    const size_t row = (size_t)u * a.nk + j;
    store_row<DH>(dk + row * dkvpitch + h * DH, gk, live ? scale : 0.f, hi);
    store_row<DH>(dv + row * dkvpitch + h * DH, gv, live ? 1.f : 0.f, hi);
  }
}

// The query side alone (D to stat[].y).
template <int DH, bool HELD>
__global__ __launch_bounds__(256, HELD ? 2 : 1) void bw_set_attn_bwd_q_kernel(SetAttn a, const __bf16* __restrict__ dob, int d,
                                                                __bf16* __restrict__ dq, int dqpitch, float2* __restrict__ stat) {
  __shared__ __attribute__((aligned(16))) KeyTiles<DH, kAttnChunk> t;
  const int rounds = (a.nq + kAttnRows - 1) / kAttnRows;
  int u, h, rd;
  if (!attn_task(a, rounds, &u, &h, &rd)) return;
  const int lane = threadIdx.x & 63, l32 = lane & 31, hi = lane >> 5;
  const int i0 = rd * kAttnRows + 32 * (threadIdx.x >> 6), i = i0 + l32;
  const size_t row = (size_t)u * a.qrows + (i < a.nq ? i : 0);
  int qd = a.qdesc[row];
  float lse = stat[row * a.heads + h].x;
  RowFrag<DH> q = row_frag<DH>(a.q + row * a.qpitch + h * DH, true, hi), g = row_frag<DH>(dob + row * d + h * DH, true, hi);
  if (i >= a.nq) { qd = -1; lse = __builtin_inff(); }
  const bool live = qd >= 0;
  q.keep(live); g.keep(live);
  const Seen see = query_sees(qd, a.gmask);
  const Span span = span_of(live, see);
  const float scale = rsqrtf((float)DH), c = 1.4426950408889634f * scale;
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  float D = 0.f;
  if constexpr (HELD) {
    stage_keys(t, a, u, h, 0, a.nk);
    __syncthreads();
    if (i0 >= a.nq) return;
    query_side_held(t, a.nk, q, g, span, see, lse, c, D, acc, lane);
  }
  for (int pass = HELD ? 2 : 0; pass < 2; ++pass) {
    for (int c0 = 0; c0 < a.nk; c0 += kAttnChunk) {
      const int n = min(kAttnChunk, a.nk - c0);
      if (pass == 0 || a.nk > kAttnChunk) {       // (a single chunk stays for the second pass)
        if (pass || c0) __syncthreads();
        stage_keys(t, a, u, h, c0, n);
        __syncthreads();
      }
      if (i0 >= a.nq) continue;
      if (pass == 0) query_side_pass<false>(t, n, q, g, span, see, lse, c, D, acc, lane);
      else query_side_pass<true>(t, n, q, g, span, see, lse, c, D, acc, lane);
    }
    if (pass == 0) D = sum_halves(D);
  }
  settle(acc);
  if (i >= a.nq) return;
  store_row<DH>(dq + row * dqpitch + h * DH, acc, live ? scale : 0.f, hi);
  if (hi == 0) stat[row * a.heads + h].y = live ? D : 0.f;
}

// The key side alone, over the user's query rows (D from stat[].y).
template <int DH>
__global__ __launch_bounds__(256) void bw_set_attn_bwd_kv_kernel(SetAttn a, const __bf16* __restrict__ dob, int d,
                                                                 __bf16* __restrict__ dk, __bf16* __restrict__ dv, int dkvpitch,
                                                                 const float2* stat) {
  __shared__ __attribute__((aligned(16))) QueryTiles<DH> t;
  const int rounds = (a.nk + kAttnRows - 1) / kAttnRows;
  int u, h, rd;
  if (!attn_task(a, rounds, &u, &h, &rd)) return;
  const int lane = threadIdx.x & 63, l32 = lane & 31, hi = lane >> 5;
  const int j0 = rd * kAttnRows + 32 * (threadIdx.x >> 6), j = j0 + l32;
  const size_t row = (size_t)u * a.nk + (j < a.nk ? j : 0);
  const int kd = a.kdesc[row];
  RowFrag<DH> kf = row_frag<DH>(a.k + row * a.kvpitch + h * DH, true, hi), vf = row_frag<DH>(a.v + row * a.kvpitch + h * DH, true, hi);
  const int ks = j < a.nk ? key_position(kd) : kNone;
  const bool live = ks != kNone;
  kf.keep(live); vf.keep(live);
  const float scale = rsqrtf((float)DH), c = 1.4426950408889634f * scale;
  f32x16 gk, gv;
#pragma unroll
  for (int r = 0; r < 16; ++r) { gk[r] = 0.f; gv[r] = 0.f; }
  for (int c0 = 0; c0 < a.nq; c0 += kQueryRows) {
    const int n = min(kQueryRows, a.nq - c0);
    if (c0) __syncthreads();
    StagedQueries<DH> s;
    s.request(a, dob, d, stat, u, h, c0, n);
    all_requested();
    s.put(t, a.gmask, n);
    __syncthreads();
    if (j0 < a.nk) key_side(t, n, kf, vf, ks, c, gk, gv, lane);
  }
  settle(gk, gv);
  if (j >= a.nk) return;
  store_row<DH>(dk + row * dkvpitch + h * DH, gk, live ? scale : 0.f, hi);
  store_row<DH>(dv + row * dkvpitch + h * DH, gv, live ? 1.f : 0.f, hi);
}

template <int DH>
static void set_attn_forward(hipStream_t st, const SetAttn& a, __bf16* o, int d, float2* stat) {
  const unsigned uh = (unsigned)((a.B + 7) / 8 * 8 * a.heads);      // (see attn_task)
  bw_set_attn_fwd_kernel<DH><<<uh * ((a.nq + kAttnRows - 1) / kAttnRows), 256, 0, st>>>(a, o, d, stat);
}
template <int DH>
static void set_attn_backward(hipStream_t st, const SetAttn& a, const __bf16* dob, int d, __bf16* dq, int dqpitch, __bf16* dk, __bf16* dv,
                              int dkvpitch, float2* stat) {
  const unsigned uh = (unsigned)((a.B + 7) / 8 * 8 * a.heads);
  if (a.nq <= kQueryRows && a.nk <= kAttnChunk) {
    if (a.nk <= 32 * kHeldTiles) bw_set_attn_bwd_kernel<DH, true><<<uh, 256, 0, st>>>(a, dob, d, dq, dqpitch, dk, dv, dkvpitch, stat);
    else bw_set_attn_bwd_kernel<DH, false><<<uh, 256, 0, st>>>(a, dob, d, dq, dqpitch, dk, dv, dkvpitch, stat);
    return;
  }
  const unsigned gq = uh * ((a.nq + kAttnRows - 1) / kAttnRows), gk = uh * ((a.nk + kAttnRows - 1) / kAttnRows);
  if (a.nk <= 32 * kHeldTiles) bw_set_attn_bwd_q_kernel<DH, true><<<gq, 256, 0, st>>>(a, dob, d, dq, dqpitch, stat);
  else bw_set_attn_bwd_q_kernel<DH, false><<<gq, 256, 0, st>>>(a, dob, d, dq, dqpitch, stat);
  bw_set_attn_bwd_kv_kernel<DH><<<gk, 256, 0, st>>>(a, dob, d, dk, dv, dkvpitch, stat);
}

}  // namespace bw
}  // namespace longer
