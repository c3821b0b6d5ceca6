// The reduced stack's row work in the training step (cross-causal and self-causal layers on B (m + k) query rows, the
// cross layer's keys on B (m + T) rows): everything between two attention launches in one launch, a tile of 32 rows
// per wave, in the registers' transposed layout (bw_block.h).
//
//   forward, between the attention of layer l and that of layer l + 1 (bw_stack_fwd_kernel):
//     [tail of l]   output projection, residual, LayerNorm, FFN, residual -> the layer's output rows
//     [head of l+1] LayerNorm, Q / K / V (the cross layer: Q of the query rows, K / V of the key rows)
//   backward, between the attention backward of layer l and that of layer l - 1 (bw_stack_bwd_kernel):
//     [tail of l]   dQ / dK / dV back through their products and the LayerNorm -> gradient of the layer's input rows
//     [head of l-1] FFN (hidden values formed again) and LayerNorm backward, back through the output projection
//
// What bounds it: a layer's rows are few (27 648 at the headline batch, 4 608 in the small model), so a launch is a
// handful of tiles per compute unit and its time the chain of a tile's products; as 18 launches a layer (LayerNorms,
// products, row masks; 5-34 us each) the row work was most of the small model's step.
// What the attention kernels read and write stays row-major [rows][..]; what the parameter gradients contract goes
// into tile records (bw_block.h); the rows between attention and FFN and their gradient are fp32 tile blocks.
#pragma once
#include "bw_block.h"

namespace longer {
namespace bw {

// Of the last layer's result only the global rows, the first m of a user's m + k, reach the loss: its tail forward and head
// backward run on those alone (m of n: tile row r is row (r / m) n + r % m; their tile blocks and records hold them side by side),
// and no other row has a gradient of Q.  Four layers of 256 users, 8 of 108 rows: 3842 -> 3767 us a step (the tail 32 -> 13, the head 44 -> 18).
struct StackRows { int m, n; };             // m = 0: all rows
__device__ __forceinline__ int stack_row(const StackRows& s, int r) { return s.m ? r / s.m * s.n + r % s.m : r; }

// The cross layer's rows straight from where they lie: row r of a user's `per` is global token r (r < m), else a merged token, the (r - m)-th (key rows) or the
// one that the row's descriptor names (query rows; learnable query tokens: row r - m of the parameter).  (Gathered to fp32 rows by a launch of their
// own: step of the small model 245.5 instead of 242.5 us, of the headline model 3660 instead of 3643.)
struct StackSource { const __bf16 *G, *M, *learned; const int* desc; int per, m, T; };      // per = 0: the rows are in x
template <int D>
__device__ __forceinline__ f32x16 stack_rows(const float* x, const StackSource& s, int row, int ft, bool in, int hi) {
  f32x16 one[1];
  if (!s.per) load_rows<__bf16, 1>(one, x, 1, (long long)row * D + 32 * ft, in, hi);
  else {
    const int u = row / s.per, r = row - u * s.per;
    const __bf16* src = s.G + ((size_t)u * s.m + r) * D;
    bool there = in;
    if (r >= s.m) {
      int t = r - s.m;
      if (s.desc) { t = s.desc[in ? row : 0] - kSeq; there = in && t >= 0; }
      src = s.desc && s.learned ? s.learned + (size_t)(r - s.m) * D : s.M + ((size_t)u * s.T + t) * D;
    }
    load_rows<__bf16, 1>(one, there ? src : s.G, 0, 32 * ft, there, hi);
  }
  return one[0];
}

struct StackFwd {
  const char* wstream;                      // packed weights of this launch
  int rows, f, act;
  StackRows only;                           // which rows (tail)
  float eps;
  const float* x;                           // tail: the layer's input rows; head alone: the rows themselves ([rows][D])
  StackSource from;                         // or where they come from
  // tail (o != NULL)
  const __bf16* o;                          // [rows][D] attention output
  const __bf16 *bo, *ln2_g, *ln2_b, *b1, *b2;
  const int* desc;                          // rows with a negative descriptor are written as zeros
  float* xmid; float* y; __bf16* rec;       // xmid: tile blocks; y: [rows][D]; rec: the layer's records
  // head (out != NULL)
  const __bf16 *ln1_g, *ln1_b, *bias[3];
  int mats;                                 // 1: Q, 2: K and V, 3: Q, K and V
  __bf16* out; int ldo;                     // [rows][ldo], the matrices' results side by side
  __bf16* rec1; int rec1_size, rec1_xh;     // records that take the normalised rows, their size and place there
};

struct StackBwd {
  const char* wstream;
  int rows, f, act;
  StackRows only;                           // head without a tail: which rows
  StackRows head;                           // tail: the rows that the head in front of it ran on
  float eps;
  // tail (dqkv != NULL)
  const __bf16* dqkv; int ldq, mats;        // [rows][ldq]
  const float* x;                           // the layer's input rows [rows][D]
  StackSource from;                         // or where they come from
  const __bf16* ln1_g;
  const float* dxm_in;                      // what reaches them through the residual connection (tile blocks; NULL: nothing)
  __bf16* rec1; int rec1_size, rec1_dqkv;   // records that take dqkv
  float* dx;                                // without a head: the result [rows][D]
  // head (xmid != NULL)
  const float* dy;                          // without a tail: gradient of the layer's output [rows][D]
  const int* desc;                          // rows written as zeros pass no gradient
  const float* xmid;
  const __bf16 *ln2_g, *ln2_b, *b1;
  float* dxm; __bf16* dob; __bf16* rec;     // dxm: tile blocks; dob: [rows][D], gradient of the attention output
};

// activation and derivative in the exact-erf form (gauss_cdf: 1.5e-7).  (Which one, and whether the wave has a chunk at all, is asked once for sixteen
// values: asked for each, every value's chain of twenty instructions stood between two branches of its own, a third of a tile's time: step of the
// small model 268 us instead of 257, with inputs 1111 instead of 1091.)
__device__ __forceinline__ void act_exact(f32x16& v, int act, bool there) {
  if (!there) v = splat16(0.f);
  else if (act == LONGER_ACT_RELU) {
#pragma unroll
    for (int r = 0; r < 16; ++r) v[r] = v[r] > 0.f ? v[r] : 0.f;
  } else {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      float c, e;
      gauss_cdf(v[r], &c, &e);
      v[r] *= c;
    }
  }
}
// v <- the activation, g <- g times its derivative (of no use without a chunk but for g, zeros)
__device__ __forceinline__ void act_exact_both(f32x16& v, f32x16& g, int act, bool there) {
  if (!there) g = splat16(0.f);
  else if (act == LONGER_ACT_RELU) {
#pragma unroll
    for (int r = 0; r < 16; ++r) { g[r] *= v[r] > 0.f ? 1.f : 0.f; v[r] = v[r] > 0.f ? v[r] : 0.f; }
  } else {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      float c, e;
      gauss_cdf(v[r], &c, &e);
      g[r] *= c + v[r] * 0.39894228040143268f * e;
      v[r] *= c;
    }
  }
}

// Sixteen features of a row-major row as an operand group, and back; zeros where it is not there (`row`: any that is; the
// request is unconditional, see load_rows).  A lane reads or writes sixteen bytes: its half's eight features, of which the lane halves
// exchange four (pieces of eight bytes, 768 apart from lane to lane, cost the address unit twice as much).
__device__ __forceinline__ u32x4 exchange_halves(u32x4 v) {
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const uint32_t a = v[e], b = v[e + 2];
    const auto x = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    v[e] = x[0]; v[e + 2] = x[1];
  }
  return v;
}
__device__ __forceinline__ bf16x8 row_request(const __bf16* row, int g, int hi) { return *(const bf16x8*)(row + 16 * g + 8 * hi); }
__device__ __forceinline__ bf16x8 row_group(bf16x8 requested, bool there) {
  u32x4 v = exchange_halves(__builtin_bit_cast(u32x4, requested));
#pragma unroll
  for (int e = 0; e < 4; ++e) { const uint32_t one = v[e]; v[e] = there ? one : 0u; }
  return __builtin_bit_cast(bf16x8, v);
}
__device__ __forceinline__ void row_put(__bf16* row, int g, int hi, bf16x8 v) {
  *(u32x4*)(row + 16 * g + 8 * hi) = exchange_halves(__builtin_bit_cast(u32x4, v));
}
// fp32 tile blocks: [tile][D / 8][64 lanes][4]
// one feature tile of fp32 tile blocks: [tile][D / 8][64 lanes][4]
template <int NT>
__device__ __forceinline__ f32x16 load_part(const float* base, int tile, int t, int lane) {
  f32x16 x;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const f32x4 v = *(const f32x4*)(base + ((size_t)tile * (4 * NT) + 4 * t + q) * 256 + 4 * lane);
#pragma unroll
    for (int e = 0; e < 4; ++e) x[4 * q + e] = v[e];
  }
  return x;
}
template <int NT>
__device__ __forceinline__ void store_part(const f32x16& x, float* base, int tile, int t, int lane) {
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    f32x4 v;
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = x[4 * q + e];
    *(f32x4*)(base + ((size_t)tile * (4 * NT) + 4 * t + q) * 256 + 4 * lane) = v;
  }
}
struct RecordOut {        // one tile's record
  char* p; int lane;
  __device__ __forceinline__ RecordOut(__bf16* base, int tile, int size, int lane_) : p((char*)base + (size_t)tile * size * 1024), lane(lane_) {}
  __device__ __forceinline__ void put(int base, int g, bf16x8 v) const { *(bf16x8*)(p + (size_t)(base + g) * 1024 + tile_lane_offset(lane, g & 1)) = v; }
};

// Four waves share a tile (eight at width 256): feature tile t of the rows, of every product's result and of the LayerNorms
// belongs to wave t; the hidden chunks of the FFN are dealt out the same way (below width 128 the waves without a feature tile
// share in those alone, going through the rest on another's).  Operand groups change hands through LDS (sixteen
// features of 32 rows, 1 KiB), row sums as one pair of numbers per row and wave.  A wave holds few registers and fetches its
// weight fragments from L2 itself, each a product ahead of its use into the registers of the one just used (the compiler
// moves no load across a barrier).  (A tile per wave with the weights streamed through LDS for four tiles, as in the block
// kernel, leaves a wave alone on its SIMD with all of the FFN's activation: 54 / 74 us forward / backward per layer at the
// headline batch, 21 / 23 us in the small model.)  A layer's launch forward / backward, with each product's fragments requested
// when it began and now: 53 / 94 and 49 / 74 us at the headline batch (864 tiles), 34 / 33 and 19 / 23 us on 203 tiles of width 128,
// 13 / 14 and 10 / 11 us in the small model.  Rows of attention outputs and of dQ, dK, dV come and go sixteen bytes a lane, each from memory in one
// wave and through LDS to the others: with every wave fetching all of them in pieces of eight bytes the address unit took 11 600 of a
// backward workgroup's 47 900 cycles for them on 203 tiles of width 128, and a step of that model 1140 us instead of 1111, of the headline batch 3976 instead of
// 3871, of the small model 278 instead of 268.
__host__ __device__ constexpr int stack_waves(int d) { return d >= 256 ? 8 : 4; }
template <int D>
struct StackTile {
  static constexpr int NT = D / 32, NG = D / 16, WV = stack_waves(D), NF = NG > 2 * WV ? NG : 2 * WV;
  typedef __attribute__((address_space(1))) const char gchar;
  typedef __attribute__((address_space(1))) const bf16x8 gfrag;
  const char* w;                                                          // the launch's weights
  int lane, hi, wave, ft;                                                 // ft: the wave's feature tile, own: its alone
  bool own;
  bf16x8 (*ops)[64];                                                      // [group][lane]
  float2 (*sums)[WV][64];                                                 // [use][wave][lane]
  bf16x8 fr[NF];                                                          // weight fragments under way
  __device__ __forceinline__ gchar* at(int seg, int s) const {            // (wave-uniform: a scalar base, the lane's part an offset)
    gchar* q = (gchar*)(w + (size_t)(seg * NG + s) * 1024);
    asm("" : "+s"(q));
    return q;
  }
  __device__ __forceinline__ bf16x8 load(gchar* q, int s) const { return *(gfrag*)(q + ((unsigned)lane * 16u + (unsigned)s * 1024u)); }
  __device__ __forceinline__ void request(gchar* q) {
#pragma unroll
    for (int s = 0; s < NG; ++s) fr[s] = load(q, s);
  }
  // acc += (32 result features) b, then(s): the request that takes the registers of fragment s
  template <typename B, typename F>
  __device__ __forceinline__ void product(f32x16& acc, const B& b, const F& then) {
#pragma unroll
    for (int s = 0; s < NG; ++s) {
      acc = ET<__bf16>::mma(fr[s], b(s), acc);
      then(s);
      __builtin_amdgcn_sched_barrier(0);                                  // (in this order: hoisted loads would need a second set of registers)
    }
    settle(acc);
  }
  // this wave's part of an operand to LDS, then all of it from there
  __device__ __forceinline__ void hand_in(const f32x16& y) const {
    if (!own) return;
#pragma unroll
    for (int g = 0; g < 2; ++g) ops[2 * ft + g][lane] = ET<__bf16>::pack(y, g);
  }
  __device__ __forceinline__ void take(bf16x8 (&b)[NG]) const {
#pragma unroll
    for (int g = 0; g < NG; ++g) b[g] = ops[g][lane];
  }
  // mean and 1 / standard deviation of the rows: every wave's own mean and squared deviations, combined (one barrier)
  __device__ __forceinline__ void stats(int use, const f32x16& x, float eps, float& mean, float& rstd) const {
    float m = 0.f, v = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) m += x[r];
    m = sum_halves(m) * (1.f / 32.f);
#pragma unroll
    for (int r = 0; r < 16; ++r) { const float q = x[r] - m; v = fmaf(q, q, v); }
    sums[use][wave][lane] = make_float2(m, sum_halves(v));
    __syncthreads();
    mean = 0.f;
    float2 p[NT];
#pragma unroll
    for (int k = 0; k < NT; ++k) {
      p[k] = sums[use][k][lane];
      mean = fmaf(p[k].x, 32.f / D, mean);
    }
    float var = 0.f;
#pragma unroll
    for (int k = 0; k < NT; ++k) {
      const float q = p[k].x - mean;
      var += p[k].y + q * q * 32.f;
    }
    rstd = 1.f / sqrtf(var * (1.f / D) + eps);
  }
  // x <- LayerNorm backward of dn at the rows x (this wave's tile)
  __device__ __forceinline__ void norm_back(int use, f32x16& x, f32x16& dn, const float* gain, float mean, float rstd) const {
    float c1 = 0.f, c2 = 0.f;
    dn *= bias_tile(gain, ft, hi);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      x[r] = (x[r] - mean) * rstd;
      c1 += dn[r];
      c2 = fmaf(dn[r], x[r], c2);
    }
    sums[use][wave][lane] = make_float2(sum_halves(c1), sum_halves(c2));
    __syncthreads();
    c1 = 0.f; c2 = 0.f;
#pragma unroll
    for (int k = 0; k < NT; ++k) { const float2 p = sums[use][k][lane]; c1 += p.x; c2 += p.y; }
    c1 *= 1.f / D; c2 *= 1.f / D;
#pragma unroll
    for (int r = 0; r < 16; ++r) x[r] = rstd * (dn[r] - c1 - x[r] * c2);
  }
};

// A launch's parameter vectors, from memory to registers (all requests at once) and on to LDS: up to N of width d and
// the hidden bias (at most 2048 values).
template <int D, int N>
struct StackVectors {
  static constexpr int THR = 64 * stack_waves(D), VD = (D + THR - 1) / THR, VF = 2048 / THR;
  __bf16 d[N][VD], f[VF];
  __device__ __forceinline__ void request(int i, const __bf16* v, int tid) {
#pragma unroll
    for (int k = 0; k < VD; ++k) { const int c = tid + THR * k; d[i][k] = v[c < D ? c : 0]; }
  }
  __device__ __forceinline__ void request_hidden(const __bf16* v, int n, int tid) {
#pragma unroll
    for (int k = 0; k < VF; ++k) { const int c = tid + THR * k; f[k] = v[c < n ? c : 0]; }
  }
  __device__ __forceinline__ void put(int i, float* to, int tid) const {
#pragma unroll
    for (int k = 0; k < VD; ++k) { const int c = tid + THR * k; if (c < D) to[c] = (float)d[i][k]; }
  }
  __device__ __forceinline__ void put_hidden(float* to, int n, int tid) const {
#pragma unroll
    for (int k = 0; k < VF; ++k) { const int c = tid + THR * k; if (c < n) to[c] = (float)f[k]; }
  }
};

__host__ __device__ inline int stack_vec_floats(int d, int f) { return 9 * d + f; }

// What bounds the two kernels: the chain of a tile at small batches; at the headline batch (864 tiles) the exact-erf activation
// beside the products, and 3.3 KB (forward) and 5.5 KB (backward) of memory traffic per row: 37 and 56 us a launch (mean of five) with four and three
// workgroups a compute unit.  MANY: see kStackManyTiles.
template <int D, bool MANY>
__global__ __launch_bounds__(64 * stack_waves(D), D >= 256 ? 1 : MANY ? 4 : 2) void bw_stack_fwd_kernel(const StackFwd p0, const StackFwd p1, int tiles0) {
  using S = StackTile<D>;
  constexpr int NT = S::NT, NG = S::NG, WV = S::WV;
  using E = ET<__bf16>;
  __shared__ bf16x8 ops[NG][64];
  __shared__ bf16x8 hid[2][WV][2][64];             // activated hidden chunks: [parity][wave][group][lane]
  __shared__ float2 sums[2][WV][64];
  extern __shared__ f32x4 vec4[];
  float* vec = (float*)vec4;
  const int tid = threadIdx.x, lane = tid & 63, j = lane & 31, hi = lane >> 5, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  StackFwd p = p0;
  if ((int)blockIdx.x >= tiles0) p = p1;
  const int tile = (int)blockIdx.x - ((int)blockIdx.x >= tiles0 ? tiles0 : 0), row = tile * 32 + j, NC = p.f / 32;
  const bool in = row < p.rows, own = wave < NT;
  const int ft = wave % NT, from = stack_row(p.only, row);
  const int oBo = 0, oG2 = D, oS2 = 2 * D, oB2 = 3 * D, oG1 = 4 * D, oS1 = 5 * D, oB = 6 * D, oB1 = 9 * D;
  S s = {p.wstream, lane, hi, wave, ft, own, ops, sums};
  // everything that is read ahead of the first product is requested at once
  f32x16 x = stack_rows<D>(p.x, p.from, from, ft, in, hi);
  bf16x8 nop[MANY ? 1 : NG], mine[2];                // (mine: this wave's part of the attention output)
  int desc = 0;
  if (p.o) {
#pragma unroll
    for (int q = 0; q < 2; ++q) mine[q] = row_request(p.o + (size_t)(in ? from : 0) * D, 2 * ft + q, hi);
    desc = p.desc[in ? from : 0];
  }
  const int head = p.o ? NT + 2 * NC : 0;          // first segment of the next layer's products
  s.request(s.at(p.o ? ft : head + min(wave, p.mats * NT - 1), 0));
  {
    StackVectors<D, 9> v;
    if (p.o) { v.request(0, p.bo, tid); v.request(1, p.ln2_g, tid); v.request(2, p.ln2_b, tid); v.request(3, p.b2, tid); v.request_hidden(p.b1, p.f, tid); }
    if (p.out) {
      v.request(4, p.ln1_g, tid); v.request(5, p.ln1_b, tid);
#pragma unroll
      for (int m = 0; m < 3; ++m) v.request(6 + m, m < p.mats ? p.bias[m] : p.bias[0], tid);
    }
    if (p.o) { v.put(0, vec + oBo, tid); v.put(1, vec + oG2, tid); v.put(2, vec + oS2, tid); v.put(3, vec + oB2, tid); v.put_hidden(vec + oB1, p.f, tid); }
    if (p.out) {
      v.put(4, vec + oG1, tid); v.put(5, vec + oS1, tid);
#pragma unroll
      for (int m = 0; m < 3; ++m)
        if (m < p.mats) v.put(6 + m, vec + oB + m * D, tid);
    }
  }
  float mean, rstd;
  // rows -> normalised rows (to the records) -> operand of the next products, in every wave
  auto normalise = [&](int use, int og, int os, const RecordOut& rec, int at) {
    s.stats(use, x, p.eps, mean, rstd);            // (its barrier: everybody is done with `ops`, and `vec` is there)
    const f32x16 g = bias_tile(vec + og, ft, hi), b = bias_tile(vec + os, ft, hi);
    f32x16 h, y;
#pragma unroll
    for (int r = 0; r < 16; ++r) { h[r] = (x[r] - mean) * rstd; y[r] = fmaf(h[r], g[r], b[r]); }
    s.hand_in(y);
    if (own) {
#pragma unroll
      for (int q = 0; q < 2; ++q) rec.put(at, 2 * ft + q, E::pack(h, q));
    }
    __syncthreads();
    if constexpr (!MANY) s.take(nop);
  };
  auto operand = [&](int k) -> bf16x8 { return MANY ? ops[k][lane] : nop[MANY ? 0 : k]; };
  if (p.o) {
    const BlockRecord at(D, p.f);
    const RecordOut rec(p.rec, tile, at.size, lane);
    if (own) {
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const bf16x8 v = row_group(mine[q], in);
        ops[2 * ft + q][lane] = v;
        rec.put(at.o, 2 * ft + q, v);
      }
    }
    __syncthreads();                               // `vec`, `ops`
    if constexpr (!MANY) s.take(nop);
    x += bias_tile(vec + oBo, ft, hi);
    typename S::gchar* first = s.at(NT + 2 * min(wave, NC - 1), 0);
    s.product(x, operand, [&](int k) { s.fr[k] = s.load(first, k); });
    if (own) store_part<NT>(x, p.xmid, tile, ft, lane);
    normalise(0, oG2, oS2, rec, at.xh2);
    x += bias_tile(vec + oB2, ft, hi);
    for (int c0 = 0, par = 0; c0 < NC; c0 += WV, par ^= 1) {
      const int c = min(c0 + wave, NC - 1);        // (a wave without a chunk goes through another's and hands in zeros)
      auto second = [&](int k) { s.fr[k] = s.load(s.at(NT + 2 * min(c0 + k / 2, NC - 1) + 1, 2 * ft), k & 1); };
#pragma unroll
      for (int k = NG; k < 2 * WV; ++k) second(k);
      f32x16 v = bias_tile(vec + oB1, c, hi);
      s.product(v, operand, second);
      act_exact(v, p.act, c0 + wave < NC);
#pragma unroll
      for (int g = 0; g < 2; ++g) hid[par][wave][g][lane] = E::pack(v, g);
      const bool end = c0 + WV >= NC;
      typename S::gchar* next = s.at(end ? head + (p.out ? min(wave, p.mats * NT - 1) : -1) : NT + 2 * min(c0 + WV + wave, NC - 1), 0);
      __syncthreads();                             // (the other parity was last read ahead of the barrier before)
#pragma unroll
      for (int k = 0; k < 2 * WV; ++k) {
        x = E::mma(s.fr[k], hid[par][k / 2][k & 1][lane], x);
        if (k < NG) s.fr[k] = s.load(next, k);
        __builtin_amdgcn_sched_barrier(0x486);
      }
    }
    const bool live = in && desc >= 0;
    settle(x);
#pragma unroll
    for (int r = 0; r < 16; ++r) x[r] = live ? x[r] : 0.f;
    const f32x16 one[1] = {x};
    if (in && own) store_rows<__bf16, 1>(one, p.y, 1, (long long)from * D + 32 * ft, true, hi);
  }
  if (p.out) {
    const RecordOut rec(p.rec1, tile, p.rec1_size, lane);
    normalise(1, oG1, oS1, rec, p.rec1_xh);
    for (int k = wave; k < p.mats * NT; k += WV) {      // segment k: matrix k % mats of feature tile k / mats
      const int t = k / p.mats, m = k - t * p.mats;
      f32x16 v = bias_tile(vec + oB + m * D, t, hi);
      typename S::gchar* next = s.at(head + min(k + WV, p.mats * NT - 1), 0);
      s.product(v, operand, [&](int i) { s.fr[i] = s.load(next, i); });
      if (in) {
#pragma unroll
        for (int g = 0; g < 2; ++g) row_put(p.out + (size_t)row * p.ldo + m * D + 32 * t, g, hi, E::pack(v, g));
      }
    }
  }
}

template <int D, bool MANY>
__global__ __launch_bounds__(64 * stack_waves(D), D >= 256 ? 1 : MANY ? 3 : 2) void bw_stack_bwd_kernel(const StackBwd p0, const StackBwd p1, int tiles0) {
  using S = StackTile<D>;
  constexpr int NT = S::NT, NG = S::NG, WV = S::WV;
  using E = ET<__bf16>;
  __shared__ bf16x8 ops[NG][64], ops2[NG][64];
  __shared__ bf16x8 hid[2][WV][2][64];             // gradients of the hidden chunks
  __shared__ float2 sums[4][WV][64];
  extern __shared__ f32x4 vec4[];
  float* vec = (float*)vec4;
  const int tid = threadIdx.x, lane = tid & 63, j = lane & 31, hi = lane >> 5, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  StackBwd p = p0;
  if ((int)blockIdx.x >= tiles0) p = p1;
  const int tile = (int)blockIdx.x - ((int)blockIdx.x >= tiles0 ? tiles0 : 0), row = tile * 32 + j, NC = p.f / 32;
  const bool in = row < p.rows, own = wave < NT;
  const int ft = wave % NT, from = stack_row(p.only, row);
  const int oG1 = 0, oG2 = D, oS2 = 2 * D, oB1 = 3 * D;
  S s = {p.wstream, lane, hi, wave, ft, own, ops, sums};
  f32x16 x, dn = splat16(0.f), xm = splat16(0.f), add = splat16(0.f);
  float mean, rstd;
  x = stack_rows<D>(p.dqkv ? p.x : p.dy, p.from, from, ft, in, hi);
  // fragment k of the products that bring dQ, dK, dV back (matrix m): 32 contracted features k / 2 of this wave's result tile
  auto back = [&](int m, int k) { s.fr[k] = s.load(s.at((k / 2) * p.mats + m, 2 * ft), k & 1); };
  bf16x8 mine[3][2];                               // this wave's part of dQ, dK, dV
  bool asked = in;                                 // the row has a gradient of Q, and one through the residual connection
  const int seg = p.dqkv ? NT * p.mats : 0;        // first segment of the FFN's products
  if (p.dqkv) {
#pragma unroll
    for (int m = 0; m < 3; ++m)
#pragma unroll
      for (int q = 0; q < 2; ++q) mine[m][q] = row_request(p.dqkv + (size_t)(in ? row : 0) * p.ldq + min(m, p.mats - 1) * D, 2 * ft + q, hi);
#pragma unroll
    for (int k = 0; k < NG; ++k) back(0, k);
    if (p.dxm_in && !p.head.m) add = load_part<NT>(p.dxm_in, tile, ft, lane);
    if (p.dxm_in && p.head.m) {
      const int r = row % p.head.n, at = row / p.head.n * p.head.m + r;
      asked = in && r < p.head.m;
      add = load_part<NT>(p.dxm_in, asked ? at / 32 : 0, ft, asked ? 32 * hi + at % 32 : 0);
#pragma unroll
      for (int e = 0; e < 16; ++e) add[e] = asked ? add[e] : 0.f;
    }
  } else {
    s.request(s.at(seg + 3 * min(wave, NC - 1), 0));
  }
  int desc = 0;
  if (p.xmid) { xm = load_part<NT>(p.xmid, tile, ft, lane); desc = p.desc[in ? from : 0]; }
  {
    StackVectors<D, 3> v;
    if (p.dqkv) v.request(0, p.ln1_g, tid);
    if (p.xmid) { v.request(1, p.ln2_g, tid); v.request(2, p.ln2_b, tid); v.request_hidden(p.b1, p.f, tid); }
    if (p.dqkv) v.put(0, vec + oG1, tid);
    if (p.xmid) { v.put(1, vec + oG2, tid); v.put(2, vec + oS2, tid); v.put_hidden(vec + oB1, p.f, tid); }
  }
  if (p.dqkv) {
    const RecordOut rec(p.rec1, tile, p.rec1_size, lane);
    typename S::gchar* first = s.at(seg + (p.xmid ? 3 * min(wave, NC - 1) : -1), 0);
    // (through the buffers of what comes later: free until the barriers behind this)
    static_assert(NG <= 4 * WV, "dV in the hidden chunks' place");
    if (own) {
#pragma unroll
      for (int m = 0; m < 3; ++m)
        if (m < p.mats) {
          bf16x8 (*to)[64] = m == 0 ? ops : m == 1 ? ops2 : &hid[0][0][0];
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            const bf16x8 v = row_group(mine[m][q], m ? in : asked);
            to[2 * ft + q][lane] = v;
            rec.put(p.rec1_dqkv + m * NG, 2 * ft + q, v);
          }
        }
    }
    __syncthreads();                               // (and `vec` is there)
    for (int m = 0; m < p.mats; ++m) {
      const bool end = m + 1 == p.mats;
      bf16x8 (*from)[64] = m == 0 ? ops : m == 1 ? ops2 : &hid[0][0][0];
#pragma unroll
      for (int k = 0; k < NG; ++k) {
        dn = E::mma(s.fr[k], from[k][lane], dn);
        s.fr[k] = s.load(end ? first + k * 1024 : s.at((k / 2) * p.mats + m + 1, 2 * ft) + (k & 1) * 1024, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    settle(dn);
    s.stats(0, x, p.eps, mean, rstd);              // (its barrier: everybody is done with the buffers)
    s.norm_back(1, x, dn, vec + oG1, mean, rstd);
    x += add;
    const f32x16 one[1] = {x};
    if (!p.xmid && in && own) store_rows<__bf16, 1>(one, p.dx, 1, (long long)row * D + 32 * ft, true, hi);
    if (!p.xmid) return;
  }
  const BlockRecord at(D, p.f);
  const RecordOut rec(p.rec, tile, at.size, lane);
  const bool live = in && desc >= 0;
  s.stats(2, xm, p.eps, mean, rstd);               // (its barrier: `vec` is there)
  // (width 256: no registers for a second operand of all features, it is read from LDS)
  constexpr bool HELD = D <= 128 && !MANY;
  bf16x8 dyop[HELD ? NG : 1], nop[MANY ? 1 : NG];
#pragma unroll
  for (int r = 0; r < 16; ++r) x[r] = live ? x[r] : 0.f;
  dn = splat16(0.f);
  {
    const f32x16 g = bias_tile(vec + oG2, ft, hi), b = bias_tile(vec + oS2, ft, hi);
    f32x16 y;
#pragma unroll
    for (int r = 0; r < 16; ++r) y[r] = fmaf((xm[r] - mean) * rstd, g[r], b[r]);
    s.hand_in(y);
    if (own) {
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const bf16x8 v = E::pack(x, q);
        ops2[2 * ft + q][lane] = v;
        rec.put(at.dyb, 2 * ft + q, v);
      }
    }
  }
  __syncthreads();
  if constexpr (!MANY) s.take(nop);
  if (HELD) {
#pragma unroll
    for (int g = 0; g < (HELD ? NG : 1); ++g) dyop[g] = ops2[g][lane];
  }
  auto operand = [&](int k) -> bf16x8 { return MANY ? ops[k][lane] : nop[MANY ? 0 : k]; };
  auto upstream = [&](int k) -> bf16x8 { return HELD ? dyop[HELD ? k : 0] : ops2[k][lane]; };
  for (int c0 = 0, par = 0; c0 < NC; c0 += WV, par ^= 1) {
    const int c = min(c0 + wave, NC - 1);          // (a wave without a chunk goes through another's and hands in zeros)
    const bool there = c0 + wave < NC;
    f32x16 v = bias_tile(vec + oB1, c, hi), g = splat16(0.f);
    typename S::gchar* second = s.at(seg + 3 * c + 1, 0);
    s.product(v, operand, [&](int k) { s.fr[k] = s.load(second, k); });
    auto third = [&](int k) { s.fr[k] = s.load(s.at(seg + 3 * min(c0 + k / 2, NC - 1) + 2, 2 * ft), k & 1); };
#pragma unroll
    for (int k = NG; k < 2 * WV; ++k) third(k);
    s.product(g, upstream, third);
    act_exact_both(v, g, p.act, there);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const bf16x8 h = E::pack(g, q);
      hid[par][wave][q][lane] = h;
      if (there) { rec.put(at.dh + 2 * c, q, h); rec.put(at.a + 2 * c, q, E::pack(v, q)); }
    }
    typename S::gchar* next = s.at(c0 + WV >= NC ? seg + 3 * NC + ft : seg + 3 * min(c0 + WV + wave, NC - 1), 0);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 2 * WV; ++k) {
      dn = E::mma(s.fr[k], hid[par][k / 2][k & 1][lane], dn);
      if (k < NG) s.fr[k] = s.load(next, k);
      __builtin_amdgcn_sched_barrier(0x486);
    }
  }
  settle(dn);
  s.norm_back(3, xm, dn, vec + oG2, mean, rstd);   // (its barrier: everybody has taken `ops`)
  x += xm;
  s.hand_in(x);
  if (own) {
    store_part<NT>(x, p.dxm, tile, ft, lane);
#pragma unroll
    for (int q = 0; q < 2; ++q) rec.put(at.dxmb, 2 * ft + q, E::pack(x, q));
  }
  __syncthreads();
  if constexpr (!MANY) s.take(nop);
  f32x16 v = splat16(0.f);
  s.product(v, operand, [](int) {});
  if (in && own) {
#pragma unroll
    for (int g = 0; g < 2; ++g) row_put(p.dob + (size_t)from * D + 32 * ft, g, hi, E::pack(v, g));
  }
}

void bw_stack_fwd_32(const StackFwd& p, const StackFwd& k, hipStream_t st);
void bw_stack_bwd_32(const StackBwd& p, const StackBwd& k, hipStream_t st);
void bw_stack_fwd_64(const StackFwd& p, const StackFwd& k, hipStream_t st);
void bw_stack_bwd_64(const StackBwd& p, const StackBwd& k, hipStream_t st);
void bw_stack_fwd_128(const StackFwd& p, const StackFwd& k, hipStream_t st);
void bw_stack_bwd_128(const StackBwd& p, const StackBwd& k, hipStream_t st);
void bw_stack_fwd_256(const StackFwd& p, const StackFwd& k, hipStream_t st);
void bw_stack_bwd_256(const StackBwd& p, const StackBwd& k, hipStream_t st);
// Beyond one round of two workgroups a compute unit the operands of the products stay in LDS (MANY) instead of a wave's registers: four
// workgroups fit forward (118 registers instead of 149) and three backward (160 instead of 224).  A training step of width 128 and 108 rows a user, 257, 439,
// 513, 642, 864, 1728 tiles, without / with it 660 / 662, 860 / 860, 1001 / 961, 1213 / 1185, 1509 / 1500, 2553 / 2524 us; width 64 and 104 rows, 260, 520, 650,
// 1664 tiles 233 / 236, 320 / 301, 344 / 325, 658 / 636.
constexpr int kStackManyTiles = 512;
// k: the cross layer's key rows, beside its query rows in one launch (no rows: none).  Two launches of their own in either direction
// were each the chain of a tile on a part of the chip.
template <int D>
inline void bw_stack_fwd_d(const StackFwd& p, const StackFwd& k, hipStream_t st) {
  const int t0 = (p.rows + 31) / 32, t1 = (k.rows + 31) / 32;
  const dim3 grid(t0 + t1), block(64 * stack_waves(D));
  const size_t lds = (size_t)stack_vec_floats(D, p.f) * 4;
  if constexpr (D == 128 || D == 64) { if (t0 + t1 > kStackManyTiles) { bw_stack_fwd_kernel<D, true><<<grid, block, lds, st>>>(p, k, t0); return; } }
  bw_stack_fwd_kernel<D, false><<<grid, block, lds, st>>>(p, k, t0);
}
template <int D>
inline void bw_stack_bwd_d(const StackBwd& p, const StackBwd& k, hipStream_t st) {
  const int t0 = (p.rows + 31) / 32, t1 = (k.rows + 31) / 32;
  const dim3 grid(t0 + t1), block(64 * stack_waves(D));
  const size_t lds = (size_t)stack_vec_floats(D, p.f) * 4;
  if constexpr (D == 128 || D == 64) { if (t0 + t1 > kStackManyTiles) { bw_stack_bwd_kernel<D, true><<<grid, block, lds, st>>>(p, k, t0); return; } }
  bw_stack_bwd_kernel<D, false><<<grid, block, lds, st>>>(p, k, t0);
}

}  // namespace bw
}  // namespace longer
