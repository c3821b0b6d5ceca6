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

struct StackFwd {
  const char* wstream; int segs;            // packed weights of this launch
  int rows, f, act;
  float eps;
  const float* x;                           // tail: the layer's input rows; head alone: the rows themselves ([rows][D])
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
  const char* wstream; int segs;
  int rows, f, act;
  float eps;
  // tail (dqkv != NULL)
  const __bf16* dqkv; int ldq, mats;        // [rows][ldq]
  const float* x;                           // the layer's input rows [rows][D]
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

// activation and derivative in the exact-erf form (gauss_cdf: 1.5e-7)
__device__ __forceinline__ float act_exact(float v, int act) {
  if (act == LONGER_ACT_RELU) return v > 0.f ? v : 0.f;
  float c, e;
  gauss_cdf(v, &c, &e);
  return v * c;
}
__device__ __forceinline__ void act_exact_both(float v, int act, float* a, float* da) {
  if (act == LONGER_ACT_RELU) { *a = v > 0.f ? v : 0.f; *da = v > 0.f ? 1.f : 0.f; return; }
  float c, e;
  gauss_cdf(v, &c, &e);
  *a = v * c;
  *da = c + v * 0.39894228040143268f * e;
}

// sixteen features of a row-major row as an operand group, and back
__device__ __forceinline__ bf16x8 row_group(const __bf16* row, int g, int hi, bool there) {
  bf16x4 a = {}, b = {};
  if (there) { a = *(const bf16x4*)(row + 16 * g + 4 * hi); b = *(const bf16x4*)(row + 16 * g + 8 + 4 * hi); }
  return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
}
__device__ __forceinline__ void row_put(__bf16* row, int g, int hi, bf16x8 v) {
  *(bf16x4*)(row + 16 * g + 4 * hi) = __builtin_shufflevector(v, v, 0, 1, 2, 3);
  *(bf16x4*)(row + 16 * g + 8 + 4 * hi) = __builtin_shufflevector(v, v, 4, 5, 6, 7);
}
// fp32 tile blocks: [tile][D / 8][64 lanes][4]
template <int NT>
__device__ __forceinline__ void load_tile(f32x16 (&x)[NT], const float* base, int tile, int lane) {
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const f32x4 v = *(const f32x4*)(base + ((size_t)tile * (4 * NT) + 4 * t + q) * 256 + 4 * lane);
#pragma unroll
      for (int e = 0; e < 4; ++e) x[t][4 * q + e] = v[e];
    }
}
template <int NT>
__device__ __forceinline__ void store_tile(const f32x16 (&x)[NT], float* base, int tile, int lane) {
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      f32x4 v;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = x[t][4 * q + e];
      *(f32x4*)(base + ((size_t)tile * (4 * NT) + 4 * t + q) * 256 + 4 * lane) = v;
    }
}
struct RecordOut {        // one tile's record
  char* p; int lane;
  __device__ __forceinline__ RecordOut(__bf16* base, int tile, int size, int lane_) : p((char*)base + (size_t)tile * size * 1024), lane(lane_) {}
  __device__ __forceinline__ void put(int base, int g, bf16x8 v) const { *(bf16x8*)(p + (size_t)(base + g) * 1024 + tile_lane_offset(lane, g & 1)) = v; }
};
template <int NT>
__device__ __forceinline__ void normalise_rows(const f32x16 (&x)[NT], float mean, float rstd, const float* gain, const float* shift, int hi,
                                               bf16x8 (&op)[2 * NT], const RecordOut* rec, int at) {
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const f32x16 g = bias_tile(gain, t, hi), b = bias_tile(shift, t, hi);
    f32x16 h, y;
#pragma unroll
    for (int r = 0; r < 16; ++r) { h[r] = (x[t][r] - mean) * rstd; y[r] = fmaf(h[r], g[r], b[r]); }
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      if (rec) rec->put(at, 2 * t + q, ET<__bf16>::pack(h, q));
      op[2 * t + q] = ET<__bf16>::pack(y, q);
    }
  }
}

template <int D, int NW>
struct StackStream {
  static constexpr int NT = D / 32, NG = D / 16, SEGV = NG * 64, PSEG = D >= 256 ? 1 : D >= 128 ? 2 : 4;
  typedef WStream<SEGV, PSEG, 3, false, 64 * NW> Stream;
  Stream ws;
  // With a wave per SIMD every product would wait out the LDS latency of its own fragment (about four times its length), and
  // scheduling hints are not followed: six reads are kept in flight by hand, the order pinned.
  template <typename F>
  __device__ __forceinline__ void fragments(F&& use) {
    constexpr int AH = NG < 6 ? NG : 6;
    bf16x8 w[AH];
#pragma unroll
    for (int i = 0; i < AH; ++i) w[i] = ws.template frag<bf16x8>(i);
#pragma unroll
    for (int i = 0; i < NG; ++i) {
      __builtin_amdgcn_sched_barrier(0);
      use(i, w[i % AH]);
      __builtin_amdgcn_sched_barrier(0);
      if (i + AH < NG) w[i % AH] = ws.template frag<bf16x8>(i + AH);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  __device__ __forceinline__ void product(f32x16& acc, const bf16x8 (&b)[NG]) {
    fragments([&](int s, const bf16x8 w) { acc = ET<__bf16>::mma(w, b[s], acc); });
    ws.advance();
    settle(acc);
  }
  __device__ __forceinline__ void spread(f32x16 (&acc)[NT], const bf16x8 (&b)[2]) {
    fragments([&](int i, const bf16x8 w) { acc[i / 2] = ET<__bf16>::mma(w, b[i % 2], acc[i / 2]); });
    ws.advance();
  }
};

__host__ __device__ inline int stack_vec_floats(int d, int f) { return 9 * d + f; }

template <int D, int NW>
__global__ __launch_bounds__(64 * NW, D >= 256 ? 1 : 2) void bw_stack_fwd_kernel(const StackFwd p) {
  using S = StackStream<D, NW>;
  constexpr int NT = S::NT, NG = S::NG;
  using E = ET<__bf16>;
  __shared__ uint4 ring[3 * S::PSEG * S::SEGV];
  extern __shared__ f32x4 vec4[];
  float* vec = (float*)vec4;
  const int tid = threadIdx.x, lane = tid & 63, j = lane & 31, hi = lane >> 5;
  const int tile = blockIdx.x * NW + __builtin_amdgcn_readfirstlane(tid >> 6), row = tile * 32 + j;
  const bool in = row < p.rows;
  const int oBo = 0, oG2 = D, oS2 = 2 * D, oB2 = 3 * D, oG1 = 4 * D, oS1 = 5 * D, oB = 6 * D, oB1 = 9 * D;
  for (int i = tid; i < D; i += 64 * NW) {
    if (p.o) { vec[oBo + i] = (float)p.bo[i]; vec[oG2 + i] = (float)p.ln2_g[i]; vec[oS2 + i] = (float)p.ln2_b[i]; vec[oB2 + i] = (float)p.b2[i]; }
    if (p.out) {
      vec[oG1 + i] = (float)p.ln1_g[i]; vec[oS1 + i] = (float)p.ln1_b[i];
      for (int m = 0; m < p.mats; ++m) vec[oB + m * D + i] = (float)p.bias[m][i];
    }
  }
  if (p.o) for (int i = tid; i < p.f; i += 64 * NW) vec[oB1 + i] = (float)p.b1[i];
  f32x16 x[NT];
  load_rows<__bf16, NT>(x, p.x, 1, (long long)row * D, in, hi);
  S s;
  s.ws.init(ring, p.wstream, p.segs);
  bf16x8 nop[NG];
  float mean, rstd;
  if (p.o) {
    const RecordOut rec(p.rec, tile, BlockRecord(D, p.f).size, lane);
    const BlockRecord at(D, p.f);
    {
      bf16x8 oop[NG];
#pragma unroll
      for (int g = 0; g < NG; ++g) { oop[g] = row_group(p.o + (size_t)row * D, g, hi, in); rec.put(at.o, g, oop[g]); }
#pragma unroll
      for (int t = 0; t < NT; ++t) { x[t] += bias_tile(vec + oBo, t, hi); s.product(x[t], oop); }
    }
    store_tile<NT>(x, p.xmid, tile, lane);
    row_stats<NT>(x, p.eps, mean, rstd);
    normalise_rows<NT>(x, mean, rstd, vec + oG2, vec + oS2, hi, nop, &rec, at.xh2);
#pragma unroll
    for (int t = 0; t < NT; ++t) x[t] += bias_tile(vec + oB2, t, hi);
    for (int c = 0; c < p.f / 32; ++c) {
      f32x16 v = bias_tile(vec + oB1, c, hi);
      s.product(v, nop);
#pragma unroll
      for (int r = 0; r < 16; ++r) v[r] = act_exact(v[r], p.act);
      const bf16x8 aop[2] = {E::pack(v, 0), E::pack(v, 1)};
      s.spread(x, aop);
    }
    const bool live = in && p.desc[in ? row : 0] >= 0;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      settle(x[t]);
#pragma unroll
      for (int r = 0; r < 16; ++r) x[t][r] = live ? x[t][r] : 0.f;
    }
    if (in) store_rows<__bf16, NT>(x, p.y, 1, (long long)row * D, true, hi);
  }
  if (p.out) {
    const RecordOut rec(p.rec1, tile, p.rec1_size, lane);
    row_stats<NT>(x, p.eps, mean, rstd);
    normalise_rows<NT>(x, mean, rstd, vec + oG1, vec + oS1, hi, nop, &rec, p.rec1_xh);
    for (int ft = 0; ft < NT; ++ft)
      for (int m = 0; m < p.mats; ++m) {
        f32x16 v = bias_tile(vec + oB + m * D, ft, hi);
        s.product(v, nop);
        if (in) {
#pragma unroll
          for (int g = 0; g < 2; ++g) row_put(p.out + (size_t)row * p.ldo + m * D + 32 * ft, g, hi, E::pack(v, g));
        }
      }
  }
}

template <int D, int NW>
__global__ __launch_bounds__(64 * NW, D >= 256 ? 1 : 2) void bw_stack_bwd_kernel(const StackBwd p) {
  using S = StackStream<D, NW>;
  constexpr int NT = S::NT, NG = S::NG;
  using E = ET<__bf16>;
  __shared__ uint4 ring[3 * S::PSEG * S::SEGV];
  extern __shared__ f32x4 vec4[];
  float* vec = (float*)vec4;
  const int tid = threadIdx.x, lane = tid & 63, j = lane & 31, hi = lane >> 5;
  const int tile = blockIdx.x * NW + __builtin_amdgcn_readfirstlane(tid >> 6), row = tile * 32 + j;
  const bool in = row < p.rows;
  const int oG1 = 0, oG2 = D, oS2 = 2 * D, oB1 = 3 * D;
  for (int i = tid; i < D; i += 64 * NW) {
    if (p.dqkv) vec[oG1 + i] = (float)p.ln1_g[i];
    if (p.xmid) { vec[oG2 + i] = (float)p.ln2_g[i]; vec[oS2 + i] = (float)p.ln2_b[i]; }
  }
  if (p.xmid) for (int i = tid; i < p.f; i += 64 * NW) vec[oB1 + i] = (float)p.b1[i];
  S s;
  s.ws.init(ring, p.wstream, p.segs);
  f32x16 x[NT], dn[NT];
  float mean, rstd;
  if (p.dqkv) {
    const RecordOut rec(p.rec1, tile, p.rec1_size, lane);
#pragma unroll
    for (int t = 0; t < NT; ++t) dn[t] = splat16(0.f);
    for (int ft = 0; ft < NT; ++ft)
      for (int m = 0; m < p.mats; ++m) {
        bf16x8 op[2];
#pragma unroll
        for (int g = 0; g < 2; ++g) {
          op[g] = row_group(p.dqkv + (size_t)row * p.ldq + m * D + 32 * ft, g, hi, in);
          rec.put(p.rec1_dqkv + m * NG + 2 * ft, g, op[g]);
        }
        s.spread(dn, op);
      }
#pragma unroll
    for (int t = 0; t < NT; ++t) settle(dn[t]);
    load_rows<__bf16, NT>(x, p.x, 1, (long long)row * D, in, hi);
    row_stats<NT>(x, p.eps, mean, rstd);
    norm_backward<NT>(x, dn, vec + oG1, mean, rstd, hi);
    if (p.dxm_in) {
      load_tile<NT>(dn, p.dxm_in, tile, lane);
#pragma unroll
      for (int t = 0; t < NT; ++t) x[t] += dn[t];
    }
    if (!p.xmid) {
      if (in) store_rows<__bf16, NT>(x, p.dx, 1, (long long)row * D, true, hi);
      return;
    }
  } else {
    load_rows<__bf16, NT>(x, p.dy, 1, (long long)row * D, in, hi);
  }
  const BlockRecord at(D, p.f);
  const RecordOut rec(p.rec, tile, at.size, lane);
  const bool live = in && p.desc[in ? row : 0] >= 0;
  bf16x8 dyop[NG], nop[NG];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
#pragma unroll
    for (int r = 0; r < 16; ++r) x[t][r] = live ? x[t][r] : 0.f;
#pragma unroll
    for (int g = 0; g < 2; ++g) { dyop[2 * t + g] = E::pack(x[t], g); rec.put(at.dyb, 2 * t + g, dyop[2 * t + g]); }
  }
  load_tile<NT>(dn, p.xmid, tile, lane);
  row_stats<NT>(dn, p.eps, mean, rstd);
  normalise_rows<NT>(dn, mean, rstd, vec + oG2, vec + oS2, hi, nop, nullptr, 0);
#pragma unroll
  for (int t = 0; t < NT; ++t) dn[t] = splat16(0.f);
  for (int c = 0; c < p.f / 32; ++c) {
    f32x16 v = bias_tile(vec + oB1, c, hi), g = splat16(0.f);
    s.product(v, nop);
    s.product(g, dyop);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      float a, da;
      act_exact_both(v[r], p.act, &a, &da);
      v[r] = a;
      g[r] *= da;
    }
    bf16x8 hop[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      hop[q] = E::pack(g, q);
      rec.put(at.dh + 2 * c, q, hop[q]);
      rec.put(at.a + 2 * c, q, E::pack(v, q));
    }
    s.spread(dn, hop);
  }
#pragma unroll
  for (int t = 0; t < NT; ++t) settle(dn[t]);
  {
    f32x16 xm[NT];
    load_tile<NT>(xm, p.xmid, tile, lane);
    norm_backward<NT>(xm, dn, vec + oG2, mean, rstd, hi);
#pragma unroll
    for (int t = 0; t < NT; ++t) x[t] += xm[t];
  }
  store_tile<NT>(x, p.dxm, tile, lane);
#pragma unroll
  for (int g = 0; g < NG; ++g) { nop[g] = E::pack(x[g / 2], g % 2); rec.put(at.dxmb, g, nop[g]); }
  for (int ft = 0; ft < NT; ++ft) {
    f32x16 v = splat16(0.f);
    s.product(v, nop);
    if (in) {
#pragma unroll
      for (int g = 0; g < 2; ++g) row_put(p.dob + (size_t)row * D + 32 * ft, g, hi, E::pack(v, g));
    }
  }
}

constexpr int kStackWaves = 4;              // most waves of a workgroup: records and tile blocks are in whole workgroups of it
void bw_stack_fwd_32(const StackFwd& p, hipStream_t st);
void bw_stack_bwd_32(const StackBwd& p, hipStream_t st);
void bw_stack_fwd_64(const StackFwd& p, hipStream_t st);
void bw_stack_bwd_64(const StackBwd& p, hipStream_t st);
void bw_stack_fwd_128(const StackFwd& p, hipStream_t st);
void bw_stack_bwd_128(const StackBwd& p, hipStream_t st);
void bw_stack_fwd_256(const StackFwd& p, hipStream_t st);
void bw_stack_bwd_256(const StackBwd& p, hipStream_t st);
// Four tiles per workgroup share a weight stream; with fewer tiles than compute units every tile gets one to itself.
template <int D>
inline void bw_stack_fwd_d(const StackFwd& p, hipStream_t st) {
  const int tiles = (p.rows + 31) / 32;
  const size_t lds = (size_t)stack_vec_floats(D, p.f) * 4;
  if (tiles > kComputeUnits) bw_stack_fwd_kernel<D, kStackWaves><<<(tiles + kStackWaves - 1) / kStackWaves, 64 * kStackWaves, lds, st>>>(p);
  else bw_stack_fwd_kernel<D, 1><<<tiles, 64, lds, st>>>(p);
}
template <int D>
inline void bw_stack_bwd_d(const StackBwd& p, hipStream_t st) {
  const int tiles = (p.rows + 31) / 32;
  const size_t lds = (size_t)stack_vec_floats(D, p.f) * 4;
  if (tiles > kComputeUnits) bw_stack_bwd_kernel<D, kStackWaves><<<(tiles + kStackWaves - 1) / kStackWaves, 64 * kStackWaves, lds, st>>>(p);
  else bw_stack_bwd_kernel<D, 1><<<tiles, 64, lds, st>>>(p);
}

}  // namespace bw
}  // namespace longer
