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
  const char* wstream;                      // packed weights of this launch
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
  const char* wstream;
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

// Four waves share a tile: feature tile t of the rows, of every product's result and of the LayerNorms belongs to wave
// t % 4; the hidden chunks of the FFN are dealt out the same way.  Operand groups change hands through LDS (sixteen
// features of 32 rows, 1 KiB), row sums as one pair of numbers per row and wave.  A wave holds few registers and fetches its
// weight fragments from L2 itself.  (A tile per wave with the weights streamed through LDS for four tiles, as in the block
// kernel, leaves a wave alone on its SIMD with all of the FFN's activation: 54 / 74 us forward / backward per layer at the
// headline batch, 21 / 23 us in the small model.)
constexpr int kStackWaves = 4;
template <int D>
struct StackTile {
  static constexpr int NT = D / 32, NG = D / 16, OT = (NT + 3) / 4;      // OT: most feature tiles of a wave
  const char* w;                                                          // the launch's weights
  int lane, hi, wave;
  bf16x8 (*ops)[64];                                                      // [group][lane]
  float2 (*sums)[64];                                                     // [wave][lane]
  __device__ __forceinline__ bool owns(int i) const { return wave + 4 * i < NT; }
  __device__ __forceinline__ bf16x8 frag(int seg, int s) const { return *(const bf16x8*)(w + ((size_t)(seg * NG + s) * 64 + lane) * 16); }
  // acc += (segment seg: 32 result features) b
  __device__ __forceinline__ void product(f32x16& acc, int seg, const bf16x8 (&b)[NG]) const {
    bf16x8 f[NG];
#pragma unroll
    for (int s = 0; s < NG; ++s) f[s] = frag(seg, s);
#pragma unroll
    for (int s = 0; s < NG; ++s) acc = ET<__bf16>::mma(f[s], b[s], acc);
  }
  // this wave's part of an operand to LDS, then all of it from there
  __device__ __forceinline__ void hand_in(int t, const f32x16& y) const {
#pragma unroll
    for (int g = 0; g < 2; ++g) ops[2 * t + g][lane] = ET<__bf16>::pack(y, g);
  }
  __device__ __forceinline__ void take(bf16x8 (&b)[NG]) const {
#pragma unroll
    for (int g = 0; g < NG; ++g) b[g] = ops[g][lane];
  }
  // mean and 1 / standard deviation of the rows: every wave's own mean and squared deviations, combined (one barrier)
  __device__ __forceinline__ void stats(const f32x16 (&x)[OT], float eps, float& mean, float& rstd) const {
    float n = 0.f, m = 0.f, v = 0.f;
#pragma unroll
    for (int i = 0; i < OT; ++i) {
      if (!owns(i)) continue;
#pragma unroll
      for (int r = 0; r < 16; ++r) m += x[i][r];
      n += 32.f;
    }
    m = sum_halves(m) / fmaxf(n, 1.f);
#pragma unroll
    for (int i = 0; i < OT; ++i) {
      if (!owns(i)) continue;
#pragma unroll
      for (int r = 0; r < 16; ++r) { const float q = x[i][r] - m; v = fmaf(q, q, v); }
    }
    __syncthreads();                               // (whatever was in `sums` has been read)
    sums[wave][lane] = make_float2(m, sum_halves(v));
    __syncthreads();
    mean = 0.f;
    float2 p[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      p[k] = sums[k][lane];
      mean = fmaf(p[k].x, (float)(32 * ((NT - k + 3) / 4)) * (1.f / D), mean);
    }
    float var = 0.f;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const float q = p[k].x - mean;
      var += p[k].y + q * q * (float)(32 * ((NT - k + 3) / 4));
    }
    rstd = 1.f / sqrtf(var * (1.f / D) + eps);
  }
  // x <- LayerNorm backward of dn at the rows x (this wave's tiles)
  __device__ __forceinline__ void norm_back(f32x16 (&x)[OT], f32x16 (&dn)[OT], const float* gain, float mean, float rstd) const {
    float c1 = 0.f, c2 = 0.f;
#pragma unroll
    for (int i = 0; i < OT; ++i) {
      if (!owns(i)) continue;
      dn[i] *= bias_tile(gain, wave + 4 * i, hi);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        x[i][r] = (x[i][r] - mean) * rstd;
        c1 += dn[i][r];
        c2 = fmaf(dn[i][r], x[i][r], c2);
      }
    }
    __syncthreads();
    sums[wave][lane] = make_float2(sum_halves(c1), sum_halves(c2));
    __syncthreads();
    c1 = 0.f; c2 = 0.f;
#pragma unroll
    for (int k = 0; k < 4; ++k) { const float2 p = sums[k][lane]; c1 += p.x; c2 += p.y; }
    c1 *= 1.f / D; c2 *= 1.f / D;
#pragma unroll
    for (int i = 0; i < OT; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) x[i][r] = rstd * (dn[i][r] - c1 - x[i][r] * c2);
  }
};

__host__ __device__ inline int stack_vec_floats(int d, int f) { return 9 * d + f; }

template <int D>
__global__ __launch_bounds__(64 * kStackWaves, 2) void bw_stack_fwd_kernel(const StackFwd p) {
  using S = StackTile<D>;
  constexpr int NT = S::NT, NG = S::NG, OT = S::OT;
  using E = ET<__bf16>;
  __shared__ bf16x8 ops[NG][64];
  __shared__ bf16x8 hid[2][4][2][64];              // activated hidden chunks: [parity][wave][group][lane]
  __shared__ float2 sums[4][64];
  extern __shared__ f32x4 vec4[];
  float* vec = (float*)vec4;
  const int tid = threadIdx.x, lane = tid & 63, j = lane & 31, hi = lane >> 5, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int tile = blockIdx.x, row = tile * 32 + j, NC = p.f / 32;
  const bool in = row < p.rows;
  const int oBo = 0, oG2 = D, oS2 = 2 * D, oB2 = 3 * D, oG1 = 4 * D, oS1 = 5 * D, oB = 6 * D, oB1 = 9 * D;
  for (int i = tid; i < D; i += 64 * kStackWaves) {
    if (p.o) { vec[oBo + i] = (float)p.bo[i]; vec[oG2 + i] = (float)p.ln2_g[i]; vec[oS2 + i] = (float)p.ln2_b[i]; vec[oB2 + i] = (float)p.b2[i]; }
    if (p.out) {
      vec[oG1 + i] = (float)p.ln1_g[i]; vec[oS1 + i] = (float)p.ln1_b[i];
      for (int m = 0; m < p.mats; ++m) vec[oB + m * D + i] = (float)p.bias[m][i];
    }
  }
  if (p.o) for (int i = tid; i < p.f; i += 64 * kStackWaves) vec[oB1 + i] = (float)p.b1[i];
  const S s = {p.wstream, lane, hi, wave, ops, sums};
  f32x16 x[OT];
#pragma unroll
  for (int i = 0; i < OT; ++i) {
    f32x16 one[1];
    load_rows<__bf16, 1>(one, p.x, 1, (long long)row * D + 32 * (wave + 4 * i), in && s.owns(i), hi);
    x[i] = one[0];
  }
  bf16x8 nop[NG];
  float mean, rstd;
  int seg = 0;
  // rows -> normalised rows (to the records) -> operand of the next products, in every wave
  auto normalise = [&](int og, int os, const RecordOut& rec, int at) {
    s.stats(x, p.eps, mean, rstd);                 // (its barriers: everybody is done with `ops`, and `vec` is there)
#pragma unroll
    for (int i = 0; i < OT; ++i) {
      if (!s.owns(i)) continue;
      const int t = wave + 4 * i;
      const f32x16 g = bias_tile(vec + og, t, hi), b = bias_tile(vec + os, t, hi);
      f32x16 h, y;
#pragma unroll
      for (int r = 0; r < 16; ++r) { h[r] = (x[i][r] - mean) * rstd; y[r] = fmaf(h[r], g[r], b[r]); }
#pragma unroll
      for (int q = 0; q < 2; ++q) rec.put(at, 2 * t + q, E::pack(h, q));
      s.hand_in(t, y);
    }
    __syncthreads();
    s.take(nop);
  };
  if (p.o) {
    const BlockRecord at(D, p.f);
    const RecordOut rec(p.rec, tile, at.size, lane);
    bf16x8 oop[NG];
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      oop[g] = row_group(p.o + (size_t)row * D, g, hi, in);
      if ((g >> 1) % 4 == wave) rec.put(at.o, g, oop[g]);
    }
    __syncthreads();                               // `vec`
#pragma unroll
    for (int i = 0; i < OT; ++i) {
      if (!s.owns(i)) continue;
      const int t = wave + 4 * i;
      x[i] += bias_tile(vec + oBo, t, hi);
      s.product(x[i], t, oop);
      settle(x[i]);
      store_part<NT>(x[i], p.xmid, tile, t, lane);
    }
    seg = NT;
    normalise(oG2, oS2, rec, at.xh2);
#pragma unroll
    for (int i = 0; i < OT; ++i)
      if (s.owns(i)) x[i] += bias_tile(vec + oB2, wave + 4 * i, hi);
    for (int c0 = 0, par = 0; c0 < NC; c0 += 4, par ^= 1) {
      const int c = c0 + wave;
      if (c < NC) {
        f32x16 v = bias_tile(vec + oB1, c, hi);
        s.product(v, seg + 2 * c, nop);
        settle(v);
#pragma unroll
        for (int r = 0; r < 16; ++r) v[r] = act_exact(v[r], p.act);
#pragma unroll
        for (int g = 0; g < 2; ++g) hid[par][wave][g][lane] = E::pack(v, g);
      }
      __syncthreads();                             // (the other parity was last read ahead of the barrier before)
#pragma unroll
      for (int i = 0; i < OT; ++i) {
        if (!s.owns(i)) continue;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          if (c0 + k >= NC) break;
#pragma unroll
          for (int g = 0; g < 2; ++g) x[i] = E::mma(s.frag(seg + 2 * (c0 + k) + 1, 2 * (wave + 4 * i) + g), hid[par][k][g][lane], x[i]);
        }
      }
    }
    seg += 2 * NC;
    const bool live = in && p.desc[in ? row : 0] >= 0;
#pragma unroll
    for (int i = 0; i < OT; ++i) {
      settle(x[i]);
#pragma unroll
      for (int r = 0; r < 16; ++r) x[i][r] = live ? x[i][r] : 0.f;
      const f32x16 one[1] = {x[i]};
      if (in && s.owns(i)) store_rows<__bf16, 1>(one, p.y, 1, (long long)row * D + 32 * (wave + 4 * i), true, hi);
    }
  }
  if (p.out) {
    const RecordOut rec(p.rec1, tile, p.rec1_size, lane);
    normalise(oG1, oS1, rec, p.rec1_xh);
    for (int k = wave; k < p.mats * NT; k += kStackWaves) {      // segment k: matrix k % mats of feature tile k / mats
      const int ft = k / p.mats, m = k - ft * p.mats;
      f32x16 v = bias_tile(vec + oB + m * D, ft, hi);
      s.product(v, seg + k, nop);
      settle(v);
      if (in) {
#pragma unroll
        for (int g = 0; g < 2; ++g) row_put(p.out + (size_t)row * p.ldo + m * D + 32 * ft, g, hi, E::pack(v, g));
      }
    }
  }
}

template <int D>
__global__ __launch_bounds__(64 * kStackWaves, 2) void bw_stack_bwd_kernel(const StackBwd p) {
  using S = StackTile<D>;
  constexpr int NT = S::NT, NG = S::NG, OT = S::OT;
  using E = ET<__bf16>;
  __shared__ bf16x8 ops[NG][64], ops2[NG][64];
  __shared__ bf16x8 hid[2][4][2][64];              // gradients of the hidden chunks
  __shared__ float2 sums[4][64];
  extern __shared__ f32x4 vec4[];
  float* vec = (float*)vec4;
  const int tid = threadIdx.x, lane = tid & 63, j = lane & 31, hi = lane >> 5, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int tile = blockIdx.x, row = tile * 32 + j, NC = p.f / 32;
  const bool in = row < p.rows;
  const int oG1 = 0, oG2 = D, oS2 = 2 * D, oB1 = 3 * D;
  for (int i = tid; i < D; i += 64 * kStackWaves) {
    if (p.dqkv) vec[oG1 + i] = (float)p.ln1_g[i];
    if (p.xmid) { vec[oG2 + i] = (float)p.ln2_g[i]; vec[oS2 + i] = (float)p.ln2_b[i]; }
  }
  if (p.xmid) for (int i = tid; i < p.f; i += 64 * kStackWaves) vec[oB1 + i] = (float)p.b1[i];
  const S s = {p.wstream, lane, hi, wave, ops, sums};
  f32x16 x[OT], dn[OT];
  float mean, rstd;
  int seg = 0;
  const float* src = p.dqkv ? p.x : p.dy;
#pragma unroll
  for (int i = 0; i < OT; ++i) {
    f32x16 one[1];
    load_rows<__bf16, 1>(one, src, 1, (long long)row * D + 32 * (wave + 4 * i), in && s.owns(i), hi);
    x[i] = one[0];
    dn[i] = splat16(0.f);
  }
  if (p.dqkv) {
    const RecordOut rec(p.rec1, tile, p.rec1_size, lane);
    for (int ft = 0; ft < NT; ++ft)
      for (int m = 0; m < p.mats; ++m, ++seg) {
        bf16x8 op[2];
#pragma unroll
        for (int g = 0; g < 2; ++g) {
          op[g] = row_group(p.dqkv + (size_t)row * p.ldq + m * D + 32 * ft, g, hi, in);
          if (seg % 4 == wave) rec.put(p.rec1_dqkv + m * NG + 2 * ft, g, op[g]);
        }
#pragma unroll
        for (int i = 0; i < OT; ++i) {
          if (!s.owns(i)) continue;
#pragma unroll
          for (int g = 0; g < 2; ++g) dn[i] = E::mma(s.frag(seg, 2 * (wave + 4 * i) + g), op[g], dn[i]);
        }
      }
#pragma unroll
    for (int i = 0; i < OT; ++i) settle(dn[i]);
    s.stats(x, p.eps, mean, rstd);
    s.norm_back(x, dn, vec + oG1, mean, rstd);
#pragma unroll
    for (int i = 0; i < OT; ++i) {
      if (!s.owns(i)) continue;
      if (p.dxm_in) x[i] += load_part<NT>(p.dxm_in, tile, wave + 4 * i, lane);
      const f32x16 one[1] = {x[i]};
      if (!p.xmid && in) store_rows<__bf16, 1>(one, p.dx, 1, (long long)row * D + 32 * (wave + 4 * i), true, hi);
    }
    if (!p.xmid) return;
  }
  const BlockRecord at(D, p.f);
  const RecordOut rec(p.rec, tile, at.size, lane);
  const bool live = in && p.desc[in ? row : 0] >= 0;
  f32x16 xm[OT];
#pragma unroll
  for (int i = 0; i < OT; ++i) xm[i] = s.owns(i) ? load_part<NT>(p.xmid, tile, wave + 4 * i, lane) : splat16(0.f);
  s.stats(xm, p.eps, mean, rstd);                  // (its barriers: `vec` is there)
  bf16x8 dyop[NG], nop[NG];
#pragma unroll
  for (int i = 0; i < OT; ++i) {
#pragma unroll
    for (int r = 0; r < 16; ++r) x[i][r] = live ? x[i][r] : 0.f;
    dn[i] = splat16(0.f);
    if (!s.owns(i)) continue;
    const int t = wave + 4 * i;
    const f32x16 g = bias_tile(vec + oG2, t, hi), b = bias_tile(vec + oS2, t, hi);
    f32x16 y;
#pragma unroll
    for (int r = 0; r < 16; ++r) y[r] = fmaf((xm[i][r] - mean) * rstd, g[r], b[r]);
    s.hand_in(t, y);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const bf16x8 v = E::pack(x[i], q);
      ops2[2 * t + q][lane] = v;
      rec.put(at.dyb, 2 * t + q, v);
    }
  }
  __syncthreads();
  s.take(nop);
#pragma unroll
  for (int g = 0; g < NG; ++g) dyop[g] = ops2[g][lane];
  for (int c0 = 0, par = 0; c0 < NC; c0 += 4, par ^= 1) {
    const int c = c0 + wave;
    if (c < NC) {
      f32x16 v = bias_tile(vec + oB1, c, hi), g = splat16(0.f);
      s.product(v, seg + 3 * c, nop);
      s.product(g, seg + 3 * c + 1, dyop);
      settle(v);
      settle(g);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        float a, da;
        act_exact_both(v[r], p.act, &a, &da);
        v[r] = a;
        g[r] *= da;
      }
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const bf16x8 h = E::pack(g, q);
        hid[par][wave][q][lane] = h;
        rec.put(at.dh + 2 * c, q, h);
        rec.put(at.a + 2 * c, q, E::pack(v, q));
      }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < OT; ++i) {
      if (!s.owns(i)) continue;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if (c0 + k >= NC) break;
#pragma unroll
        for (int g = 0; g < 2; ++g) dn[i] = E::mma(s.frag(seg + 3 * (c0 + k) + 2, 2 * (wave + 4 * i) + g), hid[par][k][g][lane], dn[i]);
      }
    }
  }
  seg += 3 * NC;
#pragma unroll
  for (int i = 0; i < OT; ++i) settle(dn[i]);
  s.norm_back(xm, dn, vec + oG2, mean, rstd);      // (its barriers: everybody has taken `ops`)
#pragma unroll
  for (int i = 0; i < OT; ++i) {
    if (!s.owns(i)) continue;
    const int t = wave + 4 * i;
    x[i] += xm[i];
    store_part<NT>(x[i], p.dxm, tile, t, lane);
    s.hand_in(t, x[i]);
#pragma unroll
    for (int q = 0; q < 2; ++q) rec.put(at.dxmb, 2 * t + q, E::pack(x[i], q));
  }
  __syncthreads();
  s.take(nop);
  for (int ft = wave; ft < NT; ft += kStackWaves) {
    f32x16 v = splat16(0.f);
    s.product(v, seg + ft, nop);
    settle(v);
    if (in) {
#pragma unroll
      for (int g = 0; g < 2; ++g) row_put(p.dob + (size_t)row * D + 32 * ft, g, hi, E::pack(v, g));
    }
  }
}

void bw_stack_fwd_32(const StackFwd& p, hipStream_t st);
void bw_stack_bwd_32(const StackBwd& p, hipStream_t st);
void bw_stack_fwd_64(const StackFwd& p, hipStream_t st);
void bw_stack_bwd_64(const StackBwd& p, hipStream_t st);
void bw_stack_fwd_128(const StackFwd& p, hipStream_t st);
void bw_stack_bwd_128(const StackBwd& p, hipStream_t st);
void bw_stack_fwd_256(const StackFwd& p, hipStream_t st);
void bw_stack_bwd_256(const StackBwd& p, hipStream_t st);
template <int D>
inline void bw_stack_fwd_d(const StackFwd& p, hipStream_t st) {
  bw_stack_fwd_kernel<D><<<(p.rows + 31) / 32, 64 * kStackWaves, (size_t)stack_vec_floats(D, p.f) * 4, st>>>(p);
}
template <int D>
inline void bw_stack_bwd_d(const StackBwd& p, hipStream_t st) {
  bw_stack_bwd_kernel<D><<<(p.rows + 31) / 32, 64 * kStackWaves, (size_t)stack_vec_floats(D, p.f) * 4, st>>>(p);
}

}  // namespace bw
}  // namespace longer
