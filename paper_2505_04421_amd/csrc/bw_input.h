// Input generation backward (Section 3.5.1: H = act(x W1 + b1) W2 + b2 with x = [E + pos ; tdiff]) in one launch, a tile of 32 tokens
// per wave, in the registers' transposed layout and with the weight stream and tile blocks of bw_block.h: the rows x are formed
// from the inputs, the hidden values and their gradient 32 features at a time, the gradient of x goes out as dE and dtdiff.  What the
// parameter gradients contract (x, dH, activated hidden values, their gradient) goes to one record per tile.
//
// What bounds it: 3.8 KB of memory traffic per token at width 128 (inputs and dH 0.75 KB, record 2.5 KB, outputs 0.5 KB) and the activation
// beside the products.  As kernels over [token, feature] tensors (rows of x, rows of dH as bf16, two GEMMs, split of the gradient)
// the same work moved 7 KB per token: 295 us for 115 000 valid tokens of 90 users, 166 us here; the parameter gradients read
// contiguous records and went from 129 to 84 us with it.
#pragma once
#include "bw_block.h"

namespace longer {
namespace bw {

struct InputBwParams {
  const char* wstream;                      // per 32 hidden features: W1 (over the width), W2 transposed (over the width), W1 back (spread)
  const __bf16 *E, *pos, *td, *b1;          // item embeddings [B][L][de], positional [L][de], time differences [B][L][D - de]
  const int32_t* lens;
  int B, L, de, f, act;
  const float* dH;                          // [B][L][D]
  float *dE, *dtd;                          // zeros for padded tokens
  __bf16* rec;                              // tile records (InputRecord); tiles count rows of [B][L]
};

struct InputRecord {                        // offsets and size in sixteens of features (bw_block.h)
  int x, dyb, a, dh, size;
  __host__ __device__ InputRecord(int d, int f) : x(0), dyb(d / 16), a(2 * d / 16), dh(a + f / 16), size(dh + f / 16) {}
};
__host__ __device__ inline int bw_input_segs(int f) { return 3 * (f / 32); }
__host__ __device__ inline int bw_input_segs_padded(int f) { return (bw_input_segs(f) + 3) / 4 * 4; }

void bw_input_launch_64(const InputBwParams& p, hipStream_t st);
void bw_input_launch_128(const InputBwParams& p, hipStream_t st);

template <int D>
__global__ __launch_bounds__(64 * kBlkWaves, 2) void bw_input_kernel(const InputBwParams p) {
  constexpr int NT = D / 32, NG = D / 16, SEGV = NG * 64, PSEG = D >= 128 ? kBlkPanel : 4, NB = 3;
  using E = ET<__bf16>;
  __shared__ uint4 ring[NB * PSEG * SEGV];
  __shared__ __attribute__((aligned(16))) float vec[2048];       // b_1 (the hidden width is at most 2048)
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), j = lane & 31, hi = lane >> 5;
  const int NC = p.f / 32, nte = p.de / 32;
  const int tile = blockIdx.x * kBlkWaves + wave, row = tile * 32 + j, u = row / p.L, at = row - u * p.L;
  const bool stored = u < p.B;
  int len = 0;
  if (stored) { len = p.lens ? p.lens[u] : p.L; len = min(max(len, 0), p.L); }
  const bool valid = stored && at < len;
  auto put_grad = [&](int t, const f32x16& v) {
    if (!stored) return;
    float* to = t < nte ? p.dE + (size_t)row * p.de + 32 * t : p.dtd + (size_t)row * (D - p.de) + 32 * (t - nte);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const f32x4 w = {v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
      *(f32x4*)(to + 8 * q + 4 * hi) = w;
    }
  };
  if (!__syncthreads_or(valid ? 1 : 0)) {
#pragma unroll
    for (int t = 0; t < NT; ++t) put_grad(t, splat16(0.f));
    return;
  }
  char* rec = (char*)p.rec + (size_t)tile * InputRecord(D, p.f).size * 1024;
  const InputRecord rc(D, p.f);
  const unsigned lane0 = tile_lane_offset(lane, 0), lane1 = tile_lane_offset(lane, 1);
  const TileBuffer recb(rec, rc.size * 1024);
  auto put_rec = [&](int base, int g, bf16x8 v) { recb.put_once(g & 1 ? lane1 : lane0, (base + g) * 1024, __builtin_bit_cast(u32x4, v)); };      // (base is even)

  // everything that is read ahead of the first product is requested at once
  f32x16 x[NT], dy[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const bool emb = t < nte;                          // (no branch between the requests; a time difference has no second addend)
    f32x16 a[1], b[1];
    load_rows<__bf16, 1>(a, emb ? p.E : p.td, 0, emb ? (long long)row * p.de + 32 * t : (long long)row * (D - p.de) + 32 * (t - nte), valid, hi);
    load_rows<__bf16, 1>(b, p.pos, 0, emb ? (long long)at * p.de + 32 * t : 0, valid && emb, hi);
    x[t] = a[0] + b[0];
  }
  load_rows<__bf16, NT>(dy, p.dH, 1, (long long)row * D, valid, hi);
  WStream<SEGV, PSEG, NB, false, 64 * kBlkWaves> ws;
  for (int i = tid; i < p.f; i += 64 * kBlkWaves) vec[i] = (float)p.b1[i];
  ws.init(ring, p.wstream, bw_input_segs(p.f));        // (its barrier: `vec` is there)
  bf16x8 xop[NG], dyop[NG];
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    xop[g] = E::pack(x[g / 2], g & 1);
    dyop[g] = E::pack(dy[g / 2], g & 1);
    put_rec(rc.x, g, xop[g]);
    put_rec(rc.dyb, g, dyop[g]);
  }
  f32x16 dn[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) dn[t] = splat16(0.f);
  auto product = [&](f32x16& acc, const bf16x8 (&b)[NG]) {      // acc += (this segment's 32 output features) b
#pragma unroll
    for (int s = 0; s < NG; ++s) acc = E::mma(ws.template frag<bf16x8>(s), b[s], acc);
    ws.advance();
    settle(acc);
  };
  for (int c = 0; c < NC; ++c) {
    f32x16 v = bias_tile(vec, c, hi), g = splat16(0.f);
    product(v, xop);
    product(g, dyop);
    if (p.act == LONGER_ACT_RELU) {
#pragma unroll
      for (int r = 0; r < 16; ++r) { float a_, d_; act_both(v[r], LONGER_ACT_RELU, &a_, &d_, g[r]); v[r] = a_; g[r] = d_; }
    } else {
#pragma unroll
      for (int r = 0; r < 16; ++r) { float a_, d_; act_both(v[r], LONGER_ACT_GELU_ERF, &a_, &d_, g[r]); v[r] = a_; g[r] = d_; }
    }
    bf16x8 hop[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      hop[q] = E::pack(g, q);
      put_rec(rc.dh, 2 * c + q, hop[q]);
      put_rec(rc.a, 2 * c + q, E::pack(v, q));
    }
#pragma unroll
    for (int t = 0; t < NT; ++t)                                // dn += (all output features of 32 contracted ones) hop
#pragma unroll
      for (int q = 0; q < 2; ++q) dn[t] = E::mma(ws.template frag<bf16x8>(2 * t + q), hop[q], dn[t]);
    ws.advance();
  }
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    settle(dn[t]);
    put_grad(t, dn[t]);                                         // (a padded token's dH, and with it this, is zero)
  }
}

template <int D>
inline void bw_input_launch_d(const InputBwParams& p, hipStream_t st) {
  const size_t tiles = ((size_t)p.B * p.L + 31) / 32;
  bw_input_kernel<D><<<(unsigned)((tiles + kBlkWaves - 1) / kBlkWaves), 64 * kBlkWaves, 0, st>>>(p);
}

}  // namespace bw
}  // namespace longer
