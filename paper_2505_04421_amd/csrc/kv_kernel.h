// Key / value side of an attention layer (Eq. 6: K, V = LN1(rows) W, stored as fragments) at width 128 / 256, bf16: what MODE_KVPROJ of
// block_kernel.h does, for many tiles.
//
// Why.  A tile is read, projected and stored; there are thousands of them (nine a user at the headline batch) and only two matrices.  The block
// kernel sent both through LDS for every four tiles and waited for all of its stores at each segment.  Here a wave owns a FEATURE tile
// and keeps its part of W_K and W_V in registers (64 at width 128, 128 at width 256) while its workgroup goes from tile to tile,
// the next tile's rows on their way; LayerNorm sums and the normalised rows change hands through LDS (two barriers a tile).
//
// A launch, block kernel / this: 66 048 rows (256 users) width 256 55.9 / 38.9 us, width 128 22.5 / 18.8; 512 ragged users of up to 321 rows,
// width 128, 33.8 / 33.2; 61 users of 196 rows, width 128, 9.1 / 6.7; 16 users of 625 rows, width 256, 18.0 / 11.9: faster at every number of
// tiles, so there is no rule.  What bounds it: memory at width 128 (68 MB in and out, 3.6 TB/s), at width 256 (134 MB, 3.4 TB/s)
// memory and the two barriers of a tile, which all eight waves of the one workgroup on a compute unit meet at together.
#pragma once
#include "block_kernel.h"

namespace longer {

template <int D>
__global__ void __launch_bounds__(2 * D, D >= 256 ? 1 : 2) kv_kernel(const BlockParams p, int tiles) {
  using T = __bf16;
  using E = ET<T>;
  using grp = typename E::grp;
  constexpr int NT = D / 32, NG = D / 16;
  __shared__ grp ops[2][NG][64];                     // normalised rows: [parity][group][lane]
  __shared__ float2 sums[2][NT][64];                 // [parity][wave][lane]: mean and squared deviations of the wave's features
  const int lane = threadIdx.x & 63, j = lane & 31, hi = lane >> 5, ft = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  typedef __attribute__((address_space(1))) const grp ggrp;
  typedef __attribute__((address_space(1))) const f32x4 gf32x4;

  // split layout: [vectors][K V of feature tile 0][K V of feature tile 1] ...
  grp wk[NG], wv[NG];
  const char* wl = p.wbase + (size_t)(1 + 2 * ft) * (NG * 1024) + 16 * lane;
#pragma unroll
  for (int s = 0; s < NG; ++s) {
    wk[s] = *(ggrp*)(wl + s * 1024);
    wv[s] = *(ggrp*)(wl + (NG + s) * 1024);
  }
  const VecLayout vl{D, p.FF};
  const float* vec = reinterpret_cast<const float*>(p.wbase);
  const f32x16 gain = bias_tile(vec + vl.ln1_g(), ft, hi), shift = bias_tile(vec + vl.ln1_b(), ft, hi);

  // Which rows exist, and which tiles somebody may read: as in block_kernel.h (user and key tile are wave-uniform)
  struct Tile { int u, kt, tu; };
  auto locate = [&](int tile) {
    Tile t;
    t.u = tile / p.tiles_per_user; t.kt = tile - t.u * p.tiles_per_user;
    int len = p.lens ? p.lens[t.u] : p.L;
    len = min(max(len, 0), p.L);
    t.tu = (len + p.K - 1) / p.K;
    return t;
  };
  auto from = [&](int tile) {                        // the first tile from here on that is needed
    for (; tile < tiles; tile += (int)gridDim.x) {
      const Tile t = locate(tile);
      if (p.key_self || 32 * t.kt < p.m0 + t.tu) break;
    }
    return tile;
  };
  auto exists = [&](const Tile& t) {
    const int c = 32 * t.kt + j, i = c - p.m0;
    return c < p.rows_per_user && (c < p.m0 || (p.key_self ? i >= first_slot(p.k, t.tu, p.q_learn) : i < t.tu));
  };
  // rows of a tile without global rows, fp32: requested a tile ahead
  auto direct = [&](const Tile& t) { return p.src1.f32 && 32 * t.kt >= p.m0; };
  f32x4 raw[4];
  auto request = [&](const Tile& t) {
    if (!direct(t)) return;
    const long long off = exists(t) ? p.src1.ustride * t.u + (long long)(32 * t.kt + j - p.m0) * D : 0;      // (one that does not exist reads the first)
    const float* row = reinterpret_cast<const float*>(p.src1.p) + off + 32 * ft + 4 * hi;
#pragma unroll
    for (int q = 0; q < 4; ++q) raw[q] = *(gf32x4*)(row + 8 * q);
  };

  int tile = from((int)blockIdx.x);
  if (tile >= tiles) return;
  request(locate(tile));
  for (int par = 0; tile < tiles; par ^= 1) {
    const Tile t = locate(tile);
    const bool valid = exists(t);
    f32x16 x;
    if (direct(t)) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int e = 0; e < 4; ++e) { const float one = raw[q][e]; x[4 * q + e] = valid ? one : 0.f; }
    } else {
      const int c = 32 * t.kt + j;
      const bool first = c < p.m0;
      f32x16 one[1];
      load_rows<T, 1>(one, first ? p.src0.p : p.src1.p, first ? p.src0.f32 : p.src1.f32,
                      (first ? p.src0.ustride : p.src1.ustride) * t.u + (long long)(first ? c : c - p.m0) * D + 32 * ft, valid, hi);
      x = one[0];
    }
    // LayerNorm over all features: every wave's own mean and squared deviations, combined
    float m = 0.f, v = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) m += x[r];
    m = sum_halves(m) * (1.f / 32.f);
#pragma unroll
    for (int r = 0; r < 16; ++r) { const float q = x[r] - m; v = fmaf(q, q, v); }
    sums[par][ft][lane] = make_float2(m, sum_halves(v));
    __syncthreads();
    float mean = 0.f, var = 0.f;
#pragma unroll
    for (int w = 0; w < NT; ++w) mean += sums[par][w][lane].x;
    mean *= 1.f / NT;
#pragma unroll
    for (int w = 0; w < NT; ++w) { const float2 q = sums[par][w][lane]; var += fmaf((q.x - mean) * (q.x - mean), 32.f, q.y); }
    const float rstd = __builtin_amdgcn_rsqf(var * (1.f / D) + p.eps);
    f32x16 y;
#pragma unroll
    for (int r = 0; r < 16; ++r) y[r] = fmaf((x[r] - mean) * rstd, gain[r], shift[r]);
#pragma unroll
    for (int g = 0; g < 2; ++g) ops[par][2 * ft + g][lane] = E::pack(y, g);
    const int next = from(tile + (int)gridDim.x);
    if (next < tiles) request(locate(next));
    __syncthreads();             // (the other parity's operands were last read ahead of the barrier before)
    f32x16 ak = splat16(0.f), av = splat16(0.f);     // no b_K, no b_V: see block_kernel.h
#pragma unroll
    for (int s = 0; s < NG; ++s) {
      const grp b = ops[par][s][lane];
      ak = E::mma(wk[s], b, ak);
      av = E::mma(b, wv[s], av);                     // operands swapped: lane = feature
    }
    settle(ak); settle(av);
    const size_t fo = (size_t)t.u * p.kv_ustride + ((size_t)(t.kt * NT + ft) * 2) * 1024 + 16 * lane;
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      *reinterpret_cast<grp*>(p.kst + fo + g * 1024) = E::pack(ak, g);
      *reinterpret_cast<grp*>(p.vst + fo + g * 1024) = E::pack(av, g);
    }
    tile = next;
  }
}

// tiles: B x tiles_per_user.  As many workgroups as run at once.
int launch_kv(int d, const BlockParams& p, int tiles, hipStream_t stream);

}  // namespace longer
