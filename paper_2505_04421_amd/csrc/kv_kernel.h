// Key / value side of an attention layer (Eq. 6: K, V = LN1(rows) W, stored as fragments) at width 128 / 256, bf16: what MODE_KVPROJ of
// block_kernel.h does, for many tiles.
//
// Why.  A tile is read, projected and stored; there are thousands of them (nine a user at the headline batch) and only two matrices.  The block
// kernel sent both through LDS for every four tiles and waited for all of its stores at each segment.  Here a wave owns a FEATURE tile
// and keeps its part of W_K and W_V in registers (64 at width 128, 128 at width 256) while its workgroup goes from tile to tile,
// the next tile's rows on their way; LayerNorm sums and the normalised rows change hands through LDS (two barriers a tile).
//
// Users of different length need different numbers of key tiles, and as many workgroups as run at once have no successor that could take a
// share of the longer ones' work: there the needed tiles are counted and dealt out evenly (dealt by a fixed stride, with key tiles a user
// that divide the number of workgroups, a workgroup met the same key tile of every user; 512 users of 2 to 100 % of 16 key tiles took
// 63 us at width 128 and 148 at 256, as long as with all tiles needed).
//
// A launch, block kernel / this, us: 512 users of 16 key tiles, all needed, width 128 62 / 57, width 256 165 / 126; lengths spread evenly over 2 to
// 100 %: 52 / 35, 138 / 75; 8 key tiles 26 / 21, 70 / 47; 4 key tiles 14.8 / 14.3, 40 / 29; 200 users of 4 10.1 / 9.9, 19 / 17; 61 users of 196 rows,
// width 128, 9.8 / 7.5; 16 users of 625 rows, width 256, 16.8 / 12.0.  What bounds it: memory at width 128 (134 MB in and
// 134 out for the first of these, 4.7 TB/s), at width 256 (twice that, 4.3 TB/s) memory and the two barriers of a tile, which
// all eight waves of the one workgroup on a compute unit meet at together.
#pragma once
#include "block_kernel.h"

namespace longer {

constexpr int kv_workgroups(int d) { return d >= 256 ? 256 : 512; }      // as many as run at once

template <int D>
__global__ void __launch_bounds__(2 * D, D >= 256 ? 1 : 2) kv_kernel(const BlockParams p) {
  using T = __bf16;
  using E = ET<T>;
  using grp = typename E::grp;
  constexpr int NT = D / 32, NG = D / 16, MOST = kv_workgroups(D);
  __shared__ grp ops[2][NG][64];                     // normalised rows: [parity][group][lane]
  __shared__ float2 sums[2][NT][64];                 // [parity][wave][lane]: mean and squared deviations of the wave's features
  const int lane = threadIdx.x & 63, j = lane & 31, hi = lane >> 5, ft = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  typedef __attribute__((address_space(1))) const grp ggrp;
  typedef __attribute__((address_space(1))) const f32x4 gf32x4;
  typedef __attribute__((address_space(1))) const bf16x4 gbf16x4;

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

  // Which rows exist, and which tiles somebody may read (a user's first `need`): as in block_kernel.h.  User and key tile are wave-uniform.
  struct Tile { int u, kt, tu, need; };
  auto user = [&](int u) {
    int len = p.lens ? p.lens[u] : p.L;
    len = min(max(len, 0), p.L);
    Tile t = {u, 0, (len + p.K - 1) / p.K, p.tiles_per_user};
    if (!p.key_self) t.need = min(t.need, (p.m0 + t.tu + 31) / 32);
    return t;
  };
  int du = 0, dk = 0;                                // tiles dealt out by a stride: users and key tiles in it
  auto step = [&](Tile t) {                          // the workgroup's next tile (the caller knows that there is one)
    if (du + dk > 0) {
      const int kt = t.kt + dk, over = kt >= p.tiles_per_user;
      t = user(t.u + du + over);
      t.kt = kt - (over ? p.tiles_per_user : 0);
      return t;
    }
    if (++t.kt < t.need) return t;
    do t = user(t.u + 1); while (t.need == 0);
    return t;
  };
  // One round of workgroups: a tile each.  More tiles: every workgroup takes as many needed tiles as the others, `left` in all.  With all of
  // them needed, by a stride: what runs at once then writes one stretch of memory (256 users of nine tiles, width 256, buffers not
  // in the caches: 40.3 us, in runs of consecutive tiles 45.2), and the workgroups that meet one key tile of every user have no less to do than
  // the others.  Else in runs: each thread counts the tiles of its share of the users to find the first.
  int left;
  Tile t;
  {
    const int b = (int)blockIdx.x, per = p.tiles_per_user;
    const long long all = (long long)p.B * per;
    const bool round = all <= MOST;
    if (round || !p.lens || p.key_self || (per == 1 && p.m0 > 0)) {      // (a user's first tile has its global rows)
      t = user(b / per);
      t.kt = b - t.u * per;
      left = round ? (t.kt < t.need ? 1 : 0) : (int)((all - b + MOST - 1) / MOST);
      du = MOST / per; dk = MOST - du * per;
    } else {
      __shared__ int count[NT];
      __shared__ Tile start;
      const int tid = (int)threadIdx.x, u0 = (int)((long long)tid * p.B / (2 * D)), u1 = (int)((long long)(tid + 1) * p.B / (2 * D));
      Tile mine = {};
      int own = 0;
      for (int u = u0; u < u1; ++u) { mine = user(u); own += mine.need; }
      int upto = own;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) { const int v = __shfl_up(upto, o, 64); if (lane >= o) upto += v; }
      if (lane == 63) count[ft] = upto;
      __syncthreads();
      int n = 0;
#pragma unroll
      for (int w = 0; w < NT; ++w) { if (w < ft) upto += count[w]; n += count[w]; }
      const int first = (int)((long long)b * n / MOST);
      left = __builtin_amdgcn_readfirstlane((int)((long long)(b + 1) * n / MOST) - first);
      if (upto - own <= first && first < upto) {       // (one thread)
        int kt = first - (upto - own);
        if (u1 - u0 > 1)
          for (mine = user(u0); kt >= mine.need; mine = user(mine.u + 1)) kt -= mine.need;
        mine.kt = kt;
        start = mine;
      }
      __syncthreads();
      t.u = __builtin_amdgcn_readfirstlane(start.u); t.kt = __builtin_amdgcn_readfirstlane(start.kt);
      t.tu = __builtin_amdgcn_readfirstlane(start.tu); t.need = __builtin_amdgcn_readfirstlane(start.need);
    }
    if (left == 0) return;
  }
  auto exists = [&](const Tile& t) {
    const int c = 32 * t.kt + j, i = c - p.m0;
    return c < p.rows_per_user && (c < p.m0 || (p.key_self ? i >= first_slot(p.k, t.tu, p.q_learn) : i < t.tu));
  };
  // fp32 rows: requested a tile ahead, the bf16 global rows in front of them (a wave-uniform question) beside them
  const bool ahead = p.src1.f32;
  f32x4 raw[4];
  bf16x4 front[4];
  auto request = [&](const Tile& t) {
    if (!ahead) return;
    const int c = 32 * t.kt + j;
    const bool there = exists(t), first = c < p.m0;
    const bool from0 = there && first && p.src0.f32, from1 = there && !first;      // (one that does not exist reads the first)
    const float* row = from0 ? reinterpret_cast<const float*>(p.src0.p) + p.src0.ustride * t.u + (long long)c * D
                             : reinterpret_cast<const float*>(p.src1.p) + (from1 ? p.src1.ustride * t.u + (long long)(c - p.m0) * D : 0);
#pragma unroll
    for (int q = 0; q < 4; ++q) raw[q] = *(gf32x4*)(row + 32 * ft + 4 * hi + 8 * q);
    if (!p.src0.f32 && 32 * t.kt < p.m0) {
      const __bf16* row0 = reinterpret_cast<const __bf16*>(p.src0.p) + (there && first ? p.src0.ustride * t.u + (long long)c * D : 0);
#pragma unroll
      for (int q = 0; q < 4; ++q) front[q] = *(gbf16x4*)(row0 + 32 * ft + 4 * hi + 8 * q);
    }
  };

  request(t);
  for (int par = 0; left > 0; par ^= 1) {
    const bool valid = exists(t);
    f32x16 x;
    if (ahead) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int e = 0; e < 4; ++e) { const float one = raw[q][e]; x[4 * q + e] = valid ? one : 0.f; }
      if (!p.src0.f32 && 32 * t.kt < p.m0) {
        const bool global = valid && 32 * t.kt + j < p.m0;
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int e = 0; e < 4; ++e) x[4 * q + e] = global ? (float)front[q][e] : x[4 * q + e];
      }
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
    const Tile now = t;
    if (--left > 0) { t = step(t); request(t); }
    __syncthreads();             // (the other parity's operands were last read ahead of the barrier before)
    f32x16 ak = splat16(0.f), av = splat16(0.f);     // no b_K, no b_V: see block_kernel.h
#pragma unroll
    for (int s = 0; s < NG; ++s) {
      const grp b = ops[par][s][lane];
      ak = E::mma(wk[s], b, ak);
      av = E::mma(b, wv[s], av);                     // operands swapped: lane = feature
    }
    settle(ak); settle(av);
    const size_t fo = (size_t)now.u * p.kv_ustride + ((size_t)(now.kt * NT + ft) * 2) * 1024 + 16 * lane;
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      *reinterpret_cast<grp*>(p.kst + fo + g * 1024) = E::pack(ak, g);
      *reinterpret_cast<grp*>(p.vst + fo + g * 1024) = E::pack(av, g);
    }
  }
}

int launch_kv(int d, const BlockParams& p, hipStream_t stream);

}  // namespace longer
