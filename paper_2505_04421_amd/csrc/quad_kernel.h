// The transformer-block kernel for launches with few tiles: a 32-row tile given to four waves, one per SIMD of a
// compute unit, or eight at width 256 (bf16).
//
//   MODE_SCORE  candidate scoring of the KV-cache serving path (Section 3.6.3), all layers;
//   MODE_ATTN   query side of one layer over stored K/V fragments (the cache build's sequence rows);
//   MODE_STACK  the whole reduced stack of a user with at most two tiles (m + k <= 64) in one workgroup of eight waves.
//
// Why.  A request scores a hundred candidates (25 tiles), a cache build runs two tiles per user: a handful of
// workgroups on 256 compute units, whose time is one tile's chain of dependent products.  Here feature tile t of the
// rows, of every product's result and its attention heads belong to wave t % 4 (t % 8), and the FFN's hidden chunks are dealt
// out the same way, so the chain is a quarter (an eighth) as long; operand groups change hands through LDS.  The waves
// share no weights, so each fetches its fragments from L2 itself, from the same packed streams as the other kernels
// (their segments are found by index).  With many tiles the streams' traffic and the idle matrix pipes cost more than the
// shorter chain gains: the rule is at quad_pays in longer_api.hip.
#pragma once
#include "block_kernel.h"

namespace longer {

// waves that share a tile: one feature tile each at width 128 and 256, hidden chunks dealt out among all
constexpr int quad_waves(int d) { return d >= 256 ? 8 : 4; }
constexpr int quad_tiles(int mode) { return mode == MODE_STACK ? 2 : 1; }      // tiles of a workgroup

// Segment indices inside one block's packed stream (layouts: device.h).  attn: the attention half of the split (or
// pair) layout, without K and V; else the fused layouts.
enum QuadLayout { QUAD_PLAIN = 0, QUAD_PAIR = 1 };
template <int LAYOUT, int D>
struct QuadSegs {
  static constexpr int NT = D / 32, V0 = LAYOUT == QUAD_PAIR ? 2 : 1;       // V0: segments in front of the matrices
  int NC; bool attn;
  __device__ __forceinline__ int q(int t) const { return V0 + (attn ? t : LAYOUT == QUAD_PAIR ? 6 * (t / 2) + (t & 1) : 3 * t); }
  __device__ __forceinline__ int k(int t) const { return q(t) + (LAYOUT == QUAD_PAIR ? 2 : 1); }
  __device__ __forceinline__ int v(int t) const { return q(t) + (LAYOUT == QUAD_PAIR ? 4 : 2); }
  __device__ __forceinline__ int o(int t) const { return V0 + (attn ? NT : 3 * NT) + t; }
  __device__ __forceinline__ int ffn() const { return V0 + (attn ? 2 * NT : 4 * NT); }
  __device__ __forceinline__ int w1(int c) const {
    if (LAYOUT == QUAD_PAIR) return ffn() + 4 * (c / 2) + (c & 1);
    return ffn() + (ffn_skewed(2, D) ? (c < 2 ? c : 2 * c) : 2 * c);
  }
  __device__ __forceinline__ int w2(int c) const {
    if (LAYOUT == QUAD_PAIR) return w1(c) + 2;
    return ffn() + (ffn_skewed(2, D) ? (c < NC - 1 ? 3 + 2 * c : 2 * NC) : 2 * c + 1);
  }
  __device__ __forceinline__ int block() const { return 2 + (attn ? 2 : 4) * NT + 2 * NC; }
};

template <int D, int DH, int MODE, int W, int LAYOUT, bool RELU>
__global__ void __launch_bounds__(64 * quad_waves(D) * quad_tiles(MODE), 1) quad_kernel(const BlockParams p) {
  using T = __bf16;
  using E = ET<T>;
  using grp = typename E::grp;
  using hgrp = typename E::hgrp;
  constexpr int WV = quad_waves(D), TS = quad_tiles(MODE), kThr = 64 * WV * TS;
  constexpr int NT = D / 32, NG = D / 16, OT = (NT + WV - 1) / WV, HPT = 32 / DH, GPH = DH / 16;
  constexpr bool SCORE = MODE == MODE_SCORE, STACK = MODE == MODE_STACK;
  static_assert(SCORE || STACK || MODE == MODE_ATTN, "quad kernel modes");
  static_assert(!STACK || OT == 1, "the stack's K / V hand-over takes one feature tile per wave");
  __shared__ grp ops_[TS][NG][64];                   // per tile, [group][lane]: operand of the next products
  __shared__ hgrp hid_[TS][2][WV][2][64];            // activated hidden chunks: [parity][wave][group][lane]
  __shared__ float2 sums_[TS][WV][64];
  __shared__ grp kvl[STACK ? TS : 1][STACK ? NT : 1][2][2][64];      // self layers: [key tile][feature tile][K, V][group][lane]
  __shared__ f32x4 vecl[D * 4];                      // the block's fp32 vectors (at most one segment)
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6), j = lane & 31, hi = lane >> 5;
  const int ts = TS == 1 ? 0 : wv / WV, wave = TS == 1 ? wv : wv % WV;     // tile of the workgroup, wave of the tile
  auto& ops = ops_[ts];
  auto& hid = hid_[ts];
  auto& sums = sums_[ts];
  const int NC = p.FF / 32;
  QuadSegs<LAYOUT, D> sg = {NC, !SCORE};               // (the stack's first block is the cross layer's attention half)
  auto owns = [&](int i) { return NT >= WV || wave + WV * i < NT; };

  // ------------------------------------------------------------------ rows
  bool valid, inrange;
  int usr, Tu, tile;
  long long out_off;
  uint32_t tilebits = 0;
  int lo1 = 0, hi1 = 0, lo2 = 0, hi2 = 0, kthi = 0;    // visible key ranges of the stored keys, their tiles
  int slo1 = 0, shi1 = 0, slo2 = 0, shi2 = 0;          // the stack's self layers
  const int widx = W == 16 ? 0 : j / (2 * W);
  uint32_t wmask[16 / W];
#pragma unroll
  for (int w = 0; w < 16 / W; ++w) { wmask[w] = widx == w ? 0xffffffffu : 0u; asm("" : "+v"(wmask[w])); }
  f32x16 x[OT];
  auto load_own = [&](const void* base, int f32, long long off) {
#pragma unroll
    for (int i = 0; i < OT; ++i) {
      f32x16 one[1];
      load_rows<T, 1>(one, base, f32, off + 32 * (wave + WV * i), valid && owns(i), hi);
      x[i] = one[0];
    }
  };
  if (SCORE) {
    // (users are dealt to the accelerator dies like in the other kernels; a few users' tiles go to all dies)
    int u;
    if (p.xcds > 1) { const int sq = (int)blockIdx.x / p.xcds; u = (int)blockIdx.x % p.xcds + p.xcds * (sq / p.wg_per_user); tile = sq % p.wg_per_user; }
    else { u = (int)blockIdx.x / p.wg_per_user; tile = (int)blockIdx.x % p.wg_per_user; }
    if (u >= p.B) return;
    const int a = 32 * tile + j, cand = a / p.m, gi = a - cand * p.m;
    inrange = valid = cand < p.C;
    int len = p.lens ? p.lens[u] : p.L; len = min(max(len, 0), p.L);
    usr = u; Tu = (len + p.K - 1) / p.K;
    out_off = ((long long)u * p.C * p.m + a) * D;
    load_own(p.Gc, 0, out_off);
    const uint32_t vb = (uint32_t)__ballot(valid);
    const int gbase = p.m * (j / p.m);
    tilebits = ((range_bits(gbase + (p.gmask_causal ? gi : 0), gbase + p.m, 0) & vb) >> (4 * hi)) >> (2 * W * widx);
  } else {
    if (STACK) { usr = (int)blockIdx.x; tile = ts; }
    else { usr = (int)blockIdx.x / p.tiles_per_user; tile = (int)blockIdx.x - usr * p.tiles_per_user; }
    const int a = p.q0 + 32 * tile + j;
    inrange = usr < p.B && (32 * tile + j) < p.rows_per_user;
    int len = p.lens ? p.lens[usr] : p.L; len = min(max(len, 0), p.L);
    const int tu = (len + p.K - 1) / p.K;
    const bool glob = a < p.m;
    const int i = a - p.m, i0 = first_slot(p.k, tu, p.q_learn);
    valid = inrange && (glob || i >= i0);
    Tu = tu;
    out_off = p.X_ustride * usr + (long long)a * D;
    const int tok = glob ? 0 : (p.q_learn ? tu - 1 : slot_token(i, p.k, tu, p.k_uni));
    const int row = glob ? a : (p.gather_recent ? tok : i);
    load_own(glob ? p.src0.p : p.src1.p, glob ? p.src0.f32 : p.src1.f32, (glob ? p.src0.ustride : p.src1.ustride) * usr + (long long)row * D);
    const int s0 = p.key_self ? i0 : 0;
    if (glob) {
      lo1 = p.gmask_causal ? a : 0; hi1 = p.KG;
      lo2 = p.KG + s0; hi2 = p.KG + (p.key_self ? p.k : tu);
    } else {
      lo2 = p.KG + s0; hi2 = p.KG + (p.key_self ? i : tok) + 1;
    }
    if (!valid) { hi1 = lo1; hi2 = lo2; }
    kthi = (p.KG + (p.key_self ? p.k : tu) + 31) / 32;
    if (STACK && valid) {      // keys of a self-causal layer: the user's own rows, key index = row index
      if (glob) { slo1 = p.gmask_causal ? a : 0; shi1 = p.m; slo2 = p.m + i0; shi2 = p.m + p.k; }
      else { slo2 = p.m + i0; shi2 = p.m + i + 1; }
    }
  }

  const char* wl = p.wbase;                            // the current block's stream
  // The chain touches every weight once, and a first touch of a die's L2 takes several times as long as a hit: the
  // workgroups of a die (every eighth) bring the whole stream in at once, each its share.
  {
    const unsigned peers = (gridDim.x + 7 - (blockIdx.x & 7)) / 8;
    const unsigned lines = (unsigned)((sg.block() + (p.n_layers - 1) * (2 + 4 * NT + 2 * NC)) * (D / 2));
    unsigned keep = 0;
    for (unsigned i = (blockIdx.x >> 3) * kThr + tid; i < lines; i += peers * kThr) keep |= *reinterpret_cast<const unsigned*>(wl + (size_t)i * 128);
    asm volatile("" :: "v"(keep));
  }
  auto frag = [&](int seg, int s) -> grp { return *reinterpret_cast<const grp*>(wl + ((size_t)(seg * NG + s) * 64 + lane) * 16); };
  // acc + (segment seg: 32 result features) b; swapped: result with lane = feature
  auto product = [&](f32x16 acc, int seg, const grp (&b)[NG], bool swapped) -> f32x16 {
    grp f[NG];
#pragma unroll
    for (int s = 0; s < NG; ++s) f[s] = frag(seg, s);
#pragma unroll
    for (int s = 0; s < NG; ++s) acc = swapped ? E::mma(b[s], f[s], acc) : E::mma(f[s], b[s], acc);
    return acc;
  };
  const VecLayout vl{D, p.FF};
  const float* vec = reinterpret_cast<const float*>(vecl);
  // row sums of all waves (two numbers per row); the barriers also say that everybody is done with `ops`
  auto row_sums = [&](float a, float b) -> float2 {
    a = sum_halves(a); b = sum_halves(b);
    __syncthreads();
    sums[wave][lane] = make_float2(a, b);
    __syncthreads();
    float2 r = make_float2(0.f, 0.f);
#pragma unroll
    for (int w = 0; w < WV; ++w) { const float2 q = sums[w][lane]; r.x += q.x; r.y += q.y; }
    return r;
  };
  // LayerNorm of the rows as the next products' operand, in every wave
  auto normalise = [&](int og, int ob, grp (&b)[NG]) {
    float s = 0.f, q = 0.f;
#pragma unroll
    for (int i = 0; i < OT; ++i) {
      if (!owns(i)) continue;
#pragma unroll
      for (int r = 0; r < 16; ++r) { s += x[i][r]; q = fmaf(x[i][r], x[i][r], q); }
    }
    const float2 t = row_sums(s, q);
    const float mean = t.x * (1.0f / D), var = fmaxf(t.y * (1.0f / D) - mean * mean, 0.f);
    const float rstd = __builtin_amdgcn_rsqf(var + p.eps), shift = -mean * rstd;
#pragma unroll
    for (int i = 0; i < OT; ++i) {
      if (!owns(i)) continue;
      const f32x16 g = bias_tile(vec + og, wave + WV * i, hi), c = bias_tile(vec + ob, wave + WV * i, hi);
      f32x16 y;
#pragma unroll
      for (int r = 0; r < 16; ++r) y[r] = fmaf(fmaf(x[i][r], rstd, shift), g[r], c[r]);
#pragma unroll
      for (int g2 = 0; g2 < 2; ++g2) ops[2 * (wave + WV * i) + g2][lane] = E::pack(y, g2);
    }
    __syncthreads();
#pragma unroll
    for (int g = 0; g < NG; ++g) b[g] = ops[g][lane];
  };

  for (int layer = 0; layer < p.n_layers; ++layer) {
    const bool selfl = STACK && layer > 0;             // K and V made here, handed to the user's other tile through LDS
    if (layer > 0) __syncthreads();                    // nobody still reads the previous block's vectors
    for (int i = tid; i < (9 * D + p.FF) / 4; i += kThr) vecl[i] = reinterpret_cast<const f32x4*>(wl)[i];
    __syncthreads();
    {
      grp xn[NG];
      normalise(vl.ln1_g(), vl.ln1_b(), xn);
      grp oo[OT][2];
#pragma unroll
      for (int i = 0; i < OT; ++i) {
        const int ft = wave + WV * i;
        f32x16 aq, ak, av;
        if (owns(i)) {
          aq = product(bias_tile(vec + vl.bq(), ft, hi), sg.q(ft), xn, false);
          if (SCORE || selfl) {
            ak = product(splat16(0.f), sg.k(ft), xn, false);     // no b_K, no b_V: see block_kernel.h
            av = product(splat16(0.f), sg.v(ft), xn, true);
          }
          if (selfl) {
            settle(ak); settle(av);
#pragma unroll
            for (int g = 0; g < 2; ++g) { kvl[ts][ft][0][g][lane] = E::pack(ak, g); kvl[ts][ft][1][g][lane] = E::pack(av, g); }
          }
        }
        if (selfl) __syncthreads();
        if (!owns(i)) continue;
        settle(aq);
        aq *= p.scale_l2e;
        grp qop[2];
#pragma unroll
        for (int g = 0; g < 2; ++g) qop[g] = E::pack(aq, g);
        float mrun[HPT], lrun[HPT];
        f32x16 acc[HPT];
#pragma unroll
        for (int hh = 0; hh < HPT; ++hh) { mrun[hh] = kNegBig; lrun[hh] = 0.f; acc[hh] = splat16(0.f); }
        // stored K/V fragments (wave-uniform user, scalar loop control); two key tiles on their way
        const char* kb; const char* vb; int nkt, rlo = 0, rhi = 0;
        const int tuu = __builtin_amdgcn_readfirstlane(Tu);
        if (selfl) {
          kb = vb = nullptr; nkt = (p.m + p.k + 31) / 32;
        } else if (!SCORE) {
          kb = p.kst + (size_t)usr * p.kv_ustride; vb = p.vst + (size_t)usr * p.kv_ustride;
          nkt = __builtin_amdgcn_readfirstlane(kthi);
        } else {
          if (layer == 0) {
            kb = p.cache + (size_t)usr * p.c0_ustride; vb = kb + p.c0_voff;
            nkt = min(p.kt0, (tuu + 31) / 32); rhi = tuu;
          } else {
            kb = p.cache + p.c1_off + (size_t)(layer - 1) * p.c1_lstride + (size_t)usr * p.c1_ustride;
            vb = kb + p.c1_voff;
            nkt = tuu > 0 ? p.kt1 : 0; rlo = first_slot(p.k, tuu, p.q_learn); rhi = p.k;
          }
          if (!valid) rhi = rlo;
        }
        grp kn[2][2], vn[2][2];
        auto fetch = [&](int kt, int b) {
          if (selfl) {
#pragma unroll
            for (int g = 0; g < 2; ++g) { kn[b][g] = kvl[STACK ? kt : 0][STACK ? ft : 0][0][g][lane]; vn[b][g] = kvl[STACK ? kt : 0][STACK ? ft : 0][1][g][lane]; }
            return;
          }
          const size_t fo = ((size_t)(kt * NT + ft) * 2) * 1024 + lane * 16;
#pragma unroll
          for (int g = 0; g < 2; ++g) {
            kn[b][g] = *reinterpret_cast<const grp*>(kb + fo + g * 1024);
            vn[b][g] = *reinterpret_cast<const grp*>(vb + fo + g * 1024);
          }
        };
        if (nkt > 0) fetch(0, 0);
        if (nkt > 1) fetch(1, 1);
        if (SCORE) {   // keys of the lane's own tile: the candidate's own globals
          grp kop[2], vop[2];
#pragma unroll
          for (int g = 0; g < 2; ++g) { kop[g] = E::pack(ak, g); vop[g] = E::pack(av, g); }
#pragma unroll
          for (int hh = 0; hh < HPT; ++hh) {
            f32x16 S = splat16(0.f);
#pragma unroll
            for (int g2 = 0; g2 < GPH; ++g2) S = E::mma(kop[hh * GPH + g2], qop[hh * GPH + g2], S);
            grp pop[2];
            softmax_window<T, W>(S, widx, wmask, tilebits, mrun[hh], lrun[hh], acc[hh], pop);
#pragma unroll
            for (int g = 0; g < 2; ++g) acc[hh] = E::mma(vop[g], pop[g], acc[hh]);
          }
        }
        auto key_tile = [&](int kt, int b) {
          const uint32_t bits = SCORE ? range_bits(rlo, rhi, 32 * kt)
                              : selfl ? range_bits(slo1, shi1, 32 * kt) | range_bits(slo2, shi2, 32 * kt) : range_bits(lo1, hi1, 32 * kt) | range_bits(lo2, hi2, 32 * kt);
          const uint32_t ab = (bits >> (4 * hi)) & kTileBits;
          const bool none = __builtin_amdgcn_ballot_w64(ab != 0) == 0;           // nobody sees any of these keys
          const bool full = __builtin_amdgcn_ballot_w64(ab != kTileBits) == 0;   // everybody sees all of them
          grp kf[2], vf[2];
#pragma unroll
          for (int g = 0; g < 2; ++g) { kf[g] = kn[b][g]; vf[g] = vn[b][g]; }
          if (kt + 2 < nkt) fetch(kt + 2, b);
          if (none) return;
          const f32x16 vis = full ? splat16(0.f) : mask_tile(ab);
#pragma unroll
          for (int hh = 0; hh < HPT; ++hh) {
            f32x16 S = vis;
#pragma unroll
            for (int g2 = 0; g2 < GPH; ++g2) S = E::mma(kf[hh * GPH + g2], qop[hh * GPH + g2], S);
            grp pop[2];
            softmax_step<T, false>(S, 0u, mrun[hh], lrun[hh], acc[hh], pop);
#pragma unroll
            for (int g = 0; g < 2; ++g) acc[hh] = E::mma(vf[g], pop[g], acc[hh]);
          }
        };
        for (int kt = 0; kt < nkt; kt += 2) {
          key_tile(kt, 0);
          if (kt + 1 < nkt) key_tile(kt + 1, 1);
        }
        f32x16 o;
        float inv[HPT];
#pragma unroll
        for (int hh = 0; hh < HPT; ++hh) { settle(acc[hh]); inv[hh] = lrun[hh] > 0.f ? __builtin_amdgcn_rcpf(lrun[hh]) : 0.f; }
#pragma unroll
        for (int r = 0; r < 16; ++r) o[r] = acc[HPT == 1 ? 0 : r / 8][r] * inv[HPT == 1 ? 0 : r / 8];
#pragma unroll
        for (int g = 0; g < 2; ++g) oo[i][g] = E::pack(o, g);
      }
      // (every wave took the normalised rows out of `ops` before its attention; this barrier says so)
      __syncthreads();
#pragma unroll
      for (int i = 0; i < OT; ++i) {
        if (!owns(i)) continue;
#pragma unroll
        for (int g = 0; g < 2; ++g) ops[2 * (wave + WV * i) + g][lane] = oo[i][g];
      }
      __syncthreads();
#pragma unroll
      for (int g = 0; g < NG; ++g) xn[g] = ops[g][lane];
#pragma unroll
      for (int i = 0; i < OT; ++i) {
        if (!owns(i)) continue;
        x[i] += bias_tile(vec + vl.bo(), wave + WV * i, hi);
        x[i] = product(x[i], sg.o(wave + WV * i), xn, false);
        settle(x[i]);
      }
    }
    grp xn[NG];
    normalise(vl.ln2_g(), vl.ln2_b(), xn);
#pragma unroll
    for (int i = 0; i < OT; ++i)
      if (owns(i)) x[i] += bias_tile(vec + vl.b2(), wave + WV * i, hi);
    for (int c0 = 0, par = 0; c0 < NC; c0 += WV, par ^= 1) {
      const int c = c0 + wave;
      if (c < NC) {
        f32x16 ah = product(bias_tile(vec + vl.b1(), c, hi), sg.w1(c), xn, false);
        settle(ah);
#pragma unroll
        for (int g = 0; g < 2; ++g) {
          f16x8 y;     // ah holds x / kFfnScale; to fp16 toward zero, then the packed activation
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const f16x2 y2 = __builtin_bit_cast(f16x2, __builtin_amdgcn_cvt_pkrtz(ah[8 * g + 2 * e], ah[8 * g + 2 * e + 1]));
            y[2 * e] = y2[0]; y[2 * e + 1] = y2[1];
          }
          hid[par][wave][g][lane] = RELU ? __builtin_elementwise_max(y, (f16x8)((_Float16)0.f)) : gelu_quarter_h8(y);
        }
      }
      __syncthreads();          // (the other parity was last read ahead of the barrier before)
#pragma unroll
      for (int i = 0; i < OT; ++i) {
        if (!owns(i)) continue;
#pragma unroll
        for (int k = 0; k < WV; ++k) {
          if (c0 + k >= NC) break;
#pragma unroll
          for (int g = 0; g < 2; ++g) x[i] = E::mma_h(frag(sg.w2(c0 + k), 2 * (wave + WV * i) + g), hid[par][k][g][lane], x[i]);
        }
      }
    }
#pragma unroll
    for (int i = 0; i < OT; ++i) settle(x[i]);
    wl += (size_t)sg.block() * D * 64;
    sg.attn = false;
  }

  // ------------------------------------------------------------------ epilogue
#pragma unroll
  for (int i = 0; i < OT; ++i) {
    const f32x16 one[1] = {x[i]};
    if (p.X_out && inrange && owns(i)) store_rows<T, 1>(one, p.X_out, p.X_f32, out_off + 32 * (wave + WV * i), valid, hi);
  }
  if (!STACK && !SCORE) return;
  if (p.logits) {
    // logit = <head_w, flatten(global rows)> + head_b: each wave sums over its own feature tiles
    const int a = STACK ? 32 * ts + j : (32 * tile + j) % p.m, width = STACK ? 32 : p.m;      // row inside the head's m rows; lanes per logit
    float part = 0.f;
    if (valid && a < p.m) {
#pragma unroll
      for (int i = 0; i < OT; ++i) {
        if (!owns(i)) continue;
        const f32x16 hw = bias_tile(p.head + (size_t)a * D, wave + WV * i, hi);
#pragma unroll
        for (int r = 0; r < 16; ++r) part += x[i][r] * hw[r];
      }
    }
    part = row_sums(part, 0.f).x;
    for (int sft = 1; sft < width; sft <<= 1) part += __shfl_xor(part, sft, 64);
    part += p.head[(size_t)p.m * D];
    if (STACK) {
      if (tid == 0) p.logits[usr] = part;
    } else {
      const int cand = (32 * tile + j) / p.m;
      if (wave == 0 && hi == 0 && (j % p.m) == 0 && cand < p.C) p.logits[(size_t)usr * p.C + cand] = part;
    }
  }
}

// Host-side launcher, one definition per (D, DH) instantiation file.  pair: the scoring stream is in the pair layout.
template <int D, int DH>
int launch_quad(int mode, int win, bool pair, const BlockParams& p, dim3 grid, hipStream_t stream);

#define LONGER_QUAD_LAUNCH(D, DH, MODEV, WV, LAY) \
  do {                                                                                                \
    if (p.act == 1) hipLaunchKernelGGL((quad_kernel<D, DH, MODEV, WV, LAY, true>), grid, dim3(64 * quad_waves(D) * quad_tiles(MODEV)), 0, stream, p); \
    else hipLaunchKernelGGL((quad_kernel<D, DH, MODEV, WV, LAY, false>), grid, dim3(64 * quad_waves(D) * quad_tiles(MODEV)), 0, stream, p); \
  } while (0)

template <int D, int DH, int LAY>
static void launch_quad_score(int win, const BlockParams& p, dim3 grid, hipStream_t stream) {
  if (win == 4) LONGER_QUAD_LAUNCH(D, DH, MODE_SCORE, 4, LAY);
  else if (win == 8) LONGER_QUAD_LAUNCH(D, DH, MODE_SCORE, 8, LAY);
  else LONGER_QUAD_LAUNCH(D, DH, MODE_SCORE, 16, LAY);
}

// (width 64 streams the plain layouts, width 128 the pair layouts unless the pair kernels are switched off)
template <int D, int DH>
static int launch_quad_stack(bool pair, const BlockParams& p, dim3 grid, hipStream_t stream) {
  if constexpr (D == 64) { if (!pair) { LONGER_QUAD_LAUNCH(D, DH, MODE_STACK, 16, QUAD_PLAIN); return 0; } }
  if constexpr (D == 128) { if (pair) { LONGER_QUAD_LAUNCH(D, DH, MODE_STACK, 16, QUAD_PAIR); return 0; } }
  return -1;
}

#define LONGER_QUAD_INSTANTIATE(D, DH)                                                                \
  template <>                                                                                         \
  int launch_quad<D, DH>(int mode, int win, bool pair, const BlockParams& p, dim3 grid, hipStream_t stream) { \
    if (mode == MODE_ATTN) LONGER_QUAD_LAUNCH(D, DH, MODE_ATTN, 16, QUAD_PLAIN);                      \
    else if (mode == MODE_STACK) { if (launch_quad_stack<D, DH>(pair, p, grid, stream)) return -1; }  \
    else if (pair) { if constexpr (D >= 128) launch_quad_score<D, DH, QUAD_PAIR>(win, p, grid, stream); else return -1; } \
    else launch_quad_score<D, DH, QUAD_PLAIN>(win, p, grid, stream);                                  \
    return hipGetLastError() == hipSuccess ? 0 : -3;                                                  \
  }

}  // namespace longer
