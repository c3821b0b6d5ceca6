// The transformer-block kernel for launches with few tiles: a 32-row tile given to four waves, one per SIMD of a
// compute unit, or eight at width 256 (bf16).
//
//   MODE_SCORE  candidate scoring of the KV-cache serving path (Section 3.6.3), all layers;
//   MODE_ATTN   query side of one layer over stored K/V fragments (the cache build's sequence rows; a small batch's reduced stack
//               layer by layer), and with kv_w the next layer's K and V of the result, which a launch of its own took 16 us for
//               (two tiles a user, 16 users, width 256);
//   MODE_STACK  the whole reduced stack of a user with at most two tiles (m + k <= 64) in one workgroup of eight waves.
//
// Why.  A request scores a hundred candidates (25 tiles), a cache build runs two tiles per user: a handful of
// workgroups on 256 compute units, whose time is one tile's chain of dependent products.  Here feature tile t of the
// rows, of every product's result and its attention heads belong to wave t % 4 (t % 8), and the FFN's hidden chunks are dealt
// out the same way, so the chain is a quarter (an eighth) as long; operand groups change hands through LDS.  The waves
// share no weights, so each fetches its fragments from L2 itself, from the same packed streams as the other kernels
// (their segments are found by index).  With many tiles the streams' traffic and the idle matrix pipes cost more than the
// shorter chain gains: the rule is at quad_pays in longer_api.hip.
//
// What bounds it: at width 128 the vector work of the attention (a third of the chain) and the two products of a hidden
// chunk; at width 256 the weights' way into the compute unit, 64 bytes a cycle (half of a layer's time).  The waves never wait for
// a weight fragment that they could have asked for earlier: with each product's fragments requested when it began, four
// layers of scoring took 53 us for 25 tiles at width 128 and 255 us for 128 tiles over 20 key tiles at width 256; requested
// behind the fragments of the product before, and four key tiles ahead, 41 and 105 us (92 with the cheaper key tile step).  (Bringing a block's stream into the
// die's L2 one block ahead, each workgroup its share, cost more than it gave: 51 and 200 us.)
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
    return ffn() + (ffn_skewed(2, D) ? min(3 + 2 * c, 2 * NC) : 2 * c + 1);
  }
  __device__ __forceinline__ int block() const { return 2 + (attn ? 2 : 4) * NT + 2 * NC; }
};

template <int D, int DH, int MODE, int W, int LAYOUT, bool RELU>
__global__ void __launch_bounds__(64 * quad_waves(D) * quad_tiles(MODE), quad_waves(D) * quad_tiles(MODE) == 4 ? 2 : 1) quad_kernel(const BlockParams p) {
  using T = __bf16;
  using E = ET<T>;
  using grp = typename E::grp;
  using hgrp = typename E::hgrp;
  constexpr int WV = quad_waves(D), TS = quad_tiles(MODE), kThr = 64 * WV * TS;
  constexpr int NT = D / 32, NG = D / 16, HPT = 32 / DH, GPH = DH / 16;
  constexpr bool SCORE = MODE == MODE_SCORE, STACK = MODE == MODE_STACK;
  static_assert(SCORE || STACK || MODE == MODE_ATTN, "quad kernel modes");
  static_assert(NT <= WV, "a wave owns at most one feature tile");
  __shared__ grp ops_[TS][2][NG][64];                // per tile, [normalised rows, attention output][group][lane]: operand of the next products
  __shared__ hgrp hid_[TS][2][WV][2][64];            // activated hidden chunks: [parity][wave][group][lane]
  __shared__ float2 sums_[TS][2][WV][64];            // row sums: [first, second LayerNorm][wave][lane]
  __shared__ grp kvl[STACK ? TS : 1][STACK ? NT : 1][2][2][64];      // self layers: [key tile][feature tile][K, V][group][lane]
  __shared__ f32x4 vecl[D * 4];                      // the block's fp32 vectors (at most one segment)
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int tid = threadIdx.x, lane = tid & 63, j = lane & 31, hi = lane >> 5;
  const int ts = TS == 1 ? 0 : wv / WV, wave = TS == 1 ? wv : wv % WV;     // tile of the workgroup, wave of the tile
  auto& ops = ops_[ts];
  auto& hid = hid_[ts];
  auto& sums = sums_[ts];
  const int NC = p.FF / 32;
  QuadSegs<LAYOUT, D> sg = {NC, !SCORE};               // (the stack's first block is the cross layer's attention half)
  const bool own = NT >= WV || wave < NT;              // the wave has a feature tile: ft
  const int ft = NT >= WV ? wave : wave % NT;          // (width 64: waves 2 and 3 share in the hidden chunks alone; their rows go nowhere)

  // ------------------------------------------------------------------ rows
  bool valid, inrange;
  int usr, Tu, tile;
  long long out_off;
  uint32_t tilebits = 0;
  KeyRanges kr = {}, skr = {};                         // visible keys among the stored ones; in the stack's self layers
  int kthi = 0;                                        // tiles of the stored keys
  const int widx = W == 16 ? 0 : j / (2 * W);
  uint32_t wmask[16 / W];
#pragma unroll
  for (int w = 0; w < 16 / W; ++w) { wmask[w] = widx == w ? 0xffffffffu : 0u; asm("" : "+v"(wmask[w])); }
  f32x16 x;
  auto load_own = [&](const void* base, int f32, long long off) {
    f32x16 one[1];
    load_rows<T, 1>(one, base, f32, off + 32 * wave, valid && own, hi);
    x = one[0];
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
    if (glob) { kr.lo1 = p.gmask_causal ? a : 0; kr.hi1 = p.KG; }
    kr.lo2 = p.KG + s0;
    kr.hi2 = p.KG + (glob ? (p.key_self ? p.k : tu) : (p.key_self ? i : tok) + 1);
    kr.settle_for(valid);
    kthi = (p.KG + (p.key_self ? p.k : tu) + 31) / 32;
    if (STACK) {      // keys of a self-causal layer: the user's own rows, key index = row index
      if (glob) { skr.lo1 = p.gmask_causal ? a : 0; skr.hi1 = p.m; }
      skr.lo2 = p.m + i0; skr.hi2 = p.m + (glob ? p.k : i + 1);
      skr.settle_for(valid);
    }
  }

  const char* wl = p.wbase;                            // the current block's stream
  const VecLayout vl{D, p.FF};
  const float* vec = reinterpret_cast<const float*>(vecl);
  // A product's weight fragments are requested while the product ahead of it runs: each takes the registers of the fragment
  // that was just used.  (The compiler moves no load across a barrier.)  Order of a wave's products: Q (K, V) of its feature
  // tile, its tile of the output projection, then W1 of a hidden chunk and its tile's rows of W2 for all waves' chunks in turn.
  constexpr int NF = NG > 2 * WV ? NG : 2 * WV;
  constexpr bool HOLD = D <= 128;                      // (width 256: no registers for them through the attention)
  grp fr[NF];
  typedef __attribute__((address_space(1))) const char gchar;
  typedef __attribute__((address_space(1))) const grp ggrp;
  unsigned lane16 = (unsigned)lane * 16u;
  // what is worked out from these is worked out again: kept through the layers it would cost the registers of the fragments
  auto afresh = [&] {
    asm volatile("" : "+v"(tid));
    lane = tid & 63; j = lane & 31; hi = lane >> 5; lane16 = (unsigned)lane * 16u;
  };
  auto segment = [&](const char* w, int seg) -> gchar* {       // (wave-uniform: a scalar base, the lane's part an offset)
    gchar* q = (gchar*)(w + (size_t)seg * (NG * 1024));
    asm("" : "+s"(q));
    return q;
  };
  auto request = [&](gchar* q) {
#pragma unroll
    for (int s = 0; s < NG; ++s) fr[s] = *(ggrp*)(q + (lane16 + (unsigned)s * 1024u));
  };
  // (products and loads stay in this order: hoisted loads would need a second set of registers)
  auto in_order = [] { __builtin_amdgcn_sched_barrier(0x486); };
  // acc + (a segment's 32 result features) b; swapped: result with lane = feature; the fragments of segment `next` follow
  auto product = [&](f32x16 acc, const grp (&b)[NG], bool swapped, bool more, gchar* next) -> f32x16 {
#pragma unroll
    for (int s = 0; s < NG; ++s) {
      acc = swapped ? E::mma(b[s], fr[s], acc) : E::mma(fr[s], b[s], acc);
      if (more) fr[s] = *(ggrp*)(next + (lane16 + (unsigned)s * 1024u));
      __builtin_amdgcn_sched_barrier(0);
    }
    return acc;
  };
  constexpr int VQ = (D * 4 + kThr - 1) / kThr;        // the block's vectors: this thread's share, on its way to LDS
  f32x4 vq[VQ];
  auto request_vec = [&](const char* w) {
    const int n = (9 * D + p.FF) / 4;
#pragma unroll
    for (int i = 0; i < VQ; ++i) { const int c = tid + kThr * i; vq[i] = reinterpret_cast<const f32x4*>(w)[c < n ? c : 0]; }
  };
  request_vec(wl);
  request(segment(wl, sg.q(ft)));
  // row sums of all waves (two numbers per row)
  auto row_sums = [&](int which, float a, float b) -> float2 {
    sums[which][wave][lane] = make_float2(sum_halves(a), sum_halves(b));
    __syncthreads();
    float2 r = make_float2(0.f, 0.f);
#pragma unroll
    for (int w = 0; w < WV; ++w) { const float2 q = sums[which][w][lane]; r.x += q.x; r.y += q.y; }
    return r;
  };
  auto take = [&](int which, grp (&b)[NG]) {
#pragma unroll
    for (int g = 0; g < NG; ++g) b[g] = ops[which][g][lane];
  };
  // LayerNorm of the rows as the next products' operand, in every wave
  auto normalise = [&](int which, int og, int ob, grp (&b)[NG]) {
    float s = 0.f, q = 0.f;
    if (own) {
#pragma unroll
      for (int r = 0; r < 16; ++r) { s += x[r]; q = fmaf(x[r], x[r], q); }
    }
    const float2 t = row_sums(which, s, q);
    const float mean = t.x * (1.0f / D), var = fmaxf(t.y * (1.0f / D) - mean * mean, 0.f);
    const float rstd = __builtin_amdgcn_rsqf(var + p.eps), shift = -mean * rstd;
    if (own) {
      const f32x16 g = bias_tile(vec + og, wave, hi), c = bias_tile(vec + ob, wave, hi);
      f32x16 y;
#pragma unroll
      for (int r = 0; r < 16; ++r) y[r] = fmaf(fmaf(x[r], rstd, shift), g[r], c[r]);
#pragma unroll
      for (int g2 = 0; g2 < 2; ++g2) ops[0][2 * wave + g2][lane] = E::pack(y, g2);
    }
    __syncthreads();
    take(0, b);
  };

  // Areas of LDS are written once a layer and each write has a barrier of that layer between itself and the last reader:
  // `vecl` the last hidden chunk's, `sums` and `ops` the other LayerNorm's and the attention output's.
  for (int layer = 0; layer < p.n_layers; ++layer) {
    const bool selfl = STACK && layer > 0;             // K and V made here, handed to the user's other tile through LDS
    const bool last = layer + 1 == p.n_layers;
    const bool project = MODE == MODE_ATTN && p.kv_w;  // (one layer)
    afresh();
    const char* wnext = wl + (size_t)sg.block() * D * 64;
#pragma unroll
    for (int i = 0; i < VQ; ++i) { const int c = tid + kThr * i; if (c < D * 4) vecl[c] = vq[i]; }
    {
      grp xn[NG];
      normalise(0, vl.ln1_g(), vl.ln1_b(), xn);
      grp oo[2];
      f32x16 aq, ak, av;
      if (own) {
        if (SCORE || selfl) {
          aq = product(bias_tile(vec + vl.bq(), wave, hi), xn, false, true, segment(wl, sg.k(wave)));
          ak = product(splat16(0.f), xn, false, true, segment(wl, sg.v(wave)));   // no b_K, no b_V: see block_kernel.h
          av = product(splat16(0.f), xn, true, HOLD, segment(wl, sg.o(wave)));
        } else {
          aq = product(bias_tile(vec + vl.bq(), wave, hi), xn, false, HOLD, segment(wl, sg.o(wave)));
        }
        if (selfl) {
          settle(ak); settle(av);
#pragma unroll
          for (int g = 0; g < 2; ++g) { kvl[ts][wave][0][g][lane] = E::pack(ak, g); kvl[ts][wave][1][g][lane] = E::pack(av, g); }
        }
      }
      if (selfl) __syncthreads();
      if (own) {
        __builtin_amdgcn_sched_barrier(0);
        settle(aq);
        aq *= p.scale_l2e;
        grp qop[2];
#pragma unroll
        for (int g = 0; g < 2; ++g) qop[g] = E::pack(aq, g);
        float mrun[HPT], lrun[HPT];
        f32x16 acc[HPT];
#pragma unroll
        for (int hh = 0; hh < HPT; ++hh) { mrun[hh] = kNegBig; lrun[hh] = 0.f; acc[hh] = splat16(0.f); }
        // stored K/V fragments (wave-uniform user, scalar loop control); KD key tiles on their way
        constexpr int KD = STACK ? 2 : 4;
        const char* kb; const char* vb; int nkt;
        const int tuu = __builtin_amdgcn_readfirstlane(Tu);
        if (selfl) {
          kb = vb = nullptr; nkt = (p.m + p.k + 31) / 32;
        } else if (!SCORE) {
          kb = p.kst + (size_t)usr * p.kv_ustride; vb = p.vst + (size_t)usr * p.kv_ustride;
          nkt = __builtin_amdgcn_readfirstlane(kthi);
        } else {
          if (layer == 0) {
            kb = p.cache + (size_t)usr * p.c0_ustride; vb = kb + p.c0_voff;
            nkt = min(p.kt0, (tuu + 31) / 32); kr = {0, 0, 0, tuu};
          } else {
            kb = p.cache + p.c1_off + (size_t)(layer - 1) * p.c1_lstride + (size_t)usr * p.c1_ustride;
            vb = kb + p.c1_voff;
            nkt = tuu > 0 ? p.kt1 : 0; kr = {0, 0, first_slot(p.k, tuu, p.q_learn), p.k};
          }
          kr.settle_for(valid);
        }
        if (nkt == 0) kb = vb = wl;                    // (readable: requests are made without asking, so that no value lives on through a branch)
        grp kn[KD][2], vn[KD][2];
        auto fetch = [&](int kt, int b) {
          if (selfl) {
#pragma unroll
            for (int g = 0; g < 2; ++g) { kn[b][g] = kvl[STACK ? kt : 0][STACK ? wave : 0][0][g][lane]; vn[b][g] = kvl[STACK ? kt : 0][STACK ? wave : 0][1][g][lane]; }
            return;
          }
          const size_t fo = ((size_t)(kt * NT + wave) * 2) * 1024 + lane * 16;
#pragma unroll
          for (int g = 0; g < 2; ++g) {
            kn[b][g] = *reinterpret_cast<const grp*>(kb + fo + g * 1024);
            vn[b][g] = *reinterpret_cast<const grp*>(vb + fo + g * 1024);
          }
        };
#pragma unroll
        for (int b = 0; b < KD; ++b) fetch(min(b, max(nkt - 1, 0)), b);
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
        auto key_tile = [&](int kt, int b) __attribute__((always_inline)) {
          key_tile_step<HPT, GPH, true>(selfl ? skr : kr, kt, kn[b], vn[b], qop, hi, mrun, lrun, acc);
          if (kt + KD < nkt) fetch(kt + KD, b);
        };
        for (int kt = 0; kt < nkt; kt += KD) {
#pragma unroll
          for (int b = 0; b < KD; ++b)
            if (kt + b < nkt) key_tile(kt + b, b);
        }
        f32x16 o;
        float inv[HPT];
#pragma unroll
        for (int hh = 0; hh < HPT; ++hh) { settle(acc[hh]); inv[hh] = lrun[hh] > 0.f ? __builtin_amdgcn_rcpf(lrun[hh]) : 0.f; }
#pragma unroll
        for (int r = 0; r < 16; ++r) o[r] = acc[HPT == 1 ? 0 : r / 8][r] * inv[HPT == 1 ? 0 : r / 8];
#pragma unroll
        for (int g = 0; g < 2; ++g) ops[1][2 * wave + g][lane] = E::pack(o, g);
      }
      if (!HOLD || !own) request(segment(wl, sg.o(ft)));
      __syncthreads();
      take(1, xn);
      x += bias_tile(vec + vl.bo(), ft, hi);
      x = product(x, xn, false, true, segment(wl, sg.w1(min(wave, NC - 1))));
      settle(x);
    }
    grp xn[NG];
    afresh();
    request_vec(project ? p.kv_w : last ? wl : wnext);
    normalise(1, vl.ln2_g(), vl.ln2_b(), xn);
    x += bias_tile(vec + vl.b2(), ft, hi);
    for (int c0 = 0, par = 0; c0 < NC; c0 += WV, par ^= 1) {
      const int c = min(c0 + wave, NC - 1);            // (a wave without a chunk goes through another's and hands in zeros)
      auto request_w2 = [&](int s) {                   // fragment s % 2 of chunk c0 + s / 2 for this wave's tile
        fr[s] = *(ggrp*)(segment(wl + 2048 * ft, sg.w2(min(c0 + s / 2, NC - 1))) + (lane16 + (unsigned)(s & 1) * 1024u));
      };
#pragma unroll
      for (int s = NG; s < 2 * WV; ++s) request_w2(s);
      f32x16 ah = bias_tile(vec + vl.b1(), c, hi);
#pragma unroll
      for (int s = 0; s < NG; ++s) {
        ah = E::mma(fr[s], xn[s], ah);
        request_w2(s);
        __builtin_amdgcn_sched_barrier(0);
      }
      settle(ah);
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        f16x8 y;     // ah holds x / kFfnScale; to fp16 toward zero, then the packed activation
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const f16x2 y2 = __builtin_bit_cast(f16x2, __builtin_amdgcn_cvt_pkrtz(ah[8 * g + 2 * e], ah[8 * g + 2 * e + 1]));
          y[2 * e] = y2[0]; y[2 * e + 1] = y2[1];
        }
        y = RELU ? __builtin_elementwise_max(y, (f16x8)((_Float16)0.f)) : gelu_quarter_h8(y);
        if (c0 + wave >= NC) y = (f16x8)((_Float16)0.f);
        hid[par][wave][g][lane] = y;
      }
      // what follows on these chunks' second product: the next hidden chunk, or the next block's first
      gchar* next = segment(wl, sg.w1(min(c0 + WV + wave, NC - 1)));
      if (c0 + WV >= NC && !last) next = segment(wnext, QuadSegs<LAYOUT, D>{NC, false}.q(ft));
      if (c0 + WV >= NC && project) next = segment(p.kv_w, 1 + 2 * ft);
      __syncthreads();          // (the other parity was last read ahead of the barrier before)
#pragma unroll
      for (int s = 0; s < 2 * WV; ++s) {
        x = E::mma_h(fr[s], hid[par][s / 2][s & 1][lane], x);
        if (s < NG) fr[s] = *(ggrp*)(next + (lane16 + (unsigned)s * 1024u));
        in_order();
      }
    }
    settle(x);
    wl = wnext;
    sg.attn = false;
  }

  // ------------------------------------------------------------------ epilogue
  const f32x16 one[1] = {x};
  if (p.X_out && inrange && own) store_rows<T, 1>(one, p.X_out, p.X_f32, out_off + 32 * wave, valid, hi);
  if (MODE == MODE_ATTN && p.kv_w) {      // split layout: [vectors][K V of feature tile 0][K V of feature tile 1] ...
    afresh();
#pragma unroll
    for (int i = 0; i < VQ; ++i) { const int c = tid + kThr * i; if (c < D * 4) vecl[c] = vq[i]; }
#pragma unroll
    for (int r = 0; r < 16; ++r) x[r] = valid ? x[r] : 0.f;      // (K and V of rows that do not exist: of zeros, nobody sees them)
    grp xn[NG];
    normalise(0, vl.ln1_g(), vl.ln1_b(), xn);
    const f32x16 ak = product(splat16(0.f), xn, false, true, segment(p.kv_w, 2 + 2 * ft));
    f32x16 av = product(splat16(0.f), xn, true, false, nullptr);
    settle(av);
    if (own) {
      const size_t fo = (size_t)usr * p.kv_w_ustride + ((size_t)(tile * NT + wave) * 2) * 1024 + lane16;
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        *reinterpret_cast<grp*>(p.kv_k + fo + g * 1024) = E::pack(ak, g);
        *reinterpret_cast<grp*>(p.kv_v + fo + g * 1024) = E::pack(av, g);
      }
    }
  }
  if (p.logits && (MODE != MODE_ATTN || p.q0 + tile == 0)) {       // (the global rows, at most 32, are all in a user's first tile)
    // logit = <head_w, flatten(global rows)> + head_b: each wave sums over its own feature tiles
    const int a = SCORE ? (32 * tile + j) % p.m : 32 * tile + j, width = SCORE ? p.m : 32;    // row inside the head's m rows; lanes per logit
    float part = 0.f;
    if (valid && a < p.m && own) {
      const f32x16 hw = bias_tile(p.head + (size_t)a * D, wave, hi);
#pragma unroll
      for (int r = 0; r < 16; ++r) part += x[r] * hw[r];
    }
    part = row_sums(0, part, 0.f).x;
    for (int sft = 1; sft < width; sft <<= 1) part += __shfl_xor(part, sft, 64);
    part += p.head[(size_t)p.m * D];
    if (!SCORE) {
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

// (width 64 streams the plain layouts, widths 128 and, in scoring, 256 the pair layouts)
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
    else if (pair != (D >= 128)) return -1;                                                           \
    else launch_quad_score<D, DH, D >= 128 ? QUAD_PAIR : QUAD_PLAIN>(win, p, grid, stream);           \
    return hipGetLastError() == hipSuccess ? 0 : -3;                                                  \
  }

}  // namespace longer
