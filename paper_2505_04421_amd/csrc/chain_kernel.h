// The transformer-block kernel for launches with few tiles, bf16, heads of 16 features, d = 64 / 128: a wave per head.  The modes are those
// of quad_kernel.h, whose kernels run the other shapes; packed streams and results are the same (sums inside a product and a softmax in
// the same order, too).
//
//   MODE_SCORE  candidate scoring (Section 3.6.3), all layers;
//   MODE_ATTN   query side of one layer over stored K/V fragments, with kv_w the next layer's K and V of the result;
//   MODE_STACK  the whole reduced stack of a user with at most two tiles (m + k <= 64), d = 64.
//
// What bounds such a launch is one tile's chain of dependent steps: the softmax over the stored keys (vector work; a wave alone on its SIMD
// issues a vector instruction every five cycles, two of them one every two and a half), the weights' and keys' way into the compute
// unit (64 bytes a cycle: 7 to 9 of the 21 thousand cycles of a scored layer of width 128) and LayerNorm's exchanges.  Here waves t and t + NT share
// feature tile t of the rows: the first keeps the rows (fp32) and makes Q, the output projection and the second FFN product, the
// second makes K and V; each takes one head, and both a hidden chunk of a round.  The FFN's weights are on their way during the output
// projection and LayerNorm, the next layer's first ones during the FFN, the first key tiles during LayerNorm.  Two heads a wave (quad_kernel.h) /
// a wave per head, microseconds: 1, 25, 128, 256 tiles of candidates at width 128 (four layers) 41.6 / 37.5, 41.9 / 37.9, 43.3 / 39.5, 46.6 /
// 42.8, at width 64 (three layers) 1, 256, 512 tiles 20.8 / 17.2, 22.5 / 18.6, 29.1 / 23.6; passes of 1, 128, 256 users of width 64 and
// 36 rows 39.6 / 34.6, 48.1 / 42.5, 59.6 / 53.9, of 61 users of width 128 and 108 rows 84.2 / 81.4.
#pragma once
#include "quad_kernel.h"

namespace longer {

constexpr int chain_waves(int d) { return d / 16; }       // waves per tile: one per head

// KEYS: the stack makes its cross layer's K and V (asked at run time instead, the stack that finds them took 26.0 instead of 25.3 us: 13 users of 5745 tokens)
template <int D, int MODE, int W, int LAYOUT, bool RELU, bool KEYS = false>
__global__ void __launch_bounds__(64 * chain_waves(D) * quad_tiles(MODE), chain_waves(D) * quad_tiles(MODE) == 4 ? 2 : 1) chain_kernel(const BlockParams p) {
  using T = __bf16;
  using E = ET<T>;
  using grp = typename E::grp;
  using hgrp = typename E::hgrp;
  constexpr int WV = chain_waves(D), TS = quad_tiles(MODE), kThr = 64 * WV * TS;
  constexpr int NT = D / 32, NG = D / 16;
  constexpr bool SCORE = MODE == MODE_SCORE, STACK = MODE == MODE_STACK;
  static_assert(SCORE || STACK || MODE == MODE_ATTN, "chain kernel modes");
  __shared__ grp ops_[TS][2][NG][64];                // per tile, [normalised rows, attention output][group][lane]: operand of the next products
  __shared__ hgrp hid_[TS][2][WV][2][64];            // activated hidden chunks: [parity][wave][group][lane]
  __shared__ float2 sums_[TS][2][NT][64];            // row sums: [first, second LayerNorm][feature tile][lane]
  __shared__ grp qx_[TS][NT][2][64];                 // Q of a feature tile: [head][lane]
  __shared__ grp kvl[TS][NT][2][2][64];              // K and V of the workgroup's own rows: [tile][feature tile][K, V][group][lane]
  __shared__ f32x4 vecl[D * 4];                      // the block's fp32 vectors (at most one segment)
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int tid = threadIdx.x, lane = tid & 63, j = lane & 31, hi = lane >> 5;
  const int ts = TS == 1 ? 0 : wv / WV, wave = TS == 1 ? wv : wv % WV;     // tile of the workgroup, wave of the tile
  const int ft = wave % NT;                          // feature tile
  auto& ops = ops_[ts];
  auto& hid = hid_[ts];
  auto& sums = sums_[ts];
  auto& qx = qx_[ts];
  const int NC = p.FF / 32;
  QuadSegs<LAYOUT, D> sg = {NC, !SCORE};               // (the stack's first block is the cross layer's attention half)

  // ------------------------------------------------------------------ rows
  bool valid, inrange;
  int usr, Tu, tile;
  long long out_off;
  uint32_t tilebits = 0;
  KeyRanges kr = {}, skr = {};                         // visible keys among the stored ones; in the stack's self layers
  int kthi = 0;                                        // tiles of the stored keys
  f32x16 x;
  auto load_own = [&](const void* base, int f32, long long off) {      // (every wave: the second of a pair does not keep them)
    f32x16 one[1];
    load_rows<T, 1>(one, base, f32, off + 32 * ft, valid, hi);
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
    tilebits = ((range_bits(gbase + (p.gmask_causal ? gi : 0), gbase + p.m, 0) & vb) >> (4 * hi)) >> (W == 16 ? 0 : 2 * W * (j / (2 * W)));
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

  // The two waves of a feature tile go through code of their own (and the same barriers): with requests of one of them under a
  // condition the compiler, which has to know how many loads are behind the one it waits for, waits for the other's as well.
  auto run = [&](auto keeper_) __attribute__((always_inline)) {
  constexpr bool keeper = decltype(keeper_)::value;    // the wave that holds the tile's rows
  constexpr int head = keeper ? 0 : 1;                 // which of the feature tile's two heads
  const char* wl = p.wbase;                            // the current block's stream
  const VecLayout vl{D, p.FF};
  const float* vec = reinterpret_cast<const float*>(vecl);
  // weight fragments: Q (the second wave of a pair: K), later the wave's hidden chunk; the output projection (V); W2 for the
  // wave's feature tile and a round's chunks
  grp fr[NG], f1[NG], f2[2 * WV];
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
  auto request = [&](grp (&f)[NG], gchar* q) {
#pragma unroll
    for (int s = 0; s < NG; ++s) f[s] = *(ggrp*)(q + (lane16 + (unsigned)s * 1024u));
  };
  auto request_w2 = [&](int c0, int s) {                       // fragment s % 2 of chunk c0 + s / 2
    f2[s] = *(ggrp*)(segment(wl + 2048 * ft, sg.w2(min(c0 + s / 2, NC - 1))) + (lane16 + (unsigned)(s & 1) * 1024u));
  };
  // acc + (a segment's 32 result features) b; swapped: result with lane = feature; the fragments of segment `next` follow
  auto product = [&](f32x16 acc, grp (&f)[NG], const grp (&b)[NG], bool swapped, bool more, gchar* next) -> f32x16 {
#pragma unroll
    for (int s = 0; s < NG; ++s) {
      acc = swapped ? E::mma(b[s], f[s], acc) : E::mma(f[s], b[s], acc);
      if (more) f[s] = *(ggrp*)(next + (lane16 + (unsigned)s * 1024u));
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
  auto store_vec = [&] {
#pragma unroll
    for (int i = 0; i < VQ; ++i) { const int c = tid + kThr * i; if (c < D * 4) vecl[c] = vq[i]; }
  };
  // row sums of the whole tile (two numbers per row) for the waves that hold rows; every wave is behind a barrier afterwards
  auto row_sums = [&](int which, float a, float b) -> float2 {
    if (keeper) sums[which][ft][lane] = make_float2(sum_halves(a), sum_halves(b));
    __syncthreads();
    float2 r = make_float2(0.f, 0.f);
    if (keeper) {
#pragma unroll
      for (int w = 0; w < NT; ++w) { const float2 q = sums[which][w][lane]; r.x += q.x; r.y += q.y; }
    }
    return r;
  };
  auto take = [&](int which, grp (&b)[NG]) {
#pragma unroll
    for (int g = 0; g < NG; ++g) b[g] = ops[which][g][lane];
  };
  // LayerNorm of the rows as the next products' operand, in every wave
  auto normalise = [&](int which, int og, int ob, grp (&b)[NG]) {
    float s = 0.f, q = 0.f;
    if (keeper) {
#pragma unroll
      for (int r = 0; r < 16; ++r) { s += x[r]; q = fmaf(x[r], x[r], q); }
    }
    const float2 t = row_sums(which, s, q);
    if (keeper) {
      const f32x16 g = bias_tile(vec + og, ft, hi), c = bias_tile(vec + ob, ft, hi);
      const float mean = t.x * (1.0f / D), var = fmaxf(t.y * (1.0f / D) - mean * mean, 0.f);
      const float rstd = __builtin_amdgcn_rsqf(var + p.eps), shift = -mean * rstd;
      f32x16 y;
#pragma unroll
      for (int r = 0; r < 16; ++r) y[r] = fmaf(fmaf(x[r], rstd, shift), g[r], c[r]);
#pragma unroll
      for (int g2 = 0; g2 < 2; ++g2) ops[0][2 * ft + g2][lane] = E::pack(y, g2);
    }
    __syncthreads();
    take(0, b);
  };

  request_vec(KEYS ? p.kv_w : wl);
  // the wave's first product of a block: Q, or (the second wave of a pair, where K and V are made here) K
  request(fr, segment(wl, keeper || !SCORE ? sg.q(ft) : sg.k(ft)));
  // The stack's cross layer finds its K and V in memory.  A short user's (KEYS; kv_w: the cross block's K / V stream, kv_k: the merged tokens) are made here, two
  // key tiles at a time, a wave of a pair each; they go the same way, but no further than the workgroup that wrote them.
  if constexpr (KEYS) {
    const f32x16 queries = x;
    request(f1, segment(p.kv_w, keeper ? 1 + 2 * ft : 2 + 2 * ft));
    auto key_rows = [&](int kt) {
      const int a = 32 * kt + j;
      const bool glob = a < p.m, ok = glob || a - p.m < Tu;
      f32x16 one[1];
      load_rows<T, 1>(one, glob ? p.src0.p : (const void*)p.kv_k, glob ? p.src0.f32 : 1,
                      (glob ? p.src0.ustride * usr + (long long)a * D : (long long)p.kv_w_ustride * usr + (long long)(a - p.m) * D) + 32 * ft, ok, hi);
      return one[0];
    };
    f32x16 ahead = key_rows(ts);
    for (int k0 = 0; k0 < kthi; k0 += TS) {            // (the same number of times for either tile: barriers)
      const int kt = k0 + ts;
      x = ahead;
      ahead = key_rows(min(kt + TS, kthi - 1));
      if (k0 == 0) { store_vec(); request_vec(wl); }
      grp xn[NG];
      normalise(0, vl.ln1_g(), vl.ln1_b(), xn);
      f32x16 o = keeper ? product(splat16(0.f), f1, xn, false, false, nullptr) : product(splat16(0.f), f1, xn, true, false, nullptr);
      settle(o);
      if (kt < kthi) {
        char* dst = (keeper ? p.kst : p.vst) + (size_t)usr * p.kv_ustride + ((size_t)(kt * NT + ft) * 2) * 1024 + lane16;
#pragma unroll
        for (int g = 0; g < 2; ++g) *reinterpret_cast<grp*>(dst + g * 1024) = E::pack(o, g);
      }
    }
    x = queries;
    wait_vmcnt<0>();                                   // (written, for the workgroup's other waves)
    __syncthreads();
  }

  // Areas of LDS are written once a layer (hid: once in two rounds) and each write has a barrier between itself and the last
  // reader: `vecl` the last round's, `sums` and `ops` the other LayerNorm's and the attention output's, `qx` and `kvl` the output
  // projection's, `hid` the next round's (which its readers reach when they have read).
  for (int layer = 0; layer < p.n_layers; ++layer) {
    const bool selfl = STACK && layer > 0;             // K and V made here, handed to the user's other tile through LDS
    const bool last = layer + 1 == p.n_layers;
    const bool project = MODE == MODE_ATTN && p.kv_w;  // (one layer)
    afresh();
    const char* wnext = wl + (size_t)sg.block() * D * 64;
    // stored K/V fragments (wave-uniform user, scalar loop control); KD key tiles on their way
    constexpr int KD = 2;
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
    if (nkt == 0) kb = vb = wl;                      // (readable: requests are made without asking, so that no value lives on through a branch)
    grp kn[KD][2], vn[KD][2];                        // (kn[..][1] stays unused: a head of 16 features is one operand group)
#pragma unroll
    for (int b = 0; b < KD; ++b) vn[b][0] = vn[b][1] = grp{};        // (the lanes of the other head's features are never loaded)
    auto fetch = [&](int kt, int b) {
      if (selfl) {
        kn[b][0] = kvl[STACK ? kt : 0][ft][0][head][lane];
#pragma unroll
        for (int g = 0; g < 2; ++g) vn[b][g] = kvl[STACK ? kt : 0][ft][1][g][lane];
        return;
      }
      const size_t fo = (size_t)(kt * NT + ft) * 2048;
      gchar *kq = (gchar*)(kb + fo + head * 1024), *vq2 = (gchar*)(vb + fo);
      asm("" : "+s"(kq), "+s"(vq2));
      kn[b][0] = *(ggrp*)(kq + lane16);
      // (V's other features belong to the other head: their lanes ask for nothing, their zeros go nowhere)
      if (((lane >> 4) & 1) == head) {
#pragma unroll
        for (int g = 0; g < 2; ++g) vn[b][g] = *(ggrp*)(vq2 + (lane16 + (unsigned)g * 1024u));
      }
    };
    if (!selfl) {
#pragma unroll
      for (int b = 0; b < KD; ++b) fetch(min(b, max(nkt - 1, 0)), b);
    }
    store_vec();
    {
      grp xn[NG];
      normalise(0, vl.ln1_g(), vl.ln1_b(), xn);
      request(f1, segment(wl, keeper || !(SCORE || selfl) ? sg.o(ft) : sg.v(ft)));
      if (keeper) {
        f32x16 aq = product(bias_tile(vec + vl.bq(), ft, hi), fr, xn, false, false, nullptr);
        settle(aq);
        aq *= p.scale_l2e;
#pragma unroll
        for (int g = 0; g < 2; ++g) qx[ft][g][lane] = E::pack(aq, g);
      } else if (SCORE || selfl) {
        f32x16 ak = product(splat16(0.f), fr, xn, false, false, nullptr);   // no b_K, no b_V: see block_kernel.h
        f32x16 av = product(splat16(0.f), f1, xn, true, false, nullptr);
        settle(ak); settle(av);
#pragma unroll
        for (int g = 0; g < 2; ++g) { kvl[ts][ft][0][g][lane] = E::pack(ak, g); kvl[ts][ft][1][g][lane] = E::pack(av, g); }
      }
    }
    float mrun[1] = {kNegBig}, lrun[1] = {0.f};            // this wave's head owns half of the accumulator's rows
    f32x16 acc[1];
    acc[0] = splat16(0.f);
    {
      __syncthreads();                                 // Q (K, V) of every feature tile
      if (selfl) {
#pragma unroll
        for (int b = 0; b < KD; ++b) fetch(min(b, max(nkt - 1, 0)), b);
      }
      grp qop[2];
      qop[0] = qop[1] = qx[ft][head][lane];
      if (SCORE) {   // keys of the lane's own tile: the candidate's own globals
        const grp kop = kvl[0][ft][0][head][lane];
        grp vop[2], pop[2];
#pragma unroll
        for (int g = 0; g < 2; ++g) vop[g] = kvl[0][ft][1][g][lane];
        f32x16 S = E::mma(kop, qop[0], splat16(0.f));
        settle(S);
        const int widx = W == 16 ? 0 : j / (2 * W);
        uint32_t wmask[16 / W];
#pragma unroll
        for (int w = 0; w < 16 / W; ++w) { wmask[w] = widx == w ? 0xffffffffu : 0u; asm("" : "+v"(wmask[w])); }
        softmax_window<T, W>(S, widx, wmask, tilebits, mrun[0], lrun[0], acc[0], pop);
#pragma unroll
        for (int g = 0; g < 2; ++g) acc[0] = E::mma(vop[g], pop[g], acc[0]);
      }
      auto key_tile = [&](int kt, int b) __attribute__((always_inline)) {
        key_tile_step<1, 1>(selfl ? skr : kr, kt, kn[b], vn[b], qop, hi, mrun, lrun, acc);
        if (kt + KD < nkt) fetch(kt + KD, b);
      };
      for (int kt = 0; kt < nkt; kt += KD) {
#pragma unroll
        for (int b = 0; b < KD; ++b)
          if (kt + b < nkt) key_tile(kt + b, b);
      }
    }
    request(fr, segment(wl, sg.w1(min(wave, NC - 1))));
    if (keeper) {
#pragma unroll
      for (int s = 0; s < 2 * WV; ++s) request_w2(0, s);
    }
    request_vec(project ? p.kv_w : last ? wl : wnext);
    {
      settle(acc[0]);
      const float inv = lrun[0] > 0.f ? __builtin_amdgcn_rcpf(lrun[0]) : 0.f;
      f32x16 o;
#pragma unroll
      for (int r = 0; r < 8; ++r) { const float lo = acc[0][r], up = acc[0][8 + r]; o[r] = (head ? up : lo) * inv; }
      ops[1][2 * ft + head][lane] = E::pack(o, 0);
    }
    __syncthreads();
    grp xn[NG];
    if (keeper) {
      take(1, xn);
      x += bias_tile(vec + vl.bo(), ft, hi);
      x = product(x, f1, xn, false, false, nullptr);
      settle(x);
    }
    afresh();
    normalise(1, vl.ln2_g(), vl.ln2_b(), xn);
    if (keeper) x += bias_tile(vec + vl.b2(), ft, hi);
    // the next product behind this block: the next block's Q (K), or the next layer's K and V
    gchar* ahead = segment(wl, sg.q(ft));
    if (!last) { const QuadSegs<LAYOUT, D> nx = {NC, false}; ahead = segment(wnext, keeper ? nx.q(ft) : nx.k(ft)); }
    if (project) ahead = segment(p.kv_w, keeper ? 1 + 2 * ft : 2 + 2 * ft);
    // a round: a hidden chunk per wave (one without a chunk goes through another's and hands in zeros), then all of them into x
    auto round = [&](auto more_, int c0, int par) {
      constexpr bool MORE = decltype(more_)::value;
      const int c = min(c0 + wave, NC - 1);
      f32x16 ah = product(bias_tile(vec + vl.b1(), c, hi), fr, xn, false, MORE, segment(wl, sg.w1(min(c0 + WV + wave, NC - 1))));
      if (!MORE) request(fr, ahead);
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
      __syncthreads();          // (the other parity was last read ahead of the barrier before)
      if (keeper) {
#pragma unroll
        for (int s = 0; s < 2 * WV; ++s) {
          x = E::mma_h(f2[s], hid[par][s / 2][s & 1][lane], x);
          if (MORE) request_w2(c0 + WV, s);
          __builtin_amdgcn_sched_barrier(0x486);
        }
      }
    };
    int c0 = 0, par = 0;
    for (; c0 + WV < NC; c0 += WV, par ^= 1) round(std::integral_constant<bool, true>{}, c0, par);
    round(std::integral_constant<bool, false>{}, c0, par);
    settle(x);
    wl = wnext;
    sg.attn = false;
  }

  // ------------------------------------------------------------------ epilogue
  const f32x16 one[1] = {x};
  if (p.X_out && inrange && keeper) store_rows<T, 1>(one, p.X_out, p.X_f32, out_off + 32 * ft, valid, hi);
  if (MODE == MODE_ATTN && p.kv_w) {      // split layout: [vectors][K V of feature tile 0][K V of feature tile 1] ...
    afresh();
    store_vec();
#pragma unroll
    for (int r = 0; r < 16; ++r) x[r] = valid ? x[r] : 0.f;      // (K and V of rows that do not exist: of zeros, nobody sees them)
    grp xn[NG];
    normalise(0, vl.ln1_g(), vl.ln1_b(), xn);
    const size_t fo = (size_t)usr * p.kv_w_ustride + ((size_t)(tile * NT + ft) * 2) * 1024 + lane16;
    f32x16 a = keeper ? product(splat16(0.f), fr, xn, false, false, nullptr) : product(splat16(0.f), fr, xn, true, false, nullptr);
    settle(a);
    char* dst = keeper ? p.kv_k : p.kv_v;
#pragma unroll
    for (int g = 0; g < 2; ++g) *reinterpret_cast<grp*>(dst + fo + g * 1024) = E::pack(a, g);
  }
  if (p.logits && (MODE != MODE_ATTN || p.q0 + tile == 0)) {       // (the global rows, at most 32, are all in a user's first tile)
    // logit = <head_w, flatten(global rows)> + head_b: each wave sums over its own feature tile
    const int a = SCORE ? (32 * tile + j) % p.m : 32 * tile + j, width = SCORE ? p.m : 32;    // row inside the head's m rows; lanes per logit
    float part = 0.f;
    if (valid && a < p.m && keeper) {
      const f32x16 hw = bias_tile(p.head + (size_t)a * D, ft, hi);
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
  };
  if (wave < NT) run(std::true_type{}); else run(std::false_type{});
}

// Host-side launcher, the signature of launch_quad (quad_kernel.h).  pair: the scoring stream is in the pair layout.
template <int D>
int launch_chain(int mode, int win, bool pair, const BlockParams& p, dim3 grid, hipStream_t stream);

#define LONGER_CHAIN_LAUNCH(D, MODEV, WV, LAY, ...)                                                                                      \
  do {                                                                                                                                   \
    constexpr int NTHR = 64 * chain_waves(D) * quad_tiles(MODEV);                                                                        \
    if (p.act == 1) hipLaunchKernelGGL((chain_kernel<D, MODEV, WV, LAY, true, ##__VA_ARGS__>), grid, dim3(NTHR), 0, stream, p);          \
    else hipLaunchKernelGGL((chain_kernel<D, MODEV, WV, LAY, false, ##__VA_ARGS__>), grid, dim3(NTHR), 0, stream, p);                    \
  } while (0)

template <int D, int LAY>
static void launch_chain_score(int win, const BlockParams& p, dim3 grid, hipStream_t stream) {
  if (win == 4) LONGER_CHAIN_LAUNCH(D, MODE_SCORE, 4, LAY);
  else if (win == 8) LONGER_CHAIN_LAUNCH(D, MODE_SCORE, 8, LAY);
  else LONGER_CHAIN_LAUNCH(D, MODE_SCORE, 16, LAY);
}

// (two tiles of width 128 would be sixteen waves, too many registers: the stack has d = 64 only; width 64 streams the plain layouts)
template <int D>
static int launch_chain_other(int mode, const BlockParams& p, dim3 grid, hipStream_t stream) {
  if (mode == MODE_ATTN) { LONGER_CHAIN_LAUNCH(D, MODE_ATTN, 16, QUAD_PLAIN); return 0; }
  if constexpr (D == 64) {
    if (p.kv_w) LONGER_CHAIN_LAUNCH(D, MODE_STACK, 16, QUAD_PLAIN, true);
    else LONGER_CHAIN_LAUNCH(D, MODE_STACK, 16, QUAD_PLAIN);
    return 0;
  }
  return -1;
}

#define LONGER_CHAIN_INSTANTIATE(D)                                                                                                      \
  template <>                                                                                                                            \
  int launch_chain<D>(int mode, int win, bool pair, const BlockParams& p, dim3 grid, hipStream_t stream) {                               \
    if (mode != MODE_SCORE) { if (pair || launch_chain_other<D>(mode, p, grid, stream)) return -1; }                                     \
    else if (pair != (D == 128)) return -1;                                                                                              \
    else launch_chain_score<D, D == 128 ? QUAD_PAIR : QUAD_PLAIN>(win, p, grid, stream);                                                 \
    return hipGetLastError() == hipSuccess ? 0 : -3;                                                                                     \
  }

}  // namespace longer
