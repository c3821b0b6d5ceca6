// Up to four tiles of 32 rows in one workgroup of eight waves (bf16), where a wave owns a FEATURE tile (its part of the rows, of
// every product's result, its heads) for several row tiles:
//
//   MODE_STACK  the whole reduced stack of a user (Eq. 10) with at most four tiles, d = 128 / 256;
//   MODE_MERGE  the InnerTrans blocks and the merge (Section 3.4) of four tiles of raw tokens, d = 256.
//
// Why.  The kernels that give a row tile to one or two waves read every weight fragment once per row tile out of an LDS ring, and at
// width 256 there is no room beside such a ring for a user's K and V: one wave per SIMD, every wait exposed.  Here a fragment
// goes from L2 to the registers of the one wave that needs it and serves all of its row tiles (4 at width 256, 2 at width 128, where
// two groups of waves take two row tiles each), LDS holds nothing but operands, and since a wave makes K and V of its heads
// for its row tiles itself, at width 256 they never leave its registers.  Eight waves, two per SIMD.
// Fragments are requested a product ahead as in quad_kernel.h.
//
// The merge at width 256: 160 000 raw tokens, one block, a wave a tile 335 us, this 303 us, with the last FFN product on
// group sums 237.  (At width 128 a tile's wave needs half the registers and two share a SIMD: the two mappings take the same time.)
//
// What bounds it: at width 256 LDS, which hands every product its row operand (1 KiB per matrix instruction and wave, the
// 128 bytes a cycle that four SIMDs can use up), at width 128 the vector work of the attention.
#pragma once
#include "quad_kernel.h"

namespace longer {

constexpr int kUserWaves = 8;
constexpr int user_groups(int d) { return kUserWaves / (d / 32); }     // groups of waves that share out the row tiles

template <int D, int DH, int RT, int LAYOUT, bool RELU, int MODE = MODE_STACK, int W = 16, bool POOL = false>
__global__ void __launch_bounds__(64 * kUserWaves, 1) user_kernel(const BlockParams p) {
  using T = __bf16;
  using E = ET<T>;
  using grp = typename E::grp;
  using hgrp = typename E::hgrp;
  constexpr int NT = D / 32, NG = D / 16, WV = NT, TG = user_groups(D), TS = TG * RT, HPT = 32 / DH, GPH = DH / 16, kThr = 64 * kUserWaves;
  constexpr bool HOLD = D <= 128;                    // (width 256: no registers for the output projection's fragments through the attention)
  constexpr bool MERGE = MODE == MODE_MERGE;
  static_assert(!MERGE || TG == 1, "the merge's keys stay in their wave");
  static_assert(2 * WV == NG, "as many fragments in a hidden chunk's second product as in its first");
  __shared__ grp ops[TS][NG][64];                    // normalised rows: [row tile][group][lane]
  __shared__ grp mid[TS][NT][2][64];                 // [row tile][wave][group][lane]: Q, then the attention output; activated hidden chunks
  __shared__ float2 sums[TS][NT][32];                // row sums: [row tile][wave][row]
  __shared__ grp kvl[TG > 1 ? TS : 1][TG > 1 ? NT : 1][2][2][64];      // self layers, several groups: [key tile][feature tile][K, V][group][lane]
  __shared__ f32x4 vecl[D * 4];                      // the block's fp32 vectors (at most one segment)
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), ft = wv % WV, t0 = (wv / WV) * RT;    // feature tile, first row tile
  int tid = threadIdx.x, lane = tid & 63, j = lane & 31, hi = lane >> 5;
  unsigned lane16 = (unsigned)lane * 16u;
  auto afresh = [&] {                                // (see quad_kernel.h)
    asm volatile("" : "+v"(tid));
    lane = tid & 63; j = lane & 31; hi = lane >> 5; lane16 = (unsigned)lane * 16u;
  };
  const int NC = p.FF / 32, usr = MERGE ? 0 : (int)blockIdx.x, rows = p.rows_per_user;
  QuadSegs<LAYOUT, D> sg = {NC, !MERGE};             // (the stack's first block is the cross layer's attention half)
  int len = MERGE ? 0 : p.lens ? p.lens[usr] : p.L; len = min(max(len, 0), p.L);
  const int tu = (len + p.K - 1) / p.K, i0 = first_slot(p.k, tu, p.q_learn);
  // merge: the lane's token in row tile rt of the workgroup (slots count [B][T K], a group never spans two tiles)
  struct Token { uint32_t gidx; int jj, left; bool stored; long long row; };      // left: the group's valid tokens (at most K)
  auto locate = [&](int rt) {
    Token k;
    const uint32_t slot = ((uint32_t)blockIdx.x * TS + (uint32_t)(t0 + rt)) * 32u + (uint32_t)j;
    k.gidx = slot >> __builtin_ctz(p.K);
    k.jj = (int)(slot & (uint32_t)(p.K - 1));
    const int u = (int)(k.gidx / (uint32_t)p.T), t = (int)(k.gidx - (uint32_t)u * (uint32_t)p.T);
    k.stored = u < p.B;
    int n = 0;
    if (k.stored) { n = p.lens ? p.lens[u] : p.L; n = min(max(n, 0), p.L); }
    k.left = min(max(n - t * p.K, 0), p.K);
    k.row = (long long)u * p.L + t * p.K + k.jj;
    return k;
  };
  uint32_t there[RT];                                // merge: which of a row tile's tokens exist

  // ------------------------------------------------------------------ rows
  auto row_valid = [&](int a) { return a < rows && (a < p.m || a - p.m >= i0); };
  auto row_token = [&](int a) { return p.q_learn ? tu - 1 : slot_token(a - p.m, p.k, tu, p.k_uni); };   // newest merged token slot row a sees
  f32x16 x[RT];
  Token at[RT];
  if constexpr (MERGE) {
    uint32_t any = 0;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      at[rt] = locate(rt);
      there[rt] = (uint32_t)__ballot(at[rt].jj < at[rt].left);
      any |= there[rt];
    }
    // Nothing but padding (the same tiles in every wave: all leave).  Zeros by all threads, a row from 64 of them, rather than by the lanes that hold a group's first
    // token, behind the row requests: 512 users of 100 to 2000 tokens, K = 8 995 / 1015 us, 128 of at most 5000, K = 16 522 / 527.
    if (POOL && any == 0) {
      const uint32_t groups = RT * (32u >> __builtin_ctz(p.K)), g0 = (uint32_t)blockIdx.x * groups;
      for (uint32_t i = threadIdx.x; i < groups * (D / 4); i += kThr) {
        const uint32_t g = g0 + i / (D / 4);
        if (g >= (uint32_t)p.B * (uint32_t)p.T) break;
        const size_t o = (size_t)g * D + 4 * (i % (D / 4));
        if (p.M_f32) *(f32x4*)(reinterpret_cast<float*>(p.M_out) + o) = f32x4{0.f, 0.f, 0.f, 0.f};
        else *(uint2*)(reinterpret_cast<__bf16*>(p.M_out) + o) = make_uint2(0u, 0u);
      }
      return;
    }
  }
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    if constexpr (MERGE) {
      const Token& k = at[rt];
      const bool valid = k.jj < k.left;
      f32x16 one[1];
      load_rows<T, 1>(one, p.H, 0, k.row * D + 32 * ft, valid, hi);
      x[rt] = one[0];
      continue;
    }
    const int a = 32 * (t0 + rt) + j;
    const bool glob = a < p.m;
    const int row = glob ? a : (p.gather_recent ? row_token(a) : a - p.m);
    f32x16 one[1];
    load_rows<T, 1>(one, glob ? p.src0.p : p.src1.p, glob ? p.src0.f32 : p.src1.f32,
                    (glob ? p.src0.ustride : p.src1.ustride) * usr + (long long)row * D + 32 * ft, row_valid(a), hi);
    x[rt] = one[0];
  }

  // The last block's second FFN product where only the groups' means leave (p.pool): it is linear, so it takes the sums of the activated values, a column
  // a group instead of a column a token: one tile of columns instead of four, in the products and in what they read from LDS.  The first
  // product runs with its operands exchanged (lane = hidden value, registers = tokens), so that the sums are in-lane: the activation's last
  // product and the sum are one dot instruction, in fp32.  A sum goes on as two fp16 values, what the first leaves over sixteen columns
  // further.  A padded token starts from a value whose activation is zero.  K = 8, 16, 32 (below, the columns are more than a tile).
  // 160 000 tokens of width 256, K = 16, one block: 291 -> 246 us, 237 with the activation of either
  // half of the row tiles behind the other one's products; as a run-time branch in the layer loop 200 registers spilled and it took 295.
  constexpr int KK = W == 4 ? 8 : 2 * W, GPW = 32 / KK;      // tokens of a group, groups of a row tile
  // merge: token rows and merged tokens of this wave's features, zeros where there are none
  auto merge_out = [&](bool zeros) {
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      const Token k = locate(rt);
      if (p.Z_out && k.stored) {
        const f32x16 one[1] = {x[rt]};
        store_rows<T, 1>(one, p.Z_out, p.Z_f32, ((long long)k.gidx * p.K + k.jj) * D + 32 * ft, !zeros && k.jj < k.left, hi);
      }
      if (!p.M_out) continue;
      f32x16 sum[1] = {x[rt] * (k.jj < k.left ? 1.0f / (float)k.left : 0.f)};      // mean over the group, on K adjacent lanes (block_kernel.h)
      if (!zeros) {
        if (p.K >= 2) lane_sum<0xB1, 1>(sum);
        if (p.K >= 4) lane_sum<0x4E, 1>(sum);
        if (p.K >= 8) lane_sum<0x141, 1>(sum);
        if (p.K >= 16) lane_sum<0x140, 1>(sum);
        if (p.K >= 32) {
#pragma unroll
          for (int r = 0; r < 16; ++r) sum[0][r] += __shfl_xor(sum[0][r], 16, 64);
        }
      }
      if (k.stored && k.jj == 0) store_rows<T, 1>(sum, p.M_out, p.M_f32, (long long)k.gidx * D + 32 * ft, !zeros, hi);
    }
  };
  if constexpr (MERGE && !POOL) {
    uint32_t any = 0;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) any |= there[rt];
    if (any == 0) { merge_out(true); return; }
  }

  const char* wl = p.wbase;                          // the current block's stream
  const VecLayout vl{D, p.FF};
  const float* vec = reinterpret_cast<const float*>(vecl);
  grp fr[NG];
  typedef __attribute__((address_space(1))) const char gchar;
  typedef __attribute__((address_space(1))) const grp ggrp;
  auto segment = [&](const char* w, int seg) -> gchar* {       // (wave-uniform: a scalar base, the lane's part an offset)
    gchar* q = (gchar*)(w + (size_t)(unsigned)__builtin_amdgcn_readfirstlane(seg * (NG * 1024)));
    asm("" : "+s"(q));
    return q;
  };
  auto load = [&](gchar* q, int s) -> grp { return *(ggrp*)(q + (lane16 + (unsigned)s * 1024u)); };
  auto request = [&](gchar* q) {
#pragma unroll
    for (int s = 0; s < NG; ++s) fr[s] = load(q, s);
  };
  // acc[rt] += (32 result features) of row tile rt's operand groups b(rt, s), which come out of LDS a step ahead; then(s): the
  // request that takes the registers of fragment s.  SWAP: result with lane = feature
  auto product = [&](f32x16 (&acc)[RT], auto swap, auto b, auto mma, auto then) __attribute__((always_inline)) {
    grp cur[RT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) cur[rt] = b(rt, 0);
#pragma unroll
    for (int s = 0; s < NG; ++s) {
      grp nxt[RT];
      if (s + 1 < NG) {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) nxt[rt] = b(rt, s + 1);
      }
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) acc[rt] = swap ? mma(cur[rt], fr[s], acc[rt]) : mma(fr[s], cur[rt], acc[rt]);
      then(s);
      __builtin_amdgcn_sched_barrier(0);
      if (s + 1 < NG) {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) cur[rt] = nxt[rt];
      }
    }
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) settle(acc[rt]);
  };
  // the same for row tiles T0 .. T1 - 1 alone, behind(n) after the n-th matrix instruction
  auto part = [&](f32x16 (&acc)[RT], auto t0_, auto t1_, auto b, auto mma, auto then, auto behind) __attribute__((always_inline)) {
    constexpr int T0 = decltype(t0_)::value, T1 = decltype(t1_)::value, N = T1 - T0;
    grp cur[N];
#pragma unroll
    for (int i = 0; i < N; ++i) cur[i] = b(T0 + i, 0);
#pragma unroll
    for (int s = 0; s < NG; ++s) {
      grp nxt[N];
      if (s + 1 < NG) {
#pragma unroll
        for (int i = 0; i < N; ++i) nxt[i] = b(T0 + i, s + 1);
      }
#pragma unroll
      for (int i = 0; i < N; ++i) {
        acc[T0 + i] = mma(fr[s], cur[i], acc[T0 + i]);
        if (i + 1 == N) then(s);
        behind(s * N + i);
        __builtin_amdgcn_sched_barrier(0);
      }
      if (s + 1 < NG) {
#pragma unroll
        for (int i = 0; i < N; ++i) cur[i] = nxt[i];
      }
    }
#pragma unroll
    for (int i = 0; i < N; ++i) settle(acc[T0 + i]);
  };
  auto mma16 = [](grp a, grp b, f32x16 c) { return E::mma(a, b, c); };
  auto mma_h = [](grp a, grp b, f32x16 c) { return E::mma_h(a, __builtin_bit_cast(hgrp, b), c); };
  auto normed = [&](int rt, int s) -> grp { return ops[t0 + rt][s][lane]; };
  auto middle = [&](int rt, int s) -> grp { return mid[t0 + rt][s / 2][s & 1][lane]; };
  constexpr std::false_type plain{};
  constexpr std::true_type swapped{};

  constexpr int VQ = (D * 4 + kThr - 1) / kThr;      // the block's vectors: this thread's share, on its way to LDS
  f32x4 vq[VQ];
  auto request_vec = [&](const char* w) {
    const int n = (9 * D + p.FF) / 4;
#pragma unroll
    for (int i = 0; i < VQ; ++i) { const int c = tid + kThr * i; vq[i] = reinterpret_cast<const f32x4*>(w)[c < n ? c : 0]; }
  };
  request_vec(wl);
  request(segment(wl, sg.q(ft)));
  // LayerNorm of the rows: the next products' operand, in LDS
  auto normalise = [&](int og, int ob) __attribute__((always_inline)) {
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      float s = 0.f, q = 0.f;
#pragma unroll
      for (int r = 0; r < 16; ++r) { s += x[rt][r]; q = fmaf(x[rt][r], x[rt][r], q); }
      const float2 both = make_float2(sum_halves(s), sum_halves(q));
      if (hi == 0) sums[t0 + rt][ft][j] = both;
    }
    __syncthreads();
    const f32x16 g = bias_tile(vec + og, ft, hi), c = bias_tile(vec + ob, ft, hi);
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      float2 t = make_float2(0.f, 0.f);
#pragma unroll
      for (int w = 0; w < NT; ++w) { const float2 q = sums[t0 + rt][w][j]; t.x += q.x; t.y += q.y; }
      const float mean = t.x * (1.0f / D), var = fmaxf(t.y * (1.0f / D) - mean * mean, 0.f);
      const float rstd = __builtin_amdgcn_rsqf(var + p.eps), shift = -mean * rstd;
      f32x16 y;
#pragma unroll
      for (int r = 0; r < 16; ++r) y[r] = fmaf(fmaf(x[rt][r], rstd, shift), g[r], c[r]);
#pragma unroll
      for (int g2 = 0; g2 < 2; ++g2) ops[t0 + rt][2 * ft + g2][lane] = E::pack(y, g2);
    }
    __syncthreads();
  };

  // One block; SELF: K and V of the user's own rows are made here.  Areas of LDS: `ops` is written by a LayerNorm when everybody
  // has passed the barriers behind its last readers (Q / K / V, W1), `sums` likewise; a wave's part of `mid` is its own up to
  // the barrier behind the attention.
  auto block = [&](auto selfl, bool last, auto pooledl) __attribute__((always_inline)) {
    constexpr bool SELF = decltype(selfl)::value, POOLED = decltype(pooledl)::value;      // POOLED: the merge's last block, see above
    const char* wnext = wl + (size_t)sg.block() * D * 64;
    afresh();
#pragma unroll
    for (int i = 0; i < VQ; ++i) { const int c = tid + kThr * i; if (c < D * 4) vecl[c] = vq[i]; }
    normalise(vl.ln1_g(), vl.ln1_b());
    grp kop[SELF && TG == 1 ? RT : 1][2], vop[SELF && TG == 1 ? RT : 1][2];
    {
      f32x16 a[RT];
      const f32x16 bias = bias_tile(vec + vl.bq(), ft, hi);
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) a[rt] = bias;
      gchar* next = segment(wl, SELF ? sg.k(ft) : sg.o(ft));
      product(a, plain, normed, mma16, [&](int s) { if (SELF || HOLD) fr[s] = load(next, s); });
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        a[rt] *= p.scale_l2e;
#pragma unroll
        for (int g = 0; g < 2; ++g) mid[t0 + rt][ft][g][lane] = E::pack(a[rt], g);
      }
      if constexpr (SELF) {
#pragma unroll
        for (int m = 0; m < 2; ++m) {                // K, V (no b_K, no b_V: see block_kernel.h; V with lane = feature)
#pragma unroll
          for (int rt = 0; rt < RT; ++rt) a[rt] = splat16(0.f);
          next = segment(wl, m == 0 ? sg.v(ft) : sg.o(ft));
          auto then = [&](int s) { if (m == 0 || HOLD) fr[s] = load(next, s); };
          if (m == 0) product(a, plain, normed, mma16, then); else product(a, swapped, normed, mma16, then);
#pragma unroll
          for (int rt = 0; rt < RT; ++rt) {
#pragma unroll
            for (int g = 0; g < 2; ++g) {
              const grp v = E::pack(a[rt], g);
              if constexpr (TG == 1) { if (m == 0) kop[rt][g] = v; else vop[rt][g] = v; }
              else kvl[t0 + rt][ft][m][g][lane] = v;
            }
          }
        }
        if (TG > 1) __syncthreads();
      }
    }
    // ---- attention of the wave's heads, a row tile at a time
    if constexpr (MERGE && SELF) {                   // inside the groups: the keys are the tile's own rows
      const int widx = W == 16 ? 0 : j / (2 * W);
      uint32_t wmask[16 / W];
#pragma unroll
      for (int w = 0; w < 16 / W; ++w) wmask[w] = widx == w ? 0xffffffffu : 0u;
      const uint32_t gb = (p.K >= 32 ? 0xffffffffu : ((1u << p.K) - 1u)) << (p.K * (j / p.K));
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        const uint32_t bits = ((gb & there[rt]) >> (4 * hi)) >> (2 * W * widx);
        grp qop[2];
#pragma unroll
        for (int g = 0; g < 2; ++g) qop[g] = mid[t0 + rt][ft][g][lane];
        f32x16 o;
#pragma unroll
        for (int hh = 0; hh < HPT; ++hh) {
          float mrun = kNegBig, lrun = 0.f;
          f32x16 acc = splat16(0.f), S = splat16(0.f);
#pragma unroll
          for (int g2 = 0; g2 < GPH; ++g2) S = E::mma(kop[rt][hh * GPH + g2], qop[hh * GPH + g2], S);
          grp pop[2];
          softmax_window<T, W>(S, widx, wmask, bits, mrun, lrun, acc, pop);
#pragma unroll
          for (int g = 0; g < 2; ++g) acc = E::mma(vop[rt][g], pop[g], acc);
          const float inv = lrun > 0.f ? __builtin_amdgcn_rcpf(lrun) : 0.f;
#pragma unroll
          for (int r = 0; r < 16 / HPT; ++r) o[16 / HPT * hh + r] = acc[16 / HPT * hh + r] * inv;
        }
#pragma unroll
        for (int g = 0; g < 2; ++g) mid[t0 + rt][ft][g][lane] = E::pack(o, g);
      }
    }
#pragma unroll 1
    for (int rt = 0; !MERGE && rt < RT; ++rt) {
      const int a = 32 * (t0 + rt) + j;
      if (32 * (t0 + rt) >= rows) break;
      const bool ok = row_valid(a), glob = a < p.m;
      // visible key ranges (Eq. 8 by token type); a self layer's keys are the user's own rows, key index = row index
      KeyRanges kr = {};
      if (glob) { kr.lo1 = p.gmask_causal ? a : 0; kr.hi1 = SELF ? p.m : p.KG; }
      if (SELF) { kr.lo2 = p.m + i0; kr.hi2 = glob ? p.m + p.k : a + 1; }
      else { kr.lo2 = p.KG; kr.hi2 = p.KG + (glob ? tu : row_token(a) + 1); }
      kr.settle_for(ok);
      grp qop[2];
#pragma unroll
      for (int g = 0; g < 2; ++g) qop[g] = mid[t0 + rt][ft][g][lane];
      float mrun[HPT], lrun[HPT];
      f32x16 acc[HPT];
#pragma unroll
      for (int hh = 0; hh < HPT; ++hh) { mrun[hh] = kNegBig; lrun[hh] = 0.f; acc[hh] = splat16(0.f); }
      auto key_tile = [&](int kt, const grp (&k)[2], const grp (&v)[2]) __attribute__((always_inline)) { key_tile_step<HPT, GPH>(kr, kt, k, v, qop, hi, mrun, lrun, acc); };
      if constexpr (SELF) {
        const int nkt = (rows + 31) / 32;
        if constexpr (TG == 1) {
#pragma unroll
          for (int kt = 0; kt < RT; ++kt)
            if (kt < nkt) key_tile(kt, kop[kt], vop[kt]);
        } else {
          for (int kt = 0; kt < nkt; ++kt) {
            grp k[2], v[2];
#pragma unroll
            for (int g = 0; g < 2; ++g) { k[g] = kvl[kt][ft][0][g][lane]; v[g] = kvl[kt][ft][1][g][lane]; }
            key_tile(kt, k, v);
          }
        }
      } else {                                       // stored K / V fragments (scalar loop control), KD key tiles on their way
        constexpr int KD = 4;
        const int nkt = __builtin_amdgcn_readfirstlane((p.KG + tu + 31) / 32);
        const char* kb = nkt > 0 ? p.kst + (size_t)usr * p.kv_ustride : wl;    // (readable in any case: requests are unconditional)
        const char* vb = nkt > 0 ? p.vst + (size_t)usr * p.kv_ustride : wl;
        grp kn[KD][2], vn[KD][2];
        auto fetch = [&](int kt, int b) {
          const size_t fo = ((size_t)(min(kt, max(nkt - 1, 0)) * NT + ft) * 2) * 1024 + lane16;
#pragma unroll
          for (int g = 0; g < 2; ++g) {
            kn[b][g] = *reinterpret_cast<const grp*>(kb + fo + g * 1024);
            vn[b][g] = *reinterpret_cast<const grp*>(vb + fo + g * 1024);
          }
        };
#pragma unroll
        for (int b = 0; b < KD; ++b) fetch(b, b);
        for (int kt = 0; kt < nkt; kt += KD) {
#pragma unroll
          for (int b = 0; b < KD; ++b) {
            if (kt + b < nkt) key_tile(kt + b, kn[b], vn[b]);
            fetch(kt + b + KD, b);
          }
        }
      }
      f32x16 o;
      float inv[HPT];
#pragma unroll
      for (int hh = 0; hh < HPT; ++hh) { settle(acc[hh]); inv[hh] = lrun[hh] > 0.f ? __builtin_amdgcn_rcpf(lrun[hh]) : 0.f; }
#pragma unroll
      for (int r = 0; r < 16; ++r) o[r] = acc[HPT == 1 ? 0 : r / 8][r] * inv[HPT == 1 ? 0 : r / 8];
#pragma unroll
      for (int g = 0; g < 2; ++g) mid[t0 + rt][ft][g][lane] = E::pack(o, g);
    }
    if (!HOLD) request(segment(wl, sg.o(ft)));
    __syncthreads();
    {
      const f32x16 bias = bias_tile(vec + vl.bo(), ft, hi);
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) x[rt] += bias;
      gchar* next = segment(wl, sg.w1(ft));          // (at least as many hidden chunks as feature tiles: FF >= d)
      product(x, plain, middle, mma16, [&](int s) { fr[s] = load(next, s); });
    }
    afresh();
    request_vec(last ? wl : wnext);
    normalise(vl.ln2_g(), vl.ln2_b());
    if constexpr (POOLED) {
      {
        // the rows' own sums, a column a group as well, are what the product starts from (and no row is held through it)
        f32x16 ffn;
        {
          float* area = (float*)&mid[0][0][0][0] + ft * (16 * 36);
#pragma unroll
          for (int rt = 0; rt < RT; ++rt) {
            f32x16 sum[1] = {x[rt] * ((there[rt] >> j) & 1u ? 1.f / KK : 0.f)};
            lane_sum<0xB1, 1>(sum); lane_sum<0x4E, 1>(sum); lane_sum<0x141, 1>(sum);
            if (KK >= 16) lane_sum<0x140, 1>(sum);
            if (KK >= 32) {
#pragma unroll
              for (int r = 0; r < 16; ++r) sum[0][r] += __shfl_xor(sum[0][r], 16, 64);
            }
            if (j % KK == 0) {
#pragma unroll
              for (int q = 0; q < 4; ++q) *(f32x4*)(area + (rt * GPW + j / KK) * 36 + 8 * q + 4 * hi) = f32x4{sum[0][4 * q], sum[0][4 * q + 1], sum[0][4 * q + 2], sum[0][4 * q + 3]};
            }
          }
          __builtin_amdgcn_wave_barrier();
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const f32x4 v = *(const f32x4*)(area + (j & 15) * 36 + 8 * q + 4 * hi);
#pragma unroll
            for (int e = 0; e < 4; ++e) { const float one = v[e]; ffn[4 * q + e] = j < RT * GPW ? one : 0.f; }
          }
          __syncthreads();                           // (hidden chunks take the place)
        }
        // the lane's hidden value as an element of the operand groups: piece (operand group, lane half) of its column
        char* put = (char*)&mid[0][ft][(lane >> 4) & 1][32 * ((lane >> 2) & 1)] + 8 * ((lane >> 3) & 1) + 2 * (lane & 3);
        typedef std::integral_constant<int, 0> T0; typedef std::integral_constant<int, (RT + 1) / 2> TH; typedef std::integral_constant<int, RT> T1;
        constexpr int H = TH::value, NS = HiddenStages<RELU>::kStages;
        f32x16 ah[RT];
        auto start = [&](int c0, int first, int count) __attribute__((always_inline)) {
          const float bias = vec[vl.b1() + 32 * (c0 + ft) + j];
#pragma unroll
          for (int rt = first; rt < first + count; ++rt) {
            ah[rt] = splat16(bias);
            if (there[rt] != 0xffffffffu) {
              uint32_t mine = there[rt] >> (4 * hi);
              asm volatile("" : "+v"(mine));             // (asked again each time: 64 answers held would be 128 registers)
#pragma unroll
              for (int r = 0; r < 16; ++r) ah[rt][r] = (mine >> (8 * (r / 4) + r % 4)) & 1u ? bias : -1e38f;
            }
          }
        };
        HiddenStages<RELU> act;
        float sum[GPW];
        // a row tile's sums, as operands, to buffer `par` of the hidden chunks
        auto finish = [&](int rt, int par) __attribute__((always_inline)) {
          auto halves = [](float a, float b) {       // lanes below 32: a's sum over the lane halves, the others: b's
            const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, a), __builtin_bit_cast(unsigned, b), false, false);
            const unsigned r0 = r[0], r1 = r[1];
            return (__builtin_bit_cast(float, r0) + __builtin_bit_cast(float, r1)) * (1.f / KK);
          };
          const float v0 = halves(sum[0], sum[GPW > 1 ? 1 : 0]), v1 = GPW == 4 ? halves(sum[GPW == 4 ? 2 : 0], sum[GPW == 4 ? 3 : 0]) : 0.f;
          const f16x2 h = __builtin_bit_cast(f16x2, __builtin_amdgcn_cvt_pkrtz(v0, v1));
          // (the rest of an infinite sum, a NaN, becomes the lowest finite number, which the infinity outweighs)
          const f16x2 l = __builtin_elementwise_max(__builtin_bit_cast(f16x2, __builtin_amdgcn_cvt_pkrtz(v0 - (float)h[0], v1 - (float)h[1])), (f16x2)((_Float16)-65504.f));
          char* at = put + par * (int)sizeof(mid[0]) + 16 * (rt * GPW + (GPW > 1 ? hi : 0));
          *(_Float16*)at = h[0];
          *(_Float16*)(at + 256) = l[0];
          if (GPW == 4) { *(_Float16*)(at + 32) = h[1]; *(_Float16*)(at + 32 + 256) = l[1]; }
        };
        // stages of row tiles first .. first + count - 1 behind the n-th of `of` matrix instructions
        auto stages = [&](int first, int count, int n, int of, int par) __attribute__((always_inline)) {
          const int all = count * 2 * NS;
#pragma unroll
          for (int i = 0; i < (all + of - 1) / of; ++i) {
            const int k = n * all / of + i;
            if (k >= (n + 1) * all / of) continue;
            const int rt = first + k / (2 * NS), g = k / NS % 2, st = k % NS;
            if (st < NS - 1) { act.run(ah[rt], g, st); continue; }
            f16x8 f;
            if (RELU) { f = (f16x8)((_Float16)1.f); HiddenStages<RELU>::pin(act.y); act.y = __builtin_elementwise_max(act.y, (f16x8)((_Float16)0.f)); }
            else { HiddenStages<RELU>::pin(act.p); f = act.p; }
#pragma unroll
            for (int e = 0; e < 4; ++e) {            // pair e: registers 8 g + 2 e, + 1; quad 2 g + e / 2
              const int at = (2 * g + e / 2) / (KK / 8), fresh = KK == 8 ? e % 2 == 0 : KK == 16 ? e == 0 : g == 0 && e == 0;
              const f16x2 y2 = {act.y[2 * e], act.y[2 * e + 1]}, f2 = {f[2 * e], f[2 * e + 1]};
              sum[at] = __builtin_amdgcn_fdot2(y2, f2, fresh ? 0.f : sum[at], false);
            }
            if (g == 1) finish(rt, par);
          }
        };
        auto nothing = [](int) {};
        auto mma_swapped = [](grp a, grp b, f32x16 c) { return E::mma(b, a, c); };
        grp fr2[NG];                                 // W2's fragments
        auto second = [&](int par) __attribute__((always_inline)) {
          grp cur = mid[par][0][0][lane];
#pragma unroll
          for (int s = 0; s < NG; ++s) {
            grp nxt = cur;
            if (s + 1 < NG) nxt = mid[par][(s + 1) / 2][(s + 1) & 1][lane];
            ffn = mma_h(fr2[s], cur, ffn);
            __builtin_amdgcn_sched_barrier(0);
            cur = nxt;
          }
        };
        auto w2_at = [&](int c0, int s) { return load(segment(wl + 2048 * ft, sg.w2(c0 + s / 2)), s & 1); };
        // Chunks c0: either half of the row tiles is activated under the other half's products, the second one's under the next chunks'; the second
        // product follows two barriers of the chunks behind (its operand is in one of two buffers)
        start(0, 0, H);
        part(ah, T0{}, TH{}, normed, mma_swapped, nothing, nothing);
        start(0, H, RT - H);
        for (int c0 = 0, par = 0;; par ^= 1) {
          gchar* next = segment(wl, sg.w1(min(c0 + WV, NC - WV) + ft));
          part(ah, TH{}, T1{}, normed, mma_swapped, [&](int s) { fr[s] = load(next, s); }, [&](int n) __attribute__((always_inline)) { stages(0, H, n, NG * (RT - H), par); });
          if (c0 > 0) second(par ^ 1);
          if (c0 + WV >= NC) {
#pragma unroll
            for (int s = 0; s < NG; ++s) fr2[s] = w2_at(c0, s);
#pragma unroll
            for (int n = 0; n < NG; ++n) stages(H, RT - H, n, NG, par);
            __syncthreads();
            second(par);
            break;
          }
          start(c0 + WV, 0, H);
          part(ah, T0{}, TH{}, normed, mma_swapped, [&](int s) { fr2[s] = w2_at(c0, s); }, [&](int n) __attribute__((always_inline)) { stages(H, RT - H, n, NG * H, par); });
          c0 += WV;
          start(c0, H, RT - H);
          __syncthreads();
        }
        settle(ffn);
        // a value and its rest: lanes below 16 of a lane half take the first eight registers of a column, the others the last eight
        const int c = lane & 15, half = (lane >> 4) & 1;
        const uint32_t gidx = (uint32_t)blockIdx.x * (RT * GPW) + (uint32_t)c;
        const int u = (int)(gidx / (uint32_t)p.T), t = (int)(gidx - (uint32_t)u * (uint32_t)p.T);
        const bool stored = c < RT * GPW && u < p.B;
        int n = 0;
        if (stored) { n = p.lens ? p.lens[u] : p.L; n = min(max(n, 0), p.L); }
        const int left = min(max(n - t * p.K, 0), p.K);
        const float share = left > 0 ? (float)KK / (float)left : 0.f;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const int f0 = 32 * ft + 16 * half + 8 * q + 4 * hi;
          const f32x4 bias = *(const f32x4*)(vec + vl.b2() + f0);
          f32x4 v;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float a = ffn[4 * q + e], b = ffn[8 + 4 * q + e];
            const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, a), __builtin_bit_cast(unsigned, b), false, false);
            const unsigned r0 = r[0], r1 = r[1];
            v[e] = left > 0 ? fmaf(__builtin_bit_cast(float, r0) + __builtin_bit_cast(float, r1), share, bias[e]) : 0.f;
          }
          if (!stored) continue;
          if (p.M_f32) *(f32x4*)(reinterpret_cast<float*>(p.M_out) + (size_t)gidx * D + f0) = v;
          else *(bf16x4*)(reinterpret_cast<__bf16*>(p.M_out) + (size_t)gidx * D + f0) = bf16x4{(__bf16)v[0], (__bf16)v[1], (__bf16)v[2], (__bf16)v[3]};
        }
      }
    }
    if constexpr (!POOLED) {
    {
      const f32x16 bias = bias_tile(vec + vl.b2(), ft, hi);
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) x[rt] += bias;
    }
    // A wave's row tiles in two halves, so that either half's activation goes behind the matrix instructions of the other one's products, first or
    // second (the two waves of a SIMD meet at every barrier and had nothing but the activation to do at the same time): 256 users of 108 rows at
    // width 256, concat merge, 340 -> 330 us a pass, with ReLU and an FFN as wide as the rows 233 -> 226.
    // Two row tiles stay together: width 256 (one wave a SIMD), 256 users of 64 rows, 69.4 us, in halves 71.1; width 128, 180 and 512 users of 72 rows 78.3 / 79.0 and
    // 172 / 175, 1000 of 108 409 / 406, with an FFN as wide as the rows 256 of 72 60.1 / 61.0, 512 of 108 149 / 150.  So do a stack's four with ReLU, two stages only, and heads of 16
    // (256 users of 108 rows, FFN of one, two, four times the width 227.9 / 232.9, 257.3 / 262.4, 320.8 / 323.2; three tiles of such rows 252.8 -> 252.0 in halves, a
    // merge's four 102.2 -> 99.5, 148.8 -> 144.6).
    constexpr bool SPLIT = RT > 2 && !(!MERGE && RT == 4 && DH == 16 && RELU);
    typedef std::integral_constant<int, 0> T0; typedef std::integral_constant<int, (RT + 1) / 2> TH; typedef std::integral_constant<int, RT> T1;
    constexpr int H = TH::value;
    for (int c0 = 0; c0 < NC; c0 += WV) {            // (FF is a multiple of d: every wave has a chunk)
      f32x16 ah[RT];
      const f32x16 bias = bias_tile(vec + vl.b1(), c0 + ft, hi);
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) ah[rt] = bias;
      HiddenStages<RELU> act;
      constexpr int NS = HiddenStages<RELU>::kStages;
      // stages of row tiles first .. first + count - 1 behind the n-th of `of` matrix instructions; a finished group goes to LDS
      auto stages = [&](int first, int count, int n, int of) __attribute__((always_inline)) {
        const int all = count * 2 * NS;
#pragma unroll
        for (int i = 0; i < (all + of - 1) / of; ++i) {
          const int k = n * all / of + i;
          if (k >= (n + 1) * all / of) continue;
          const int rt = first + k / (2 * NS), g = k / NS % 2, st = k % NS;
          const f16x8 y = act.run(ah[rt], g, st);
          if (st == NS - 1) mid[t0 + rt][ft][g][lane] = __builtin_bit_cast(grp, y);
        }
      };
      auto nothing = [](int) {};
      // what follows on these chunks' second product: the next hidden chunk, or the next block's first (chosen by a conditional expression, both places are
      // held through the product: four tiles with heads of 16, 84 instead of 64 registers spilled together, 62 instead of 51 in halves)
      auto following = [&]() __attribute__((always_inline)) -> gchar* {
        gchar* next = segment(wl, sg.w1(min(c0 + WV, NC - WV) + ft));
        if (c0 + WV >= NC && !last) next = segment(wnext, QuadSegs<LAYOUT, D>{NC, false}.q(ft));
        return next;
      };
      if constexpr (!SPLIT) {
        product(ah, plain, normed, mma16, [&](int s) { fr[s] = load(segment(wl + 2048 * ft, sg.w2(c0 + s / 2)), s & 1); });
        if (c0 > 0) __syncthreads();                 // everybody has read the chunks before
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
#pragma unroll
          for (int g = 0; g < 2; ++g) {
            f16x8 y;     // ah holds x / kFfnScale; to fp16 toward zero, then the packed activation
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const f16x2 y2 = __builtin_bit_cast(f16x2, __builtin_amdgcn_cvt_pkrtz(ah[rt][8 * g + 2 * e], ah[rt][8 * g + 2 * e + 1]));
              y[2 * e] = y2[0]; y[2 * e + 1] = y2[1];
            }
            y = RELU ? __builtin_elementwise_max(y, (f16x8)((_Float16)0.f)) : gelu_quarter_h8(y);
            mid[t0 + rt][ft][g][lane] = __builtin_bit_cast(grp, y);
          }
        }
        gchar* next = following();
        __syncthreads();
        product(x, plain, middle, mma_h, [&](int s) { fr[s] = load(next, s); });
        continue;
      }
      part(ah, T0{}, TH{}, normed, mma16, nothing, nothing);
      part(ah, TH{}, T1{}, normed, mma16, [&](int s) { fr[s] = load(segment(wl + 2048 * ft, sg.w2(c0 + s / 2)), s & 1); },
           [&](int n) __attribute__((always_inline)) { stages(0, H, n, NG * (RT - H)); });
      __syncthreads();
      part(x, T0{}, TH{}, middle, mma_h, nothing, [&](int n) __attribute__((always_inline)) { stages(H, RT - H, n, NG * H); });
      gchar* next = following();
      __syncthreads();
      part(x, TH{}, T1{}, middle, mma_h, [&](int s) { fr[s] = load(next, s); }, nothing);
    }
    }
    wl = wnext;
    sg.attn = false;
  };
  if constexpr (!MERGE) block(std::false_type{}, p.n_layers == 1, std::false_type{});
  for (int layer = MERGE ? 0 : 1; layer < p.n_layers - POOL; ++layer) block(std::true_type{}, layer + 1 == p.n_layers, std::false_type{});
  if constexpr (POOL) block(std::true_type{}, true, std::true_type{});

  // ------------------------------------------------------------------ epilogue
  afresh();
  if constexpr (MERGE) { if (!POOL) merge_out(false); return; }
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    const int a = 32 * (t0 + rt) + j;
    const f32x16 one[1] = {x[rt]};
    if (p.X_out && a < rows) store_rows<T, 1>(one, p.X_out, p.X_f32, p.X_ustride * usr + (long long)a * D + 32 * ft, row_valid(a), hi);
  }
  if (p.logits) {      // logit = <head_w, flatten(global rows)> + head_b: all global rows are in the first tile (m <= 32)
    float part = 0.f;
    if (t0 == 0 && j < p.m) {
      const f32x16 hw = bias_tile(p.head + (size_t)j * D, ft, hi);
#pragma unroll
      for (int r = 0; r < 16; ++r) part += x[0][r] * hw[r];
    }
    part = sum_halves(part);
    for (int sft = 1; sft < 32; sft <<= 1) part += __shfl_xor(part, sft, 64);
    if (t0 == 0 && lane == 0) sums[0][ft][0].x = part;      // (last read ahead of the FFN's barriers)
    __syncthreads();
    if (threadIdx.x == 0) {
      float logit = p.head[(size_t)p.m * D];
#pragma unroll
      for (int w = 0; w < NT; ++w) logit += sums[0][w][0].x;
      p.logits[usr] = logit;
    }
  }
}

// Host-side launchers, one definition per (D, DH) instantiation file; tiles: row tiles of a user (at most four); win: as in block_kernel.h
template <int D, int DH>
int launch_user(int tiles, const BlockParams& p, dim3 grid, hipStream_t stream);
constexpr int kUserMergeTiles = 4;
template <int D, int DH>
int launch_user_merge(int win, const BlockParams& p, dim3 grid, hipStream_t stream);

#define LONGER_USER_LAUNCH(D, DH, RT, LAY) \
  do {                                                                                                \
    if (p.act == 1) hipLaunchKernelGGL((user_kernel<D, DH, RT, LAY, true>), grid, dim3(64 * kUserWaves), 0, stream, p); \
    else hipLaunchKernelGGL((user_kernel<D, DH, RT, LAY, false>), grid, dim3(64 * kUserWaves), 0, stream, p); \
  } while (0)

// (width 128 streams the pair layouts, width 256 the plain ones)
#define LONGER_USER_INSTANTIATE_128(DH)                                                               \
  template <>                                                                                         \
  int launch_user<128, DH>(int, const BlockParams& p, dim3 grid, hipStream_t stream) {                \
    LONGER_USER_LAUNCH(128, DH, 2, QUAD_PAIR);                                                        \
    return hipGetLastError() == hipSuccess ? 0 : -3;                                                  \
  }
#define LONGER_USER_INSTANTIATE_256(DH)                                                               \
  template <>                                                                                         \
  int launch_user<256, DH>(int tiles, const BlockParams& p, dim3 grid, hipStream_t stream) {          \
    if (tiles <= 2) LONGER_USER_LAUNCH(256, DH, 2, QUAD_PLAIN);                                       \
    else if (tiles == 3) LONGER_USER_LAUNCH(256, DH, 3, QUAD_PLAIN);                                  \
    else LONGER_USER_LAUNCH(256, DH, 4, QUAD_PLAIN);                                                  \
    return hipGetLastError() == hipSuccess ? 0 : -3;                                                  \
  }
#define LONGER_USER_MERGE_LAUNCH(D, DH, WV, POOL) \
  do {                                                                                                \
    if (p.act == 1) hipLaunchKernelGGL((user_kernel<D, DH, kUserMergeTiles, QUAD_PLAIN, true, MODE_MERGE, WV, POOL>), grid, dim3(64 * kUserWaves), 0, stream, p); \
    else hipLaunchKernelGGL((user_kernel<D, DH, kUserMergeTiles, QUAD_PLAIN, false, MODE_MERGE, WV, POOL>), grid, dim3(64 * kUserWaves), 0, stream, p); \
  } while (0)
#define LONGER_USER_MERGE_WIN(D, DH, POOL) \
  do {                                                                                                \
    if (win == 4) LONGER_USER_MERGE_LAUNCH(D, DH, 4, POOL);                                           \
    else if (win == 8) LONGER_USER_MERGE_LAUNCH(D, DH, 8, POOL);                                      \
    else LONGER_USER_MERGE_LAUNCH(D, DH, 16, POOL);                                                   \
  } while (0)
#define LONGER_USER_MERGE_INSTANTIATE_256(DH)                                                         \
  template <>                                                                                         \
  int launch_user_merge<256, DH>(int win, const BlockParams& p, dim3 grid, hipStream_t stream) {      \
    if (p.pool) LONGER_USER_MERGE_WIN(256, DH, true); else LONGER_USER_MERGE_WIN(256, DH, false);     \
    return hipGetLastError() == hipSuccess ? 0 : -3;                                                  \
  }

}  // namespace longer
