// The transformer-block kernel with a 32-row tile given to a PAIR of waves (bf16, d = 128 / 256): candidate scoring of
// the KV-cache serving path (Section 3.6.3).
//
// Why.  Registers at d = 256 allow one tile-wave per SIMD only, and a single wave per SIMD is bound by its own
// instruction issue and dependency latencies.  Here a workgroup has 8 waves, two per SIMD: waves t
// and t + 4 share tile t.  They split every GEMM by output feature tile (wave half h owns tiles
// 2 i + h), so neither holds fp32 partial sums of the other:
//   - the fp32 residual rows are split by feature tile; LayerNorm exchanges two partial sums per row,
//     then each wave normalises its own tiles and the pair swaps the bf16 results through LDS (each
//     wave then holds all of LN(x), the B operand of Q / K / V and of the first FFN GEMM);
//   - Q, K, V and the attention heads of a wave's own tiles are private to it; the attention output
//     is swapped like the normalised rows and the output projection produces the own residual tiles;
//   - FFN: hidden chunks alternate between the two waves (first GEMM + activation), the activated
//     chunk goes through LDS, and each wave runs the second GEMM for its own output tiles over both;
//   - the packed stream brings the even and the odd tile of a matrix side by side (pair layouts,
//     device.h) in panels of two segments: one segment of work for either wave in every panel.
// Register indices never depend on the half (only LDS / global addresses do): a wave keeps its own
// operand groups and its partner's in separate arrays.
#pragma once
#include "block_kernel.h"

namespace longer {

constexpr int kPairThreads = 512;   // 8 waves: tile t is shared by waves t and t + 4 (the same SIMD)

template <int NTH>
__device__ __forceinline__ void load_rows_half(f32x16 (&x)[NTH], const void* base, int is_f32, long long off,
                                               bool valid, int hi, int h) {
#pragma unroll
  for (int i = 0; i < NTH; ++i) {
    f32x16 one[1];
    load_rows<__bf16, 1>(one, base, is_f32, off + 32 * (2 * i + h), valid, hi);
    x[i] = one[0];
  }
}

template <int NTH>
__device__ __forceinline__ void store_rows_half(const f32x16 (&x)[NTH], void* base, int is_f32, long long off,
                                                bool nonzero, int hi, int h) {
#pragma unroll
  for (int i = 0; i < NTH; ++i) {
    f32x16 one[1];
    one[0] = x[i];
    store_rows<__bf16, 1>(one, base, is_f32, off + 32 * (2 * i + h), nonzero, hi);
  }
}

// The stream's panels with the FFN skewed by a pair of hidden chunks: W1 of pair i + 1 comes ahead of W2 of pair i, which lies in front of it.
struct SkewedFfn {
  int front, panels, first;        // panels of a block in front of its FFN, in all; the current block's first
  __device__ __forceinline__ int at(int n) {
    if (n == first + panels) first += panels;
    const int q = n - first - front;
    return q < 1 || q == panels - front - 1 ? n : q & 1 ? n + 1 : n - 1;
  }
};

// SKEW: the activation of a pair of hidden chunks behind the second products of the pair before (where: pair_start)
template <int D, int DH, int W, bool RELU, bool SKEW>
__global__ void __launch_bounds__(kPairThreads, 1) pair_kernel(const BlockParams p) {
  using T = __bf16;
  using E = ET<T>;
  using grp = typename E::grp;
  constexpr int NT = D / 32, NTH = NT / 2, NG = D / E::GF, GPT = E::GPT, NGH = NG / 2;
  constexpr int SEGV = NG * 64;
  constexpr int HPT = 32 / DH;        // heads per 32-feature tile
  constexpr int GPH = DH / E::GF;     // operand groups per head
  static_assert(NT % 2 == 0 && (DH == 16 || DH == 32), "shape");
  constexpr int PSEG = 2;                           // a panel = the even and the odd tile's segment
  constexpr int NB = D >= 256 ? 2 : 3;              // ring depth in panels
  __shared__ uint4 lds[NB * PSEG * SEGV];
  __shared__ uint4 vecl[SEGV];                      // the current block's fp32 vectors
  __shared__ uint4 xch[4 * NG * 64];                // per tile: operand groups swapped inside the pair
  __shared__ float stat[4][2][2][32];               // per tile, half: LayerNorm partial sums / logit parts per row

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, j = lane & 31, hi = lane >> 5;
  const int ts = wave & 3, h = wave >> 2;           // tile slot in the workgroup; which half of the pair
  const int NC = p.FF / 32;

  // ------------------------------------------------------------------ rows of this wave's tile
  bool valid, inrange;
  int usr = 0, Tu = 0;
  long long out_off = 0;
  uint32_t tilebits = 0;
  const int widx = W == 16 ? 0 : j / (2 * W);
  uint32_t wmask[16 / W];
#pragma unroll
  for (int w = 0; w < 16 / W; ++w) { wmask[w] = widx == w ? 0xffffffffu : 0u; asm("" : "+v"(wmask[w])); }
  f32x16 resid[NTH];

  // all candidate tiles of a user on one XCD (see block_kernel.h)
  const int sq = (int)blockIdx.x / p.xcds, su = (int)blockIdx.x % p.xcds + p.xcds * (sq / p.wg_per_user);
  if (su >= p.B) return;
  const int tile = (sq % p.wg_per_user) * 4 + ts;
  {
    const int a = 32 * tile + j;
    const int cand = a / p.m, gi = a - cand * p.m;
    inrange = cand < p.C;
    valid = inrange;
    int len = p.lens ? p.lens[su] : p.L; len = min(max(len, 0), p.L);
    usr = su; Tu = (len + p.K - 1) / p.K;
    out_off = ((long long)su * p.C * p.m + a) * D;
    load_rows_half<NTH>(resid, p.Gc, 0, out_off, valid, hi, h);
    const uint32_t vb = (uint32_t)__ballot(valid);
    const int gbase = p.m * (j / p.m);
    tilebits = ((range_bits(gbase + (p.gmask_causal ? gi : 0), gbase + p.m, 0) & vb) >> (4 * hi)) >> (2 * W * widx);
  }

  WStream<SEGV, PSEG, NB, false, kPairThreads, std::conditional_t<SKEW, SkewedFfn, InOrder>> ws;
  if constexpr (SKEW) ws.order = SkewedFfn{1 + 2 * NT, 1 + 2 * NT + NC, 0};
  ws.init(lds, p.wbase, (2 + 4 * NT + 2 * NC) * p.n_layers);

  uint4* const xt = xch + (size_t)ts * NG * 64 + lane;      // this tile's exchange area, this lane's 16 bytes of a group
  // operand groups of own tiles go to the exchange area, the partner's come back
  auto swap_groups = [&](const grp (&own)[NGH], grp (&oth)[NGH]) {
#pragma unroll
    for (int i = 0; i < NTH; ++i)
#pragma unroll
      for (int g = 0; g < GPT; ++g) *reinterpret_cast<grp*>(xt + ((2 * i + h) * GPT + g) * 64) = own[i * GPT + g];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NTH; ++i)
#pragma unroll
      for (int g = 0; g < GPT; ++g) oth[i * GPT + g] = *reinterpret_cast<const grp*>(xt + ((2 * i + (h ^ 1)) * GPT + g) * 64);
  };
  // one 32-wide output tile of a GEMM over all of the pair's operand groups; `which` = the segment
  // of the current panel (0 / 1) that holds the weights
  auto gemm_tile = [&](f32x16 acc, int which, const grp (&own)[NGH], const grp (&oth)[NGH]) -> f32x16 {
#pragma unroll
    for (int i = 0; i < NTH; ++i)
#pragma unroll
      for (int g = 0; g < GPT; ++g) {
        acc = E::mma(ws.template frag_at<grp>(which, (2 * i + h) * GPT + g), own[i * GPT + g], acc);
        acc = E::mma(ws.template frag_at<grp>(which, (2 * i + (h ^ 1)) * GPT + g), oth[i * GPT + g], acc);
      }
    return acc;
  };
  const VecLayout vl{D, p.FF};
  const float* vec = reinterpret_cast<const float*>(vecl);
  // the tile's operand groups back from the exchange area: own[] = this wave's tiles, oth[] = the partner's
  auto load_groups = [&](grp (&own)[NGH], grp (&oth)[NGH]) {
#pragma unroll
    for (int i = 0; i < NTH; ++i)
#pragma unroll
      for (int g = 0; g < GPT; ++g) {
        own[i * GPT + g] = *reinterpret_cast<const grp*>(xt + ((2 * i + h) * GPT + g) * 64);
        oth[i * GPT + g] = *reinterpret_cast<const grp*>(xt + ((2 * i + (h ^ 1)) * GPT + g) * 64);
      }
  };
  // LayerNorm of the pair's rows, as B-operand groups in the exchange area (each wave writes its tiles)
  auto layer_norm_pair = [&](const float* gam, const float* bet) {
    float s = 0.f, q = 0.f;
#pragma unroll
    for (int i = 0; i < NTH; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) { s += resid[i][r]; q = fmaf(resid[i][r], resid[i][r], q); }
    s = sum_halves(s); q = sum_halves(q);
    if (hi == 0) { stat[ts][h][0][j] = s; stat[ts][h][1][j] = q; }
    __syncthreads();
    s += stat[ts][h ^ 1][0][j]; q += stat[ts][h ^ 1][1][j];
    const float mean = s * (1.0f / D);
    const float var = fmaxf(q * (1.0f / D) - mean * mean, 0.f);
    const float rstd = __builtin_amdgcn_rsqf(var + p.eps);
    const float shift = -mean * rstd;
#pragma unroll
    for (int i = 0; i < NTH; ++i) {
      const f32x16 gt = bias_tile(gam, 2 * i + h, hi), bt = bias_tile(bet, 2 * i + h, hi);
      f32x16 y;
#pragma unroll
      for (int r = 0; r < 16; ++r) y[r] = fmaf(fmaf(resid[i][r], rstd, shift), gt[r], bt[r]);
#pragma unroll
      for (int g = 0; g < GPT; ++g) *reinterpret_cast<grp*>(xt + ((2 * i + h) * GPT + g) * 64) = E::pack(y, g);
    }
    __syncthreads();
  };

  for (int layer = 0; layer < p.n_layers; ++layer) {
    // the block's first segment holds its fp32 vectors: keep a copy for the whole layer
    // (barriers: nobody still reads the previous block's copy; everybody sees the new one)
    if (layer > 0) __syncthreads();
#pragma unroll
    for (int i = 0; i < SEGV / kPairThreads; ++i) vecl[tid + kPairThreads * i] = ws.cur()[tid + kPairThreads * i];
    __syncthreads();
    ws.advance();
    ws.advance();            // [vec][unused]
    layer_norm_pair(vec + vl.ln1_g(), vec + vl.ln1_b());
    grp oo[NGH], op[NGH];     // attention output of the own tiles / the partner's

#pragma unroll
    for (int i = 0; i < NTH; ++i) {
      const int ft = 2 * i + h;               // the feature tile (= its heads) this wave works on
      // the normalised rows are read again for every feature tile instead of being held through
      // the attention in between (registers: two waves per SIMD have 256 each)
      grp xo[NGH], xp[NGH];
      load_groups(xo, xp);
      f32x16 aq = gemm_tile(bias_tile(vec + vl.bq(), ft, hi), h, xo, xp);
      ws.advance();
      ws.advance();
      f32x16 ak = gemm_tile(splat16(0.f), h, xo, xp);   // no b_K: a per-query constant in the scores, softmax drops it
      ws.advance();
      ws.advance();
      // no b_V (folded into the output bias); operands swapped: lane = feature
      f32x16 av = splat16(0.f);
#pragma unroll
      for (int i2 = 0; i2 < NTH; ++i2)
#pragma unroll
        for (int g = 0; g < GPT; ++g) {
          av = E::mma(xo[i2 * GPT + g], ws.template frag_at<grp>(h, (2 * i2 + h) * GPT + g), av);
          av = E::mma(xp[i2 * GPT + g], ws.template frag_at<grp>(h, (2 * i2 + (h ^ 1)) * GPT + g), av);
        }
      ws.advance();
      ws.advance();

      grp qop[GPT];   // Q carries log2(e) / sqrt(head width): the scores come out ready for exp2
      aq *= p.scale_l2e;
#pragma unroll
      for (int g = 0; g < GPT; ++g) qop[g] = E::pack(aq, g);
      float mrun[HPT], lrun[HPT];
      f32x16 acc[HPT];
#pragma unroll
      for (int hh = 0; hh < HPT; ++hh) { mrun[hh] = kNegBig; lrun[hh] = 0.f; acc[hh] = splat16(0.f); }

      {   // keys of the lane's own tile: the candidate's own globals
        grp kop[GPT], vop[GPT];
#pragma unroll
        for (int g = 0; g < GPT; ++g) { kop[g] = E::pack(ak, g); vop[g] = E::pack(av, g); }
#pragma unroll
        for (int hh = 0; hh < HPT; ++hh) {
          f32x16 S = splat16(0.f);
#pragma unroll
          for (int g2 = 0; g2 < GPH; ++g2) S = E::mma(kop[hh * GPH + g2], qop[hh * GPH + g2], S);
          grp pop[GPT];
          softmax_window<T, W>(S, widx, wmask, tilebits, mrun[hh], lrun[hh], acc[hh], pop);
#pragma unroll
          for (int g = 0; g < GPT; ++g) acc[hh] = E::mma(vop[g], pop[g], acc[hh]);
        }
      }
      {     // stored K/V fragments (wave-uniform user, scalar loop control)
        const int uu = __builtin_amdgcn_readfirstlane(usr);
        const int tuu = __builtin_amdgcn_readfirstlane(Tu);
        const char* kb; const char* vb; int nkt; KeyRanges kr = {};
        if (layer == 0) {
          kb = p.cache + (size_t)uu * p.c0_ustride; vb = kb + p.c0_voff;
          nkt = min(p.kt0, (tuu + 31) / 32); kr.hi2 = tuu;
        } else {
          kb = p.cache + p.c1_off + (size_t)(layer - 1) * p.c1_lstride + (size_t)uu * p.c1_ustride;
          vb = kb + p.c1_voff;
          nkt = tuu > 0 ? p.kt1 : 0; kr.lo2 = first_slot(p.k, tuu, p.q_learn); kr.hi2 = p.k;
        }
        kr.settle_for(valid);
        // the fragments of key tile kt + 1 are requested before tile kt is worked on (d = 128; at
        // d = 256 the registers for that are not there, and the SIMD's other wave covers the latency)
        constexpr bool AHEAD = D < 256;
        grp knx[GPT], vnx[GPT];
        if (AHEAD && nkt > 0) {
          const size_t fo = ((size_t)ft * GPT) * 1024 + lane * 16;
#pragma unroll
          for (int g = 0; g < GPT; ++g) {
            knx[g] = *reinterpret_cast<const grp*>(kb + fo + g * 1024);
            vnx[g] = *reinterpret_cast<const grp*>(vb + fo + g * 1024);
          }
        }
        for (int kt = 0; kt < nkt; ++kt) {
          grp kfr[GPT], vfr[GPT];
          if (AHEAD) {
#pragma unroll
            for (int g = 0; g < GPT; ++g) { kfr[g] = knx[g]; vfr[g] = vnx[g]; }
          } else {
            const size_t fo = ((size_t)(kt * NT + ft) * GPT) * 1024 + lane * 16;
#pragma unroll
            for (int g = 0; g < GPT; ++g) {
              kfr[g] = *reinterpret_cast<const grp*>(kb + fo + g * 1024);
              vfr[g] = *reinterpret_cast<const grp*>(vb + fo + g * 1024);
            }
          }
          if (AHEAD && kt + 1 < nkt) {
            const size_t fo = ((size_t)((kt + 1) * NT + ft) * GPT) * 1024 + lane * 16;
#pragma unroll
            for (int g = 0; g < GPT; ++g) {
              knx[g] = *reinterpret_cast<const grp*>(kb + fo + g * 1024);
              vnx[g] = *reinterpret_cast<const grp*>(vb + fo + g * 1024);
            }
          }
          key_tile_step<HPT, GPH>(kr, kt, kfr, vfr, qop, hi, mrun, lrun, acc);
        }
      }
      // normalise; with two heads per tile each head owns half of the accumulator rows
      f32x16 o;
      float inv[HPT];
#pragma unroll
      for (int hh = 0; hh < HPT; ++hh) inv[hh] = lrun[hh] > 0.f ? __builtin_amdgcn_rcpf(lrun[hh]) : 0.f;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int hh = HPT == 1 ? 0 : r / 8;
        o[r] = acc[hh][r] * inv[hh];
      }
#pragma unroll
      for (int g = 0; g < GPT; ++g) oo[i * GPT + g] = E::pack(o, g);
    }
    swap_groups(oo, op);

    // output projection + residual: own output tiles
#pragma unroll
    for (int i = 0; i < NTH; ++i) {
      resid[i] += bias_tile(vec + vl.bo(), 2 * i + h, hi);
      resid[i] = gemm_tile(resid[i], h, oo, op);
      ws.advance();
      ws.advance();
    }

    // FFN: hidden chunks 2 c2 + h are this wave's; the activated chunks go through the exchange area
    layer_norm_pair(vec + vl.ln2_g(), vec + vl.ln2_b());
    grp xo[NGH], xp[NGH];
    load_groups(xo, xp);
    __syncthreads();          // everybody has its copy: the exchange area is free for the activated chunks
#pragma unroll
    for (int i = 0; i < NTH; ++i) resid[i] += bias_tile(vec + vl.b2(), 2 * i + h, hi);
    if constexpr (!SKEW) {
#pragma unroll 1
      for (int c2 = 0; c2 < NC / 2; ++c2) {
        // panel [w1(2 c2) w1(2 c2 + 1)]: first GEMM + activation of the own chunk
        f32x16 ah = gemm_tile(bias_tile(vec + vl.b1(), 2 * c2 + h, hi), h, xo, xp);
        typename E::hgrp hown[GPT], hoth[GPT];
#pragma unroll
        for (int g = 0; g < GPT; ++g) {
          f16x8 y;     // ah holds x / kFfnScale; to fp16 toward zero, then the packed activation
#pragma unroll
          for (int e = 0; e < E::EPL / 2; ++e) {
            const f16x2 y2 = __builtin_bit_cast(f16x2, __builtin_amdgcn_cvt_pkrtz(ah[E::EPL * g + 2 * e], ah[E::EPL * g + 2 * e + 1]));
            y[2 * e] = y2[0]; y[2 * e + 1] = y2[1];
          }
          hown[g] = RELU ? __builtin_elementwise_max(y, (f16x8)((_Float16)0.f)) : gelu_quarter_h8(y);
          *reinterpret_cast<typename E::hgrp*>(xt + (h * GPT + g) * 64) = hown[g];
        }
        ws.advance();
        ws.advance();          // (the panel switch's barrier also orders the exchange: written above, read below)
#pragma unroll
        for (int g = 0; g < GPT; ++g) hoth[g] = *reinterpret_cast<const typename E::hgrp*>(xt + ((h ^ 1) * GPT + g) * 64);
        // panel [w2(2 c2) w2(2 c2 + 1)]: second GEMM of both chunks for the own output tiles
#pragma unroll
        for (int g = 0; g < GPT; ++g)
#pragma unroll
          for (int i = 0; i < NTH; ++i) {
            resid[i] = E::mma_h(ws.template frag_at<grp>(h, (2 * i + h) * GPT + g), hown[g], resid[i]);
            resid[i] = E::mma_h(ws.template frag_at<grp>(h ^ 1, (2 * i + h) * GPT + g), hoth[g], resid[i]);
          }
        ws.advance();
        ws.advance();          // (its barrier: the partner has read this chunk pair before the next one is written)
      }
    } else {
      // The activation of a chunk goes behind the second products of the pair of chunks before it (both waves of a SIMD are at the same place
      // of the loop: with a chunk's activation between its own products the matrix pipe stood still for it).
      HiddenStages<RELU> act;
      constexpr int NS = HiddenStages<RELU>::kStages, NP = GPT * NS, NM = 2 * GPT * NTH;
      typename E::hgrp hown[GPT], hoth[GPT], hnew[GPT];
      // chunk pairs alternate between two places of the exchange area
      auto hand = [&](int par) {
#pragma unroll
        for (int g = 0; g < GPT; ++g) *reinterpret_cast<typename E::hgrp*>(xt + (par * 2 * GPT + h * GPT + g) * 64) = hown[g];
      };
      auto take = [&](int par) {
#pragma unroll
        for (int g = 0; g < GPT; ++g) hoth[g] = *reinterpret_cast<const typename E::hgrp*>(xt + (par * 2 * GPT + (h ^ 1) * GPT + g) * 64);
      };
      // second GEMM of a pair of chunks for the own output tiles, then(n) behind the n-th product
      auto second = [&](auto then) __attribute__((always_inline)) {
        constexpr int AH = 4;
        auto frag = [&](int q) { return ws.template frag_at<grp>(q & 1 ? h ^ 1 : h, (2 * (q / 2 % NTH) + h) * GPT + q / 2 / NTH); };
        grp fr[AH];
#pragma unroll
        for (int q = 0; q < AH; ++q) fr[q] = frag(q);
#pragma unroll
        for (int q = 0; q < NM; ++q) {
          __builtin_amdgcn_sched_barrier(0);
          const int i = q / 2 % NTH, g = q / 2 / NTH;
          resid[i] = E::mma_h(fr[q % AH], q & 1 ? hoth[g] : hown[g], resid[i]);
          if (q + AH < NM) fr[q % AH] = frag(q + AH);
          then(q);
        }
        __builtin_amdgcn_sched_barrier(0);
      };
      auto first = [&](int c) { return gemm_tile(bias_tile(vec + vl.b1(), 2 * c + h, hi), h, xo, xp); };
      f32x16 ah = first(0);
      ws.advance();
      ws.advance();
#pragma unroll
      for (int k = 0; k < NP; ++k) { const f16x8 y = act.run(ah, k / NS, k % NS); if (k % NS == NS - 1) hown[k / NS] = y; }
      hand(0);
#pragma unroll 1
      for (int c = 0; c + 1 < NC / 2; ++c) {
        ah = first(c + 1);
        ws.advance();
        ws.advance();          // (the panel switch's barrier also orders the exchange: written above, read below)
        take(c & 1);
        second([&](int q) __attribute__((always_inline)) {
#pragma unroll
          for (int k = 0; k < (NP + NM - 1) / NM; ++k) {
            const int at = q * NP / NM + k;
            if (at >= (q + 1) * NP / NM) continue;
            const f16x8 y = act.run(ah, at / NS, at % NS);
            if (at % NS == NS - 1) hnew[at / NS] = y;
          }
        });
#pragma unroll
        for (int g = 0; g < GPT; ++g) hown[g] = hnew[g];
        hand((c & 1) ^ 1);
        ws.advance();
        ws.advance();
      }
      take((NC / 2 - 1) & 1);          // (at least two pairs: FF is a multiple of D; the loop's barriers lie between)
      second([](int) {});
      ws.advance();
      ws.advance();
    }
  }

  wait_vmcnt<0>();   // nothing of the weight stream may still be in flight when the wave ends
  // ------------------------------------------------------------------ epilogue
  if (p.X_out && inrange) store_rows_half<NTH>(resid, p.X_out, p.X_f32, out_off, valid, hi, h);
  if (p.logits) {
    // logit = <head_w, flatten(global rows)> + head_b: each wave sums over its own feature tiles
    const int a = (32 * tile + j) % p.m;       // row inside the head's m rows (lanes per logit)
    float part = 0.f;
    if (valid) {
#pragma unroll
      for (int i = 0; i < NTH; ++i) {
        const f32x16 hw = bias_tile(p.head + (size_t)a * D, 2 * i + h, hi);
#pragma unroll
        for (int r = 0; r < 16; ++r) part += resid[i][r] * hw[r];
      }
    }
    part = sum_halves(part);
    __syncthreads();                       // the LayerNorm sums in `stat` have been read by everybody
    if (hi == 0) stat[ts][h][0][j] = part;
    __syncthreads();
    part = stat[ts][0][0][j] + stat[ts][1][0][j];
    for (int sft = 1; sft < p.m; sft <<= 1) part += __shfl_xor(part, sft, 64);
    part += p.head[(size_t)p.m * D];
    const int cand = (32 * tile + j) / p.m;
    if (h == 0 && hi == 0 && (j % p.m) == 0 && cand < p.C) p.logits[(size_t)usr * p.C + cand] = part;
  }
}

// Host-side launcher, one definition per (D, DH) instantiation file.
template <int D, int DH>
int launch_pair(int win, const BlockParams& p, dim3 grid, hipStream_t stream);

// The skewed FFN (plain order / skewed, microseconds, FFN of one, two, four times the width): width 256, heads of 32, 16 x 300 candidates over 125 groups, GELU 263 / 265,
// 322 / 317, 438 / 422, ReLU 260 / 261, 315 / 313, 425 / 415; heads of 16, two, three, four times, ReLU 347 / 343, 402 / 393, 458 / 445, but GELU 356 / 358, 414 / 418,
// 474 / 478.  Width 128, 16 x 500 candidates, GELU 158 / 161, 175 / 179, 211 / 218, ReLU 156 / 160, 172 / 176, 202 / 211: a panel is half as long there, and finding its place
// in the skewed order and the order held between products cost more than the hidden activation.
template <int D, int DH, int W, bool RELU>
void pair_start(const BlockParams& p, dim3 grid, hipStream_t stream) {
  if constexpr (D == 256 && (DH == 32 || RELU)) {
    if (p.FF > D) { hipLaunchKernelGGL((pair_kernel<D, DH, W, RELU, true>), grid, dim3(kPairThreads), 0, stream, p); return; }
  }
  hipLaunchKernelGGL((pair_kernel<D, DH, W, RELU, false>), grid, dim3(kPairThreads), 0, stream, p);
}

#define LONGER_PAIR_LAUNCH(D, DH, WV) \
  do {                                                                                                \
    if (p.act == 1) pair_start<D, DH, WV, true>(p, grid, stream); else pair_start<D, DH, WV, false>(p, grid, stream); \
  } while (0)

#define LONGER_PAIR_INSTANTIATE(D, DH)                                                                \
  template <>                                                                                         \
  int launch_pair<D, DH>(int win, const BlockParams& p, dim3 grid, hipStream_t stream) {              \
    if (win == 4) LONGER_PAIR_LAUNCH(D, DH, 4);                                                       \
    else if (win == 8) LONGER_PAIR_LAUNCH(D, DH, 8);                                                  \
    else LONGER_PAIR_LAUNCH(D, DH, 16);                                                               \
    return hipGetLastError() == hipSuccess ? 0 : -3;                                                  \
  }

}  // namespace longer
