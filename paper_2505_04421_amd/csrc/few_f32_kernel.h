// The block kernel for small launches in full precision at width 32 (head width 16): a 32-row tile given to four waves.
//
//   MODE_MERGE  the InnerTrans blocks and the mean merge (Section 3.4);
//   MODE_STACK  the whole reduced stack of a user with at most two tiles (Eq. 10); with few merged tokens the cross layer's K and V too.
//
// Why.  A handful of short histories is one or two tiles a user; the launch takes as long as one tile's chain of fp32 products (1024
// cycles each), exact activations and waits for the weight ring.  Here Q, K and V are made by three waves at once, the
// two heads by two, the hidden chunks by four (their contributions summed through LDS, in chunk order); every wave keeps the rows
// themselves, so LayerNorm and the output projection need no exchange and a layer has four barriers.  Weight fragments come from
// L2 into registers a layer ahead.  Forward pass of four users of 64 raw tokens (two layers): 50.6 -> 30.9 us; with the waves of a second tile that has
// no rows gone (they shared the first's matrix pipes) 25.8, of the stack's 15.7 us (37 000 cycles) two layers of five products 16, attention 6.5, the erf 4.6,
// start and first weights 5 thousand.
#pragma once
#include "block_kernel.h"

namespace longer {

constexpr int kFewWaves = 4;
constexpr int few_tiles(int mode) { return mode == MODE_STACK ? 2 : 1; }      // tiles of a workgroup

template <int MODE, int W, bool RELU>
__global__ void __launch_bounds__(64 * kFewWaves * few_tiles(MODE), 1) few_f32_kernel(const BlockParams p) {
  using E = ET<float>;
  using grp = E::grp;
  constexpr int D = 32, TS = few_tiles(MODE), kThr = 64 * kFewWaves * TS;
  constexpr bool STACK = MODE == MODE_STACK;
  static_assert(STACK || MODE == MODE_MERGE, "modes");
  __shared__ grp qkv[TS][3][4][64];                  // per tile: Q, K, V operands [group][lane]
  __shared__ grp ops[TS][4][64];                     // attention output
  __shared__ f32x4 part[TS][kFewWaves][4][64];       // the hidden chunks' contributions
  __shared__ f32x4 vecl[256];                        // the block's fp32 vectors (at most one segment)
  const int tid = threadIdx.x, lane = tid & 63, j = lane & 31, hi = lane >> 5, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ts = wv / kFewWaves, wave = wv % kFewWaves, NC = p.FF / 32;

  // the user and its length: requested first, the weights behind it, and only then waited for
  const bool inline_kv = STACK && p.kst == nullptr;
  int usr = (int)blockIdx.x;
  uint32_t slot = 0;
  bool inrange = true;
  if (!STACK) {
    slot = (uint32_t)blockIdx.x * 32u + (uint32_t)j;
    usr = (int)((slot >> __builtin_ctz(p.K)) / (uint32_t)p.T);
    inrange = usr < p.B;
  }
  int len = p.lens ? p.lens[inrange ? usr : 0] : p.L;

  // ------------------------------------------------------------------ weights: segments of four fragments (layouts: device.h)
  const char* wl = p.wbase;                          // the current block's stream
  bool attn = STACK;                                 // the first block of the stack is the cross layer's attention half: no K, V
  auto request = [&](grp (&f)[4], const char* w, int seg) {
#pragma unroll
    for (int s = 0; s < 4; ++s) f[s] = *reinterpret_cast<const grp*>(w + ((size_t)(seg * 4 + s) * 64 + lane) * 16);
  };
  auto product = [&](f32x16 acc, const grp (&f)[4], const grp (&b)[4]) -> f32x16 {
#pragma unroll
    for (int s = 0; s < 4; ++s) acc = E::mma(f[s], b[s], acc);
    return acc;
  };
  const int role = wave < 3 ? wave : 0;              // Q, K, V (the fourth wave has none of them)
  grp wr[4], wo[4], w1[4], w2[4];
  if (attn && role > 0 && inline_kv) request(wr, p.kv_w, role);
  else request(wr, wl, attn ? 1 : 1 + role);
  request(wo, wl, attn ? 2 : 4);
  const int c0 = wave < NC ? wave : 0;
  request(w1, wl, (attn ? 3 : 5) + 2 * c0);
  request(w2, wl, (attn ? 4 : 6) + 2 * c0);
  const VecLayout vl{D, p.FF};
  const float* vec = reinterpret_cast<const float*>(vecl);
  const int nv = (9 * D + p.FF) / 4;
  f32x4 vq = reinterpret_cast<const f32x4*>(wl)[tid < nv ? tid : 0];

  asm volatile("" ::: "memory");

  // ------------------------------------------------------------------ rows
  len = inrange ? min(max(len, 0), p.L) : 0;
  f32x16 x[1][1], key[1][1];                         // key: the cross layer's key rows (their K and V made here)
  bool valid;
  int tu = 0, nk0 = 0;                               // nk0: keys of the cross layer
  long long out_off = 0;
  uint32_t tilebits = 0;
  KeyRanges kr = {}, skr = {};
  const int widx = W == 16 ? 0 : j / (2 * W);
  uint32_t wmask[16 / W];
#pragma unroll
  for (int w = 0; w < 16 / W; ++w) wmask[w] = widx == w ? 0xffffffffu : 0u;
  if (STACK) {
    const int a = 32 * ts + j;
    inrange = a < p.rows_per_user;
    tu = (len + p.K - 1) / p.K;
    const bool glob = a < p.m;
    const int i = a - p.m, i0 = first_slot(p.k, tu, p.q_learn);
    valid = inrange && (glob || i >= i0);
    out_off = p.X_ustride * usr + (long long)a * D;
    const int tok = glob ? 0 : (p.q_learn ? tu - 1 : slot_token(i, p.k, tu, p.k_uni));
    const int row = glob ? a : (p.gather_recent ? tok : i);
    load_rows<float, 1>(x[0], glob ? p.src0.p : p.src1.p, 1, (glob ? p.src0.ustride : p.src1.ustride) * usr + (long long)row * D, valid, hi);
    key[0][0] = splat16(0.f);
    if (inline_kv) {
      const bool there = glob || i < tu;             // key a: global token, then merged token
      load_rows<float, 1>(key[0], glob ? p.src0.p : p.kv_k, 1, (glob ? p.src0.ustride : (long long)p.T * D) * usr + (long long)(glob ? a : i) * D, there, hi);
    }
    if (glob) { kr.lo1 = skr.lo1 = p.gmask_causal ? a : 0; kr.hi1 = p.KG; skr.hi1 = p.m; }
    kr.lo2 = p.KG; kr.hi2 = p.KG + (glob ? tu : tok + 1);
    skr.lo2 = p.m + i0; skr.hi2 = p.m + (glob ? p.k : i + 1);
    kr.settle_for(valid); skr.settle_for(valid);
    nk0 = __builtin_amdgcn_readfirstlane(p.KG + tu);
    // a second tile without rows or keys: its waves leave the matrix pipes to the first's (a barrier waits for those still there only)
    if (ts > 0 && p.rows_per_user <= 32 && !(inline_kv && nk0 > 32)) return;
  } else {
    const uint32_t gidx = slot >> __builtin_ctz(p.K);
    const int pos = (int)(gidx - (uint32_t)usr * (uint32_t)p.T) * p.K + (int)(slot & (uint32_t)(p.K - 1));
    tu = len;                                        // (the raw length here)
    valid = inrange && pos < len;
    load_rows<float, 1>(x[0], p.H, 1, ((long long)usr * p.L + pos) * D, valid, hi);
    const uint32_t vb = (uint32_t)__ballot(valid);
    const uint32_t gb = (p.K >= 32 ? 0xffffffffu : ((1u << p.K) - 1u)) << (p.K * (j / p.K));
    tilebits = ((gb & vb) >> (4 * hi)) >> (2 * W * widx);
    if (vb == 0) {                                   // nothing but padding
      if (wave == 0 && inrange && (slot & (uint32_t)(p.K - 1)) == 0) store_rows<float, 1>(x[0], p.M_out, 1, (long long)gidx * D, false, hi);
      return;
    }
  }

  for (int layer = 0; layer < p.n_layers; ++layer) {
    const bool selfl = STACK && layer > 0, last = layer + 1 == p.n_layers;
    const char* wnext = last ? wl : wl + (size_t)((attn ? 4 : 6) + 2 * NC) * 4096;     // (after the last block: requests that nobody waits for)
    if (tid < 256) vecl[tid] = vq;                   // (last read ahead of the FFN's barrier)
    __syncthreads();
    vq = reinterpret_cast<const f32x4*>(wnext)[tid < nv ? tid : 0];
    grp xn[1][4];
    {
      f32x16 rows[1][1];
      rows[0][0] = layer == 0 && inline_kv && role > 0 ? key[0][0] : x[0][0];
      layer_norm<float, D, 1>(rows, vec + vl.ln1_g(), vec + vl.ln1_b(), p.eps, hi, xn);
    }
    {
      f32x16 a;
      if (role == 0) a = product(bias_tile(vec + vl.bq(), 0, hi), wr, xn[0]);
      else if (role == 1) a = product(splat16(0.f), wr, xn[0]);      // no b_K, no b_V: see block_kernel.h
      else a = product(splat16(0.f), xn[0], wr);     // operands swapped: lane = feature
      settle(a);
      if (role == 0) a *= p.scale_l2e;
      if (wave < 3) {
#pragma unroll
        for (int g = 0; g < 4; ++g) qkv[ts][wave][g][lane] = E::pack(a, g);
      }
      request(wr, wnext, 1 + role);                  // (every block after the first is in the fused layout)
    }
    __syncthreads();
    if (STACK && ts > 0 && p.rows_per_user <= 32) return;      // (it had keys only)
    if (wave < 2) {                                  // a head each
      const int h = wave;
      const grp q[2] = {qkv[ts][0][2 * h][lane], qkv[ts][0][2 * h + 1][lane]};
      float mrun = kNegBig, lrun = 0.f;
      f32x16 acc = splat16(0.f);
      auto keys = [&](f32x16 S, const grp (&k)[2]) -> f32x16 {
#pragma unroll
        for (int g = 0; g < 2; ++g) S = E::mma(k[g], q[g], S);
        return S;
      };
      auto values = [&](const grp (&v)[4], const grp (&pop)[4], int n) {      // (the first n keys: the others' weights are zeros)
#pragma unroll
        for (int g = 0; g < 4; ++g)
          if (g == 0 || 8 * g < n) acc = E::mma(v[g], pop[g], acc);
      };
      auto tile_of = [&](const KeyRanges& r, int n, int kt, const grp (&k)[2], const grp (&v)[4]) {
        const uint32_t ab = ((range_bits(r.lo1, r.hi1, 32 * kt) | range_bits(r.lo2, r.hi2, 32 * kt)) >> (4 * hi)) & kTileBits;
        f32x16 S = keys(mask_tile(ab), k);
        grp pop[4];
        softmax_step<float, false>(S, 0u, mrun, lrun, acc, pop);
        values(v, pop, n - 32 * kt);
      };
      if (!STACK) {
        const grp k[2] = {qkv[ts][1][2 * h][lane], qkv[ts][1][2 * h + 1][lane]};
        const grp v[4] = {qkv[ts][2][0][lane], qkv[ts][2][1][lane], qkv[ts][2][2][lane], qkv[ts][2][3][lane]};
        const f32x16 S = keys(splat16(0.f), k);
        grp pop[4];
        softmax_window<float, W>(S, widx, wmask, tilebits, mrun, lrun, acc, pop);
        values(v, pop, 32);
      } else if (selfl || inline_kv) {
        const int n = selfl ? p.rows_per_user : nk0;
        for (int kt = 0; 32 * kt < n; ++kt) {
          const grp k[2] = {qkv[kt][1][2 * h][lane], qkv[kt][1][2 * h + 1][lane]};
          const grp v[4] = {qkv[kt][2][0][lane], qkv[kt][2][1][lane], qkv[kt][2][2][lane], qkv[kt][2][3][lane]};
          tile_of(selfl ? skr : kr, n, kt, k, v);
        }
      } else {                                       // stored K / V fragments, the next tile's on their way
        const char* kb = p.kst + (size_t)usr * p.kv_ustride;
        const char* vb = p.vst + (size_t)usr * p.kv_ustride;
        grp kn[2], vn[4];
        auto fetch = [&](int kt) {
          const size_t fo = (size_t)kt * 4096 + lane * 16;
#pragma unroll
          for (int g = 0; g < 2; ++g) kn[g] = *reinterpret_cast<const grp*>(kb + fo + (2 * h + g) * 1024);
#pragma unroll
          for (int g = 0; g < 4; ++g) vn[g] = *reinterpret_cast<const grp*>(vb + fo + g * 1024);
        };
        if (nk0 > 0) fetch(0);
        for (int kt = 0; 32 * kt < nk0; ++kt) {
          const grp k[2] = {kn[0], kn[1]}, v[4] = {vn[0], vn[1], vn[2], vn[3]};
          if (32 * (kt + 1) < nk0) fetch(kt + 1);
          tile_of(kr, nk0, kt, k, v);
        }
      }
      settle(acc);
      const float inv = lrun > 0.f ? 1.0f / lrun : 0.f;
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        grp o;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float lo = acc[4 * g + e], up = acc[8 + 4 * g + e];
          o[e] = (h ? up : lo) * inv;
        }
        ops[ts][2 * h + g][lane] = o;
      }
    }
    __syncthreads();
    {
      const grp o[4] = {ops[ts][0][lane], ops[ts][1][lane], ops[ts][2][lane], ops[ts][3][lane]};
      x[0][0] = product(x[0][0] + bias_tile(vec + vl.bo(), 0, hi), wo, o);
      settle(x[0][0]);
      request(wo, wnext, 4);
    }
    layer_norm<float, D, 1>(x, vec + vl.ln2_g(), vec + vl.ln2_b(), p.eps, hi, xn);
    f32x16 sum = splat16(0.f);
    const int ffn = attn ? 3 : 5;
    for (int c = wave; c < NC; c += kFewWaves) {
      f32x16 ah = product(bias_tile(vec + vl.b1(), c, hi), w1, xn[0]);
      settle(ah);
      const bool more = c + kFewWaves < NC;
      request(w1, more ? wl : wnext, more ? ffn + 2 * (c + kFewWaves) : 5 + 2 * wave);
      grp hop[4];
#pragma unroll
      for (int r = 0; r < 16; ++r) ah[r] = RELU ? fmaxf(ah[r], 0.f) : gelu_fn<true>(ah[r]);
#pragma unroll
      for (int g = 0; g < 4; ++g) hop[g] = E::pack(ah, g);
      sum = product(sum, w2, hop);
      request(w2, more ? wl : wnext, more ? ffn + 2 * (c + kFewWaves) + 1 : 6 + 2 * wave);
    }
    settle(sum);
#pragma unroll
    for (int q = 0; q < 4; ++q) part[ts][wave][q][lane] = E::pack(sum, q);
    x[0][0] += bias_tile(vec + vl.b2(), 0, hi);
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kFewWaves; ++w)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f32x4 v = part[ts][w][q][lane];
#pragma unroll
        for (int e = 0; e < 4; ++e) x[0][0][4 * q + e] += v[e];
      }
    wl = wnext;
    attn = false;
  }

  // ------------------------------------------------------------------ epilogue: every wave has the rows
  if (wave > 0) return;
  if (STACK) {
    if (p.X_out && inrange) store_rows<float, 1>(x[0], p.X_out, 1, out_off, valid, hi);
    if (p.logits && ts == 0) {       // logit = <head_w, flatten(global rows)> + head_b (m <= 32: all in the first tile)
      float sum = 0.f;
      if (j < p.m) {
        const f32x16 hw = bias_tile(p.head + (size_t)j * D, 0, hi);
#pragma unroll
        for (int r = 0; r < 16; ++r) sum += x[0][0][r] * hw[r];
      }
      sum = sum_halves(sum);
      for (int sft = 1; sft < 32; sft <<= 1) sum += __shfl_xor(sum, sft, 64);
      if (lane == 0) p.logits[usr] = sum + p.head[(size_t)p.m * D];
    }
  } else {                           // mean over a group's valid tokens, on K adjacent lanes (as in block_kernel.h)
    const uint32_t gidx = slot >> __builtin_ctz(p.K);
    const int t = (int)(gidx % (uint32_t)p.T), n = min(max(tu - t * p.K, 0), p.K);
    x[0][0] *= valid ? 1.0f / (float)n : 0.f;
    if (p.K >= 2) lane_sum<0xB1, 1>(x[0]);
    if (p.K >= 4) lane_sum<0x4E, 1>(x[0]);
    if (p.K >= 8) lane_sum<0x141, 1>(x[0]);
    if (p.K >= 16) lane_sum<0x140, 1>(x[0]);
    if (p.K >= 32) {
#pragma unroll
      for (int r = 0; r < 16; ++r) x[0][0][r] += __shfl_xor(x[0][0][r], 16, 64);
    }
    if (inrange && (slot & (uint32_t)(p.K - 1)) == 0) store_rows<float, 1>(x[0], p.M_out, 1, (long long)gidx * D, true, hi);
  }
}

int launch_few_f32(int mode, int win, const BlockParams& p, dim3 grid, hipStream_t stream);

}  // namespace longer
