// Token merge and input generation, bf16, d = 64 and 128 (the block kernel's modes of the same names, same packed streams, same results):
//
//   MODE_MERGE       K-groups of raw tokens through the InnerTrans blocks, mean of each group (Section 3.4);
//   MODE_MERGE_KEEP  the same, every later block's input rows written as well (a training step's merge);
//   MODE_MERGE_IN    the same from the raw inputs: the input MLP (Section 3.5.1) is the pass in front of the blocks;
//   MODE_INPUT       the input MLP alone.
//
// A wave owns 32 tokens in registers and streams the weights through LDS (device.h).  What bounds it is the issue of matrix and
// vector instructions under the chip's power limit (the shader clock is 1.7 to 1.9 GHz here), so the wave must not wait as well: one that had
// the SIMD to itself took (d = 128) 74 cycles per MFMA of the FFN (32 are the pipe's); of those the fragment reads behind each barrier, the
// barriers and the burst of eight load-to-LDS instructions per panel were 36.  Here a panel is one step of the FFN (two segments, 16 KiB) in a ring of four; a
// panel is known to have landed one barrier before its use, so that a segment's first fragments are read under the last products of the
// one before, and the loads of the panel three ahead go out one by one behind products.  FFN loop alone, two workgroups a compute unit: 702 ->
// 633 ns per pair of segments; a wave's life in the merge of two blocks 100.8k -> 93.4k cycles (alone on its SIMD 80.6k -> 73.6k).  Whole passes: 256 users of 2000
// tokens, two blocks 559 -> 543 us, 512 of at most 5000, one block 858 -> 831, 61 of 1501 from the raw inputs 183 -> 176.  Width 64 (three workgroups a
// compute unit): 128 users of 512 tokens 43.4 -> 42.6, 512 of 4000, two blocks 687 -> 681.
#pragma once
#include "block_kernel.h"

namespace longer {

// The weight stream, 256 threads.  A piece is 4 KiB: every thread loads 16 bytes of it straight into LDS.  Pieces go out in stream
// order, two panels and more ahead of their use, always SEGV / 256 a segment; past the stream's end the last one is read again.
// A piece of panel q + 3 goes out while panel q is in use, into the place of panel q - 1, which every wave has left at the last barrier.
// The barrier in front of panel q has seen all but this wave's youngest panel land: q and q + 1 are whole.  (Loads return in
// order, so "at most one panel's loads outstanding" proves that; other loads and stores can only make the wait longer.)
template <int SEGV>
struct FlowStream {
  static constexpr unsigned kSeg = SEGV * 16, kPanel = 2 * kSeg, kRing = 4 * kPanel;
  static constexpr int kPieces = SEGV / 256;         // per segment
  static constexpr int kAhead = 4;                   // fragments a wave may have requested from the next panel when it leaves one
  static_assert(SEGV % 256 == 0, "segments in whole pieces");
  const char* lds; const char* g;
  unsigned off, last, lane_off, dst, wr, cur;        // next piece: byte in the stream, in the ring; cur: the current panel
  int lane;
  __device__ __forceinline__ void piece() {
    gload_lds16(g + off, lane_off, dst + wr);
    off = min(off + 4096u, last);
    wr = (wr + 4096u) & (kRing - 1);
  }
  __device__ __forceinline__ void init(const void* lds_, const void* gbase, int segments) {
    const int tid = threadIdx.x;
    lds = reinterpret_cast<const char*>(lds_); g = reinterpret_cast<const char*>(gbase);
    lane = tid & 63; lane_off = (unsigned)tid * 16u;
    dst = __builtin_amdgcn_readfirstlane((unsigned)(unsigned long long)lds_ + (unsigned)(tid >> 6) * 1024u);
    off = wr = cur = 0; last = (unsigned)segments * kSeg - 4096u;
#pragma unroll
    for (int i = 0; i < 6 * kPieces; ++i) piece();
    next_panel();
    cur = 0;
  }
  // every wave is done with the current panel; the next one and the one after are whole.  (LDS answers in order: all but the
  // youngest requests, which are of the next panel, have been answered.)
  __device__ __forceinline__ void next_panel() {
    __builtin_amdgcn_sched_barrier(0);
    wait_vmcnt<2 * kPieces>();
    asm volatile("s_waitcnt lgkmcnt(%0)\n\ts_barrier" :: "n"(kAhead) : "memory");
    __builtin_amdgcn_sched_barrier(0);
    cur = (cur + kPanel) & (kRing - 1);
  }
  // fragment f of segment s (0, 1) of the current panel, of the one behind it
  __device__ __forceinline__ bf16x8 frag(int s, int f) const { return *reinterpret_cast<const bf16x8*>(lds + cur + lane * 16 + s * kSeg + f * 1024); }
  __device__ __forceinline__ unsigned behind() const { return (cur + kPanel) & (kRing - 1); }
  __device__ __forceinline__ bf16x8 frag_behind(unsigned byte) const { return *reinterpret_cast<const bf16x8*>(lds + behind() + lane * 16 + byte); }
};

template <int D, int DH, int MODE, int W, bool RELU>
__global__ void __launch_bounds__(256, D == 64 ? 3 : 2) merge_kernel(const BlockParams p) {
  typedef __bf16 T;
  using E = ET<T>;
  using grp = E::grp;
  constexpr int NT = D / 32, NG = D / 16, GPT = 2, SEGV = NG * 64, HPT = 32 / DH, GPH = DH / 16;
  constexpr bool MERGE = MODE != MODE_INPUT, FROM_IN = MODE == MODE_MERGE_IN || MODE == MODE_INPUT;
  constexpr int AH = FlowStream<SEGV>::kAhead;
  static_assert(NG % AH == 0, "the ring of fragments turns whole times per segment");
  __shared__ uint4 lds[8 * SEGV];
  __shared__ uint4 vecl[SEGV];               // the block's fp32 vectors
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, j = lane & 31, hi = lane >> 5;
  const int NC = p.FF / 32;                  // even

  // ------------------------------------------------------------------ rows of this wave
  const int tile = (int)blockIdx.x * 4 + wave;
  const uint32_t slot = (uint32_t)tile * 32u + (uint32_t)j;      // below 2^31 (the launcher)
  int u, pos, len = 0;
  if (MERGE) {       // K divides 32, so it is a power of two
    const uint32_t gidx = slot >> __builtin_ctz(p.K);
    u = (int)(gidx / (uint32_t)p.T);
    pos = (int)(gidx - (uint32_t)u * (uint32_t)p.T) * p.K + (int)(slot & (uint32_t)(p.K - 1));
  } else {
    u = (int)(slot / (uint32_t)p.L);
    pos = (int)(slot - (uint32_t)u * (uint32_t)p.L);
  }
  const bool inrange = u < p.B;
  if (inrange) { len = p.lens ? p.lens[u] : p.L; len = min(max(len, 0), p.L); }
  const bool valid = inrange && pos < len;

  // A workgroup whose tokens are all padding writes zeros and leaves.  Without `lens` there is none.  Raw tokens, workgroups that follow one another: before any row is asked
  // for (half of the workgroups of users of 100 to 5000 tokens; asked behind the row requests, and with a group's zeros from one lane a row: 512 such users, one block
  // 659 / 645 us, two blocks 1145 / 1130, 128 of them 171 / 165, 2000 users of at most 600 tokens 376 / 371, width 64 314 / 310).  Where all workgroups start at once the barrier
  // ahead of the requests is time lost (59 users of at most 218 tokens 59.4 / 59.8 us a pass), and so from the inputs, whose requests have arithmetic in front of
  // them (100 users of 2000 tokens, width 64: 54.3 / 54.8).
  const bool ask_first = !FROM_IN && gridDim.x > (D == 64 ? 768u : 512u);
  auto all_padding = [&]() {
    if (__syncthreads_or(valid ? 1 : 0)) return false;
    const uint32_t slot0 = (uint32_t)blockIdx.x * 128u;
    auto zeros = [&](void* out, int is_f32, uint32_t row0, uint32_t rows, long long all) {       // rows row0 .. row0 + rows - 1 of `all`
      const long long end = min((long long)row0 + rows, all) * D;
      for (long long i = (long long)row0 * D + 4 * tid; i < end; i += 4 * 256) {
        if (is_f32) *(f32x4*)(reinterpret_cast<float*>(out) + i) = f32x4{0.f, 0.f, 0.f, 0.f};
        else *(uint2*)(reinterpret_cast<__bf16*>(out) + i) = make_uint2(0u, 0u);
      }
    };
    const int kl = __builtin_ctz(p.K);
    const long long groups = (long long)p.B * p.T;
    if (p.Z_out) zeros(p.Z_out, p.Z_f32, slot0, 128u, groups << kl);
    if (p.M_out) zeros(p.M_out, p.M_f32, slot0 >> kl, 128u >> kl, groups);
    return true;
  };
  if constexpr (!FROM_IN) { if (ask_first && p.lens && all_padding()) return; }

  const int widx = W == 16 ? 0 : j / (2 * W);
  uint32_t wmask[16 / W];
#pragma unroll
  for (int w = 0; w < 16 / W; ++w) { wmask[w] = widx == w ? 0xffffffffu : 0u; asm("" : "+v"(wmask[w])); }
  f32x16 resid[NT];
  const long long row = (long long)u * p.L + pos;
  if (FROM_IN) input_rows<T, NT>(resid, p, row, pos, valid, hi);
  else load_rows<T, NT>(resid, p.H, 0, row * D, valid, hi);
  uint32_t tilebits = 0;                     // keys of the lane's group, as bits of its window
  if (MERGE) {
    const uint32_t vb = (uint32_t)__ballot(valid);
    const uint32_t gb = (p.K >= 32 ? 0xffffffffu : ((1u << p.K) - 1u)) << (p.K * (j / p.K));
    tilebits = ((gb & vb) >> (4 * hi)) >> (2 * W * widx);
  }

  if (!ask_first && p.lens && !__syncthreads_or(valid ? 1 : 0)) {      // (zeros from the lanes that have the rows: shorter, and one round does not wait for them)
    if (inrange) {
      if (MODE == MODE_INPUT) store_rows<T, NT>(resid, p.X_out, 0, (long long)slot * D, false, hi);
      else {
        if (p.Z_out) store_rows<T, NT>(resid, p.Z_out, p.Z_f32, (long long)slot * D, false, hi);
        if (p.M_out && (slot & (uint32_t)(p.K - 1)) == 0)
          store_rows<T, NT>(resid, p.M_out, p.M_f32, (long long)(slot >> __builtin_ctz(p.K)) * D, false, hi);
      }
    }
    return;
  }

  const int block_segs = 2 + 4 * NT + 2 * NC, mlp_segments = 2 + 2 * NC;
  FlowStream<SEGV> ws;
  ws.init(lds, p.wbase, MODE == MODE_INPUT ? mlp_segments : (FROM_IN ? mlp_segments + (p.n_layers - 1) * block_segs : p.n_layers * block_segs));
  const float* vec = reinterpret_cast<const float*>(vecl);
  const VecLayout vl{D, p.FF};
  // the vectors of a block: segment 0 of the panel at `at`
  auto take_vectors = [&](unsigned at) {
#pragma unroll
    for (int i = 0; i < SEGV / 256; ++i) vecl[tid + 256 * i] = *reinterpret_cast<const uint4*>(ws.lds + at + (tid + 256 * i) * 16);
  };
  take_vectors(0);
  __syncthreads();

  grp fr[AH];                                // the weight fragments on their way
  auto keep_order = [] { __builtin_amdgcn_sched_barrier(0); };
  // one segment (place S of the panel) of NG products, use(s, fragment s); its pieces of the stream go out on the way.  The fragments
  // behind it are requested as its last products are issued: what(n, request) names the n-th, or nothing.
  auto segment = [&](auto s_, auto&& use, auto&& follow) {
    constexpr int S = decltype(s_)::value;
#pragma unroll
    for (int s = 0; s < NG; ++s) {
      __builtin_amdgcn_sched_barrier(0x6);
      use(s, fr[s % AH]);
      if (s + AH < NG) fr[s % AH] = ws.frag(S, s + AH);
      else follow(s + AH - NG);
      if ((s & 1) && s / 2 < FlowStream<SEGV>::kPieces) ws.piece();
    }
    keep_order();
    if constexpr (S == 1) ws.next_panel();
  };
  using std::integral_constant;
  typedef integral_constant<int, 0> I0; typedef integral_constant<int, 1> I1;
  typedef integral_constant<bool, true> Yes; typedef integral_constant<bool, false> No;
  // what follows: the next segment in order (place 0: the same panel's, place 1: the next panel's)
  auto then0 = [&](int n) { fr[n] = ws.frag(1, n); };
  auto then1 = [&](int n) { fr[n] = ws.frag_behind(n * 1024); };
  auto nothing = [](int) {};
#pragma unroll
  for (int n = 0; n < AH; ++n) fr[n] = ws.frag(1, n);

  for (int layer = 0; layer < p.n_layers; ++layer) {
#pragma unroll
    for (int i = 0; i < FlowStream<SEGV>::kPieces; ++i) ws.piece();         // those of the vectors' segment
    if constexpr (MODE == MODE_MERGE_KEEP) {
      if (layer > 0 && inrange) store_rows<T, NT>(resid, reinterpret_cast<float*>(p.X_out) + (size_t)(layer - 1) * p.X_ustride, 1, (long long)slot * D, valid, hi);
    }
    grp xn[1][NG];
    f32x16 (&rr)[1][NT] = reinterpret_cast<f32x16 (&)[1][NT]>(resid);
    // input generation: no norm, no attention, no residual; the rows themselves are the first product's operand
    if (FROM_IN && layer == 0) {
#pragma unroll
      for (int t = 0; t < NT; ++t) {
#pragma unroll
        for (int g = 0; g < GPT; ++g) xn[0][t * GPT + g] = E::pack(resid[t], g);
        resid[t] = splat16(0.f);
      }
    } else if constexpr (MERGE) {
      layer_norm<T, D, 1>(rr, vec + vl.ln1_g(), vec + vl.ln1_b(), p.eps, hi, xn);
      grp oop[NG];
      // Q, K, V of feature tile ft are segments 1 + 3 ft ..: place 1, 0, 1 of their panels for even ft, 0, 1, 0 for odd ones
      auto heads = [&](auto par_, int ft) {
        constexpr bool ODD = decltype(par_)::value == 1;
        typedef integral_constant<int, ODD ? 0 : 1> A;
        typedef integral_constant<int, ODD ? 1 : 0> Bp;
        f32x16 aq = bias_tile(vec + vl.bq(), ft, hi), ak = splat16(0.f), av = splat16(0.f);   // (b_K and b_V: block_kernel.h)
        auto q_use = [&](int s, const grp w) { aq = E::mma(w, xn[0][s], aq); };
        auto k_use = [&](int s, const grp w) { ak = E::mma(w, xn[0][s], ak); };
        auto v_use = [&](int s, const grp w) { av = E::mma(xn[0][s], w, av); };
        if constexpr (ODD) { segment(A{}, q_use, then0); segment(Bp{}, k_use, then1); segment(A{}, v_use, nothing); }
        else { segment(A{}, q_use, then1); segment(Bp{}, k_use, then0); segment(A{}, v_use, nothing); }
        grp qop[GPT], kop[GPT], vop[GPT];
        aq *= p.scale_l2e;
#pragma unroll
        for (int g = 0; g < GPT; ++g) { qop[g] = E::pack(aq, g); kop[g] = E::pack(ak, g); vop[g] = E::pack(av, g); }
        float lrun[HPT];
        f32x16 acc[HPT];
#pragma unroll
        for (int hh = 0; hh < HPT; ++hh) {
          f32x16 S = splat16(0.f);
#pragma unroll
          for (int g2 = 0; g2 < GPH; ++g2) S = E::mma(kop[hh * GPH + g2], qop[hh * GPH + g2], S);
          grp pop[GPT];
          float mrun = kNegBig;
          lrun[hh] = 0.f; acc[hh] = splat16(0.f);
          softmax_window<T, W>(S, widx, wmask, tilebits, mrun, lrun[hh], acc[hh], pop);
#pragma unroll
          for (int g = 0; g < GPT; ++g) acc[hh] = E::mma(vop[g], pop[g], acc[hh]);
        }
        // the next segment's first fragments: its place is 1 behind an odd tile's V (place 0), 0 of the panel that next_panel() has just brought else
#pragma unroll
        for (int n = 0; n < AH; ++n) fr[n] = ws.frag(ODD ? 1 : 0, n);
        f32x16 o;       // with two heads per tile each owns half of the accumulator rows
        float inv[HPT];
#pragma unroll
        for (int hh = 0; hh < HPT; ++hh) inv[hh] = lrun[hh] > 0.f ? __builtin_amdgcn_rcpf(lrun[hh]) : 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) { const int hh = HPT == 1 ? 0 : r / 8; o[r] = acc[hh][r] * inv[hh]; }
#pragma unroll
        for (int g = 0; g < GPT; ++g) oop[ft * GPT + g] = E::pack(o, g);
      };
#pragma unroll
      for (int f2 = 0; f2 < NT / 2; ++f2) { heads(I0{}, 2 * f2); heads(I1{}, 2 * f2 + 1); }
      // output projection and residual: segments 1 + 3 NT .., place 1 first
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        resid[nt] += bias_tile(vec + vl.bo(), nt, hi);
        auto o_use = [&](int s, const grp w) { resid[nt] = E::mma(w, oop[s], resid[nt]); };
        if (nt & 1) segment(I0{}, o_use, then0); else segment(I1{}, o_use, then1);
      }
      layer_norm<T, D, 1>(rr, vec + vl.ln2_g(), vec + vl.ln2_b(), p.eps, hi, xn);
    }
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) resid[nt] += bias_tile(vec + vl.b2(), nt, hi);

    // FFN, software pipelined over its hidden chunks as in block_kernel.h: under the products of the second GEMM of chunk i - 1 and the first
    // of chunk i + 1, which alternate, the activation of chunk i, a stage behind each
    f32x16 ah[2];
    E::hgrp hop[2][GPT];
    constexpr int NS = RELU ? 2 : 8;          // stages of one operand group's activation
    constexpr int NP = GPT * NS;              // stages of a chunk
    f16x8 ay, av, ap;
    auto pin = [&](f16x8& x) {
      u32x4 t = __builtin_bit_cast(u32x4, x);
      asm volatile("" : "+v"(t));
      x = __builtin_bit_cast(f16x8, t);
    };
    auto act_stage = [&](const f32x16& a, int gg, int st, E::hgrp& out) {
      if (st == 0) {          // pairs of elements to fp16 (toward zero: never to infinity)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float lo = a[8 * gg + 2 * e], up = a[8 * gg + 2 * e + 1];
          asm volatile("" : "+v"(lo), "+v"(up));
          const f16x2 y2 = __builtin_bit_cast(f16x2, __builtin_amdgcn_cvt_pkrtz(lo, up));
          ay[2 * e] = y2[0]; ay[2 * e + 1] = y2[1];
        }
        return;
      }
      if (st == 1 || RELU) pin(ay); else if (st == 2) pin(av); else pin(ap);
      if (RELU) out = __builtin_elementwise_max(ay, (f16x8)((_Float16)0.f));
      else if (st == 1) av = ay * ay;
      else if (st == 2) ap = __builtin_elementwise_fma((f16x8)((_Float16)2.4554419175668456f), av, (f16x8)((_Float16)-6.304095499217479f));
      else if (st == 3) ap = __builtin_elementwise_fma(ap, av, (f16x8)((_Float16)6.604333663059149f));
      else if (st == 4) ap = __builtin_elementwise_fma(ap, av, (f16x8)((_Float16)-3.771901897714043f));
      else if (st == 5) ap = __builtin_elementwise_fma(ap, av, (f16x8)((_Float16)1.5736394077430096f));
      else if (st == 6) {
        ap = __builtin_elementwise_fma(ay, ap, (f16x8)((_Float16)0.5f));
        ap = __builtin_elementwise_min(__builtin_elementwise_max(ap, (f16x8)((_Float16)0.f)), (f16x8)((_Float16)1.f));
      } else out = ay * ap;
    };
    auto w2_frag = [](int jj) { return (jj % NT) * GPT + jj / NT; };      // product jj of a second GEMM: output tile jj % NT, operand group jj / NT
    // the first requests of a panel {W2, W1} that is the current one's successor; of the last one {W2(NC-2), W2(NC-1)}
    constexpr unsigned kSeg = FlowStream<SEGV>::kSeg;
    auto then_pair = [&](int n, bool tail) {
      const unsigned a = n & 1 ? kSeg + (n / 2) * 1024 : w2_frag(n / 2) * 1024, b = w2_frag(n) * 1024;
      fr[n] = ws.frag_behind(a == b ? a : tail ? b : a);
    };
    ah[0] = bias_tile(vec + vl.b1(), 0, hi);
    segment(I1{}, [&](int s, const grp w) { ah[0] = E::mma(w, xn[0][s], ah[0]); }, then1);          // {.., W1(0)}
    ah[1] = bias_tile(vec + vl.b1(), 1, hi);
    // {W1(1), unused}: the first GEMM of chunk 1, the activation of chunk 0
#pragma unroll
    for (int q = 0; q < NG; ++q) {
      keep_order();
      ah[1] = E::mma(fr[q % AH], xn[0][q], ah[1]);
      if (q + AH < NG) fr[q % AH] = ws.frag(0, q + AH);
      else then_pair(q + AH - NG, NC == 2);
      if (q & 1) { if (q / 2 < 2 * FlowStream<SEGV>::kPieces) ws.piece(); }
#pragma unroll
      for (int pc = q * NP / NG; pc < (q + 1) * NP / NG; ++pc) act_stage(ah[0], pc / NS, pc % NS, hop[0][pc / NS]);
    }
    ah[0] = bias_tile(vec + vl.b1(), min(2, NC - 1), hi);
    ws.next_panel();
    // {W2(i-1), W1(i+1)} with the activation of chunk i, PA = i & 1
    auto step = [&](auto pa_, int i) {
      constexpr int PA = decltype(pa_)::value, PB = PA ^ 1, NM = 2 * NG;
#pragma unroll
      for (int q = 0; q < NM; ++q) {
        keep_order();
        const int jj = q / 2;
        if ((q & 1) == 0) resid[jj % NT] = E::mma_h(fr[q % AH], hop[PB][jj / NT], resid[jj % NT]);
        else ah[PB] = E::mma(fr[q % AH], xn[0][jj], ah[PB]);
        if (q + AH < NM) { const int q2 = q + AH, j2 = q2 / 2; fr[q % AH] = (q2 & 1) == 0 ? ws.frag(0, w2_frag(j2)) : ws.frag(1, j2); }
        else then_pair(q + AH - NM, i == NC - 2);
        if ((q & 1) && q / 2 < 2 * FlowStream<SEGV>::kPieces) ws.piece();
#pragma unroll
        for (int pc = q * NP / NM; pc < (q + 1) * NP / NM; ++pc) act_stage(ah[PA], pc / NS, pc % NS, hop[PA][pc / NS]);
        if (q == NM - (NG > 4 ? 4 : 2)) ah[PA] = bias_tile(vec + vl.b1(), min(i + 2, NC - 1), hi);      // chunk i + 2 starts from its bias (chunk i's values are taken)
      }
      ws.next_panel();
    };
#pragma unroll 1
    for (int i = 1; i + 1 <= NC - 2; i += 2) { step(I1{}, i); step(I0{}, i + 1); }
    // {W2(NC-2), W2(NC-1)}: the activation of chunk NC - 1 (odd) under the first half
    if (layer + 1 < p.n_layers) take_vectors(ws.behind());      // nobody reads this block's any more
#pragma unroll
    for (int q = 0; q < 2 * NG; ++q) {
      keep_order();
      const int jj = q % NG;
      resid[jj % NT] = E::mma_h(fr[q % AH], hop[q < NG ? 0 : 1][jj / NT], resid[jj % NT]);
      if (q + AH < 2 * NG) { const int q2 = q + AH; fr[q % AH] = ws.frag(q2 / NG, w2_frag(q2 % NG)); }
      else fr[q % AH] = ws.frag_behind(kSeg + (q + AH - 2 * NG) * 1024);      // behind the next block's vectors
      if ((q & 1) && q / 2 < 2 * FlowStream<SEGV>::kPieces) ws.piece();
      if (q < NG) {
#pragma unroll
        for (int pc = q * NP / NG; pc < (q + 1) * NP / NG; ++pc) act_stage(ah[1], pc / NS, pc % NS, hop[1][pc / NS]);
      }
    }
    ws.next_panel();
  }

  wait_vmcnt<0>();   // nothing of the weight stream may still be in flight when the wave ends
  // ------------------------------------------------------------------ results
  if constexpr (MODE == MODE_INPUT) {
    if (inrange) store_rows<T, NT>(resid, p.X_out, 0, (long long)slot * D, valid, hi);
  } else {
    if (p.Z_out && inrange) store_rows<T, NT>(resid, p.Z_out, p.Z_f32, (long long)slot * D, valid, hi);
    if (p.M_out) {
      // mean over the valid tokens of each group: tokens of a group sit on K adjacent lanes
      const uint32_t gidx = slot >> __builtin_ctz(p.K);
      const int t0 = pos & ~(p.K - 1), nv = min(max(len - t0, 0), p.K);
      const float wgt = valid ? 1.0f / (float)nv : 0.f;
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) resid[nt] *= wgt;
      // butterfly over the K lanes of a group, one level for all values at a time; the mirrors serve as the xor-4 / xor-8
      // exchanges because the partial sums are already uniform inside each block of 4 / 8 lanes
      if (p.K >= 2) lane_sum<0xB1, NT>(resid);     // quad_perm [1,0,3,2]
      if (p.K >= 4) lane_sum<0x4E, NT>(resid);     // quad_perm [2,3,0,1]
      if (p.K >= 8) lane_sum<0x141, NT>(resid);    // row_half_mirror
      if (p.K >= 16) lane_sum<0x140, NT>(resid);   // row_mirror
      if (p.K >= 32) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
          for (int r = 0; r < 16; ++r) resid[nt][r] += __shfl_xor(resid[nt][r], 16, 64);
      }
      if (inrange && (slot & (uint32_t)(p.K - 1)) == 0) store_rows<T, NT>(resid, p.M_out, p.M_f32, (long long)gidx * D, true, hi);
    }
  }
}

// `win`: the register window of the in-tile softmax (4, 8 or 16)
template <int D, int DH, int MODE>
static int launch_merge_mode(int win, const BlockParams& p, dim3 grid, hipStream_t stream) {
#define LONGER_MERGE_LAUNCH(WV)                                                                                              \
  do {                                                                                                                       \
    if (p.act == 1) hipLaunchKernelGGL((merge_kernel<D, DH, MODE, WV, true>), grid, dim3(256), 0, stream, p);                \
    else hipLaunchKernelGGL((merge_kernel<D, DH, MODE, WV, false>), grid, dim3(256), 0, stream, p);                          \
  } while (0)
  if constexpr (MODE == MODE_INPUT) LONGER_MERGE_LAUNCH(16);
  else if (win == 4) LONGER_MERGE_LAUNCH(4);
  else if (win == 8) LONGER_MERGE_LAUNCH(8);
  else LONGER_MERGE_LAUNCH(16);
#undef LONGER_MERGE_LAUNCH
  return 0;
}

#define LONGER_INSTANTIATE_MERGE(D, DH)                                                                           \
  template <>                                                                                                     \
  int launch_merge<D, DH>(int mode, int win, const BlockParams& p, dim3 grid, hipStream_t stream) {               \
    return mode == MODE_MERGE ? launch_merge_mode<D, DH, MODE_MERGE>(win, p, grid, stream)                        \
         : mode == MODE_MERGE_IN ? launch_merge_mode<D, DH, MODE_MERGE_IN>(win, p, grid, stream)                  \
         : mode == MODE_MERGE_KEEP ? launch_merge_mode<D, DH, MODE_MERGE_KEEP>(win, p, grid, stream)              \
         : launch_merge_mode<D, DH, MODE_INPUT>(win, p, grid, stream);                                            \
  }

}  // namespace longer
