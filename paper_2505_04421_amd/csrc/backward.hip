// Backward pass with activation recomputation and mixed precision (Section 3.6.2):
// longer_token_merge_backward (the token merge of Section 3.4 alone), longer_forward_backward
// (the whole model: loss of Eq. 1-2 and the gradient of every input and parameter),
// longer_input_generation_backward (the stage of Section 3.5.1 in front of the merge) and their
// size queries.
//
// Token merge: nothing is kept from a forward call.  The pass reads the raw tokens H, gets every
// block's input rows (fp32) from the fused forward kernel, then walks the InnerTrans blocks from
// the last to the first; for each block it recomputes the block's intermediates from the block's
// input and takes the gradients.  Reduced stack (cross-causal and self-causal layers on B (m + k)
// query rows): its intermediates are a twentieth of the merge's and are kept.
// Precision policy: every GEMM runs on the matrix cores with bf16 operands and fp32
// accumulation; the residual stream, its gradient, LayerNorm and softmax statistics and every
// parameter gradient are fp32; activations and activation gradients between two GEMMs are
// stored as bf16.
//
// A parameter gradient is a sum over every token of the batch, i.e. a product whose contraction runs over the tokens
// (bw_grads.h), so what it contracts has to exist for the whole batch.  Everything else is fused per tile of 32 rows:
//   * InnerTrans blocks up to width 128: one launch per block (bw_block.h);
//   * the reduced stack: one launch between two attention launches (bw_stack.h, bw_set_attn.h).
// InnerTrans blocks of width 256, whose tile does not fit a wave's registers, and the input generation run as kernels over
// row-major [token, feature] tensors in the workspace, below:
//   * bf16 MFMA GEMMs, operands with the contraction index contiguous: y = x W (+ epilogues), dx = dy W^T, and the middle
//     of the FFN backward as two products under one epilogue (the hidden pre-activation is formed again there and
//     never stored);
//   * row kernels: LayerNorm forward / backward (+ gain / shift gradients), the merge's backward;
//   * attention inside a group of K tokens, forward and backward, one thread per (row, head), heads kept as packed
//     bf16 (two-feature dot products, fp32 sums).
// Padded token rows are never read and cost only the zeros written for them.
#include "bw_grads.h"
#include "bw_set_attn.h"
#include "bw_stack.h"
#include "bw_input.h"

#include <cstdio>

namespace longer {

int api_error(int code, const char* fmt, ...);   // longer_api.hip
size_t least_workspace_bytes(const longer_config* cfg, int B, int L);
int inner_chain_f32(const longer_config* cfg, const longer_block* inner, int layers, const void* H, const int32_t* lens,
                    int B, int L, float* Z_out, void* ws, size_t ws_bytes, void* stream);   // longer_api.hip
int merge_keep_f32(const longer_config* cfg, const longer_block* inner, const void* H, const int32_t* lens, int B, int L, void* M_out,
                   float* keep, size_t stride, void* ws, size_t ws_bytes, void* stream);   // longer_api.hip

namespace bw {

constexpr int kMaxGroup = 32;   // K <= 32

// ------------------------------------------------------------------------------------
// GEMM  C[M, N] = A[M, Kc] B[Kc, N]  (bf16 operands, fp32 accumulation)
//   A is stored [M][Kc] (contraction contiguous);
//   B is stored [N][Kc] (contraction contiguous).
// Workgroup tile 128 x 128, contraction step 32, four waves in 2 x 2, each 64 x 64 (2 x 2 MFMA
// tiles of 32 x 32).  Requirements checked by the host: strides multiples of 8 elements,
// 16-byte aligned bases; the contraction dimension is a multiple of 32.  Rows / columns / contraction
// slices past the extents read as zeros.
enum Epilogue {
  EPI_BF16 = 0,      // out[m][n] = bf16(acc + bias[n])
  EPI_RES_F32 = 1,   // outf[m][n] = res[m][n] + acc + bias[n]
  EPI_F32 = 5,       // outf[m][n] = acc + bias[n]
  EPI_FFN_MID = 6    // two products in one launch, v = A B + bias and g = A2 B2 (same shapes):
                     // out[m][n] = bf16(g * act'(v)), out2[m][n] = bf16(act(v)); v itself is not stored
};

struct GemmArgs {
  RowsValid rows;             // of the token dimension M
  const __bf16* A; const __bf16* B;
  int lda, ldb;
  int M, N, Kc;
  int epi, act;
  void* out; void* out2; int ldo;
  const __bf16* bias; const float* res;
  const __bf16* A2; const __bf16* B2; int lda2, ldb2;   // the second product of a two-product launch (EPI_FFN_MID)
};

constexpr int kStagePitch = 68;         // floats per row of the epilogue's staging area (64 + 4 pad)

// KS: contraction elements per step.  Every launch uses 32: steps of 64 and 128 (one LDS buffer per operand
// at 128) were measured for the two-product launch, whose contraction is only the model width, and
// changed nothing (6.49 - 6.56 ms per merge backward at the headline shape for the three widths).
template <bool DUAL, int KS = 32>
__global__ __launch_bounds__(256, DUAL ? 2 : 4) void bw_gemm_kernel(GemmArgs g) {
  constexpr int kPitchKC = KS + 8;            // elements per row of a contraction-contiguous LDS tile (8 pad)
  constexpr int kTileElems = 128 * kPitchKC;
  constexpr int CPR = KS / 8;                 // 16-byte chunks per tile row (contraction-contiguous form)
  constexpr int NCH = KS / 16;                // chunks per thread and operand tile
  constexpr int NBUF = KS >= 128 ? 1 : 2;
  __shared__ __attribute__((aligned(16))) __bf16 smem[2 * NBUF * kTileElems];
  auto sA = [&](int buf) { return smem + buf * kTileElems; };          // NBUF buffers per operand
  auto sB = [&](int buf) { return smem + (NBUF + buf) * kTileElems; };
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int wm = w & 1, wn = w >> 1, hi = lane >> 5, l32 = lane & 31;
  // Tile order.  Workgroups go to the 8 accelerator dies round-robin by index, each die with an L2 of
  // its own: the N tiles of one M tile (which share the A rows) get consecutive slots on one die.
  const int ntn = (g.N + 127) / 128, ntm = (g.M + 127) / 128;
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  const int mt = (slot / ntn) * 8 + xcd, nt_ = slot % ntn;
  if (mt >= ntm) return;
  const int m0 = mt * 128, n0 = nt_ * 128;
  const int nk = (g.Kc + KS - 1) / KS, kend = g.Kc;
  if (!rows_any_valid(g.rows, m0, min(g.M, m0 + 128))) return;   // a tile of padded rows: nobody reads its result

  constexpr int NPH = DUAL ? 2 : 1;     // products of the launch
  f32x16 accs[NPH][2][2];
#pragma unroll
  for (int ph = 0; ph < NPH; ++ph)
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) accs[ph][a][b][r] = 0.f;
  const __bf16* opA = g.A; const __bf16* opB = g.B;
  int ldA = g.lda, ldB = g.ldb;

  // Operand tiles travel global -> registers -> LDS.  One tile = 512 chunks of 16 bytes, two per
  // thread.  (Keeping the loads of four steps in flight was measured: 188 registers, two waves per
  // SIMD instead of four, every GEMM slower.)
  bf16x8 ra[1][NCH], rb[1][NCH];
  auto gload = [&](int kt, bf16x8* pa, bf16x8* pb) {
    const int k0 = kt * KS;
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      const int c = tid + 256 * i;
      bf16x8 z;
#pragma unroll
      for (int e = 0; e < 8; ++e) z[e] = (__bf16)0.f;
      pa[i] = z; pb[i] = z;
      {
        const int row = c / CPR, kc = c % CPR;
        const int gr = m0 + row, gk = k0 + 8 * kc;
        if (gr < g.M && gk < kend) pa[i] = *(const bf16x8*)(opA + (size_t)gr * ldA + gk);
      }
      {
        const int row = c / CPR, kc = c % CPR;
        const int gr = n0 + row, gk = k0 + 8 * kc;
        if (gr < g.N && gk < kend) pb[i] = *(const bf16x8*)(opB + (size_t)gr * ldB + gk);
      }
    }
  };
  auto sstore = [&](int buf, const bf16x8* pa, const bf16x8* pb) {
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      const int c = tid + 256 * i;
      *(bf16x8*)&sA(buf)[(c / CPR) * kPitchKC + 8 * (c % CPR)] = pa[i];
      *(bf16x8*)&sB(buf)[(c / CPR) * kPitchKC + 8 * (c % CPR)] = pb[i];
    }
  };
  // fragment of the 32 x 16 operand slice: lane (x = l32, hi) holds contraction slots 8 hi .. 8 hi + 7
  auto frag = [&](const __bf16* s, int x, int ks) -> bf16x8 { return *(const bf16x8*)&s[(x + l32) * kPitchKC + 16 * ks + 8 * hi]; };
  // Contraction steps, two LDS buffers: step's tile goes to LDS (the buffer was last read two steps ago,
  // which every thread left before the previous step's barrier), the registers are refilled with the
  // next step's tile, barrier, MFMAs.
  int buf = 0;
#pragma unroll
  for (int ph = 0; ph < NPH; ++ph) {
  f32x16 (&acc)[2][2] = accs[ph];
  int kt = 0;
  if (kt < nk && !(DUAL && ph == 1)) gload(kt, ra[0], rb[0]);   // (the second product's first tile is on its way already)
  while (kt < nk) {
    if (NBUF == 1) __syncthreads();          // the one buffer is still being read by the step before
    sstore(buf, ra[0], rb[0]);
    const int kn = kt + 1;
    if (kn < nk) {
      gload(kn, ra[0], rb[0]);
    } else if (DUAL && ph == 0) {            // last step of the first product: request the second product's first tile
      opA = g.A2; opB = g.B2; ldA = g.lda2; ldB = g.ldb2;
      gload(0, ra[0], rb[0]);
    }
    __syncthreads();
#pragma unroll
    for (int ks = 0; ks < KS / 16; ++ks) {
      bf16x8 fa[2], fb[2];
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        fa[t] = frag(sA(buf), 64 * wm + 32 * t, ks);
        fb[t] = frag(sB(buf), 64 * wn + 32 * t, ks);
      }
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
          acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[a], fb[b], acc[a][b], 0, 0, 0);
    }
    buf ^= NBUF - 1;
    kt = kn;
  }
  }
  f32x16 (&acc)[2][2] = accs[0];

  float* stage = (float*)smem + w * (32 * kStagePitch);
  static_assert(4 * 32 * kStagePitch * 4 <= 2 * NBUF * kTileElems * 2, "staging area fits the operand buffers");
  // Loads and stores leave one in-order queue: a load that follows a store is not back before the store
  // has been acknowledged.  What the epilogue reads from memory is therefore requested ahead of its
  // stores: the bias chunk once (a thread's chunks all lie in the same eight columns), the residual /
  // pre-activation rows of a 32-row slab before the slab's first store.
  const int ecc = lane & 7, en = n0 + 64 * wn + 8 * ecc;
  float biasv[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) biasv[e] = 0.f;
  if (g.bias && en < g.N) {
    const bf16x8 bv = *(const bf16x8*)(g.bias + en);
#pragma unroll
    for (int e = 0; e < 8; ++e) biasv[e] = (float)bv[e];
  }
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    f32x4 ld[4][2];                   // EPI_RES_F32: the chunk's residual values
    if (g.epi == EPI_RES_F32) {
#pragma unroll
      for (int it = 0; it < 4; ++it) {
        const int m = m0 + 64 * wm + 32 * a + it * 8 + (lane >> 3);
        ld[it][0] = f32x4{0.f, 0.f, 0.f, 0.f}; ld[it][1] = ld[it][0];
        if (m >= g.M || en >= g.N) continue;
        const size_t o = (size_t)m * g.ldo + en;
        ld[it][0] = *(const f32x4*)(g.res + o); ld[it][1] = *(const f32x4*)(g.res + o + 4);
      }
    }
    float v2[DUAL ? 4 : 1][8];        // two-product launch: the second product's values of this thread's chunks
    if constexpr (DUAL) {
      __syncthreads();
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) stage[tile_row(r, hi) * kStagePitch + 32 * b + l32] = accs[NPH - 1][a][b][r];
      __syncthreads();
#pragma unroll
      for (int it = 0; it < 4; ++it) {
        const int id = it * 64 + lane, row = id >> 3, cc = id & 7;
        *(f32x4*)&v2[it][0] = *(const f32x4*)&stage[row * kStagePitch + 8 * cc];
        *(f32x4*)&v2[it][4] = *(const f32x4*)&stage[row * kStagePitch + 8 * cc + 4];
      }
    }
    __syncthreads();
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) stage[tile_row(r, hi) * kStagePitch + 32 * b + l32] = acc[a][b][r];
    __syncthreads();
#pragma unroll
    for (int it = 0; it < 4; ++it) {
      const int id = it * 64 + lane, row = id >> 3, cc = id & 7;
      const int m = m0 + 64 * wm + 32 * a + row, n = n0 + 64 * wn + 8 * cc;
      if (m >= g.M || n >= g.N) continue;
      float v[8];
      *(f32x4*)&v[0] = *(const f32x4*)&stage[row * kStagePitch + 8 * cc];
      *(f32x4*)&v[4] = *(const f32x4*)&stage[row * kStagePitch + 8 * cc + 4];
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] += biasv[e];
      const size_t o = (size_t)m * g.ldo + n;
      bf16x8 ob;
      if (g.epi == EPI_BF16) {
#pragma unroll
        for (int e = 0; e < 8; ++e) ob[e] = (__bf16)v[e];
        *(bf16x8*)((__bf16*)g.out + o) = ob;
      } else if (g.epi == EPI_RES_F32) {
        const f32x4 r0 = ld[it][0], r1 = ld[it][1];
        f32x4 o0, o1;
#pragma unroll
        for (int e = 0; e < 4; ++e) { o0[e] = r0[e] + v[e]; o1[e] = r1[e] + v[4 + e]; }
        *(f32x4*)((float*)g.out + o) = o0;
        *(f32x4*)((float*)g.out + o + 4) = o1;
      } else if (DUAL && g.epi == EPI_FFN_MID) {
        bf16x8 oa;
        auto both = [&](int act) {                    // (which activation: asked once, not between the chains of eight values)
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            float av, dv;
            act_both(v[e], act, &av, &dv);
            oa[e] = (__bf16)av;
            ob[e] = (__bf16)(v2[DUAL ? it : 0][e] * dv);
          }
        };
        if (g.act == LONGER_ACT_RELU) both(LONGER_ACT_RELU); else both(LONGER_ACT_GELU_ERF);
        *(bf16x8*)((__bf16*)g.out + o) = ob;
        *(bf16x8*)((__bf16*)g.out2 + o) = oa;
      } else {
        *(f32x4*)((float*)g.out + o) = *(const f32x4*)&v[0];
        *(f32x4*)((float*)g.out + o + 4) = *(const f32x4*)&v[4];
      }
    }
  }
}

// ------------------------------------------------------------------------------------
// Row GEMM with a short contraction (Kc = K <= 128, the model width): y = x W (+ epilogue) or dx = dy W^T,
// both operands with the contraction index contiguous (the caller hands W transposed where needed).
// With so short a contraction a tile per workgroup spends its time on the way from L2 to the compute unit:
// the weights tile weighs as much as the activation tile and is fetched again by every workgroup, and a
// step's loads are not back before the previous step's few MFMAs are done.  Here a workgroup stays: it
// loads its 128 columns of W (both matrices of the two-product launch) into LDS once, then walks over
// row tiles; the next row tile's activations travel to registers while the current one is multiplied
// and stored.  512 threads: wave w works on rows 32 (w & 3) .. + 31, columns 64 (w >> 2) .. + 63 of
// the 128 x 128 tile; the epilogue turns a wave's result through LDS for 16-byte stores.
// Epilogues: EPI_BF16, EPI_RES_F32, EPI_F32, and with DUAL EPI_FFN_MID.
template <int K, bool DUAL>
__global__ __launch_bounds__(512, 1) void bw_rowgemm_kernel(GemmArgs g, int P) {
  constexpr int PITCH = K + 8, TILE = 128 * PITCH, NPH = DUAL ? 2 : 1, CPR = K / 8;
  constexpr int NCH = (128 * CPR + 511) / 512;              // 16-byte chunks per thread and operand tile
  constexpr int STAGE_BYTES = 8 * 32 * kStagePitch * 4;
  constexpr int A_BYTES = NPH * TILE * 2 > STAGE_BYTES ? NPH * TILE * 2 : STAGE_BYTES;
  __shared__ __attribute__((aligned(16))) unsigned char smem_a[A_BYTES];   // activation tile(s); the epilogue's staging area
  __shared__ __attribute__((aligned(16))) __bf16 sB[NPH * TILE];           // weights, resident
  __bf16* sA = (__bf16*)smem_a;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int wm = w & 3, wn = w >> 2, hi = lane >> 5, l32 = lane & 31;
  float* stage = (float*)smem_a + w * (32 * kStagePitch);
  const int ntn = (g.N + 127) / 128, ntm = (g.M + 127) / 128;
  // workgroups of one row-tile sequence (they read the same activations) sit on one die
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  const int p = (slot / ntn) * 8 + xcd, nt_ = slot % ntn;
  if (p >= P) return;
  const int n0 = nt_ * 128;

  const __bf16* opA[2] = {g.A, DUAL ? g.A2 : g.A};
  const __bf16* opB[2] = {g.B, DUAL ? g.B2 : g.B};
  const int ldA[2] = {g.lda, DUAL ? g.lda2 : g.lda}, ldB[2] = {g.ldb, DUAL ? g.ldb2 : g.ldb};

#pragma unroll
  for (int ph = 0; ph < NPH; ++ph)
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      const int c = tid + 512 * i;
      if (c >= 128 * CPR) continue;
      const int row = c / CPR, kc = c % CPR, gr = n0 + row;
      bf16x8 v;
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = (__bf16)0.f;
      if (gr < g.N) v = *(const bf16x8*)(opB[ph] + (size_t)gr * ldB[ph] + 8 * kc);
      *(bf16x8*)&sB[ph * TILE + row * PITCH + 8 * kc] = v;
    }
  const int ecc = lane & 7, en = n0 + 64 * wn + 8 * ecc;
  float biasv[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) biasv[e] = 0.f;
  if (g.bias && en < g.N) {
    const bf16x8 bv = *(const bf16x8*)(g.bias + en);
#pragma unroll
    for (int e = 0; e < 8; ++e) biasv[e] = (float)bv[e];
  }

  bf16x8 ra[NPH][NCH];
  auto gload = [&](int mt) {
#pragma unroll
    for (int ph = 0; ph < NPH; ++ph)
#pragma unroll
      for (int i = 0; i < NCH; ++i) {
        const int c = tid + 512 * i;
        bf16x8 v;
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = (__bf16)0.f;
        const int row = c / CPR, kc = c % CPR, gr = mt * 128 + row;
        if (c < 128 * CPR && gr < g.M) v = *(const bf16x8*)(opA[ph] + (size_t)gr * ldA[ph] + 8 * kc);
        ra[ph][i] = v;
      }
  };
  auto next_tile = [&](int mt) {      // row tiles without a valid row are passed over: nobody reads their result
    while (mt < ntm && !rows_any_valid(g.rows, mt * 128, min(g.M, mt * 128 + 128))) mt += P;
    return mt;
  };
  auto frag = [&](const __bf16* s_, int x, int ks) -> bf16x8 { return *(const bf16x8*)&s_[x * PITCH + 16 * ks + 8 * hi]; };

  int mt = next_tile(p);
  if (mt < ntm) gload(mt);
  while (mt < ntm) {
    __syncthreads();                  // the staging area of the tile before is read out (and, first time, sB is written)
#pragma unroll
    for (int ph = 0; ph < NPH; ++ph)
#pragma unroll
      for (int i = 0; i < NCH; ++i) {
        const int c = tid + 512 * i;
        if (c < 128 * CPR) *(bf16x8*)&sA[ph * TILE + (c / CPR) * PITCH + 8 * (c % CPR)] = ra[ph][i];
      }
    const int mn = next_tile(mt + P);
    if (mn < ntm) gload(mn);          // on its way during the products and the epilogue below
    __syncthreads();
    f32x16 acc[NPH][2];
#pragma unroll
    for (int ph = 0; ph < NPH; ++ph)
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[ph][t][r] = 0.f;
#pragma unroll
    for (int ph = 0; ph < NPH; ++ph)
#pragma unroll
      for (int ks = 0; ks < K / 16; ++ks) {
        const bf16x8 fa = frag(sA + ph * TILE, 32 * wm + l32, ks);
#pragma unroll
        for (int t = 0; t < 2; ++t)
          acc[ph][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa, frag(sB + ph * TILE, 64 * wn + 32 * t + l32, ks), acc[ph][t], 0, 0, 0);
      }
    __syncthreads();                  // every wave is done with the activation tile: its place becomes the staging area

    const int m0 = mt * 128 + 32 * wm;
    f32x4 ld[4][2];                   // EPI_RES_F32: the chunks' residual values, requested ahead of the stores
    if (g.epi == EPI_RES_F32) {
#pragma unroll
      for (int it = 0; it < 4; ++it) {
        const int m = m0 + it * 8 + (lane >> 3);
        ld[it][0] = f32x4{0.f, 0.f, 0.f, 0.f}; ld[it][1] = ld[it][0];
        if (m >= g.M || en >= g.N) continue;
        const size_t o = (size_t)m * g.ldo + en;
        ld[it][0] = *(const f32x4*)(g.res + o); ld[it][1] = *(const f32x4*)(g.res + o + 4);
      }
    }
    float v2[DUAL ? 4 : 1][8];
    if constexpr (DUAL) {             // (a wave's staging area is its own: LDS keeps a wave's accesses in order)
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) stage[tile_row(r, hi) * kStagePitch + 32 * t + l32] = acc[1][t][r];
#pragma unroll
      for (int it = 0; it < 4; ++it) {
        const int id = it * 64 + lane, row = id >> 3, cc = id & 7;
        *(f32x4*)&v2[it][0] = *(const f32x4*)&stage[row * kStagePitch + 8 * cc];
        *(f32x4*)&v2[it][4] = *(const f32x4*)&stage[row * kStagePitch + 8 * cc + 4];
      }
    }
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) stage[tile_row(r, hi) * kStagePitch + 32 * t + l32] = acc[0][t][r];
#pragma unroll
    for (int it = 0; it < 4; ++it) {
      const int id = it * 64 + lane, row = id >> 3, cc = id & 7;
      const int m = m0 + row, n = n0 + 64 * wn + 8 * cc;
      float v[8];
      *(f32x4*)&v[0] = *(const f32x4*)&stage[row * kStagePitch + 8 * cc];
      *(f32x4*)&v[4] = *(const f32x4*)&stage[row * kStagePitch + 8 * cc + 4];
      if (m >= g.M || n >= g.N) continue;
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] += biasv[e];
      const size_t o = (size_t)m * g.ldo + n;
      bf16x8 ob;
      if (DUAL) {
        bf16x8 oa;
        auto both = [&](int act) {                    // (which activation: asked once, not between the chains of eight values)
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            float av, dv;
            act_both(v[e], act, &av, &dv);
            oa[e] = (__bf16)av;
            ob[e] = (__bf16)(v2[DUAL ? it : 0][e] * dv);
          }
        };
        if (g.act == LONGER_ACT_RELU) both(LONGER_ACT_RELU); else both(LONGER_ACT_GELU_ERF);
        *(bf16x8*)((__bf16*)g.out + o) = ob;
        *(bf16x8*)((__bf16*)g.out2 + o) = oa;
      } else if (g.epi == EPI_BF16) {
#pragma unroll
        for (int e = 0; e < 8; ++e) ob[e] = (__bf16)v[e];
        *(bf16x8*)((__bf16*)g.out + o) = ob;
      } else if (g.epi == EPI_RES_F32) {
        f32x4 o0, o1;
#pragma unroll
        for (int e = 0; e < 4; ++e) { o0[e] = ld[it][0][e] + v[e]; o1[e] = ld[it][1][e] + v[4 + e]; }
        *(f32x4*)((float*)g.out + o) = o0;
        *(f32x4*)((float*)g.out + o + 4) = o1;
      } else {
        *(f32x4*)((float*)g.out + o) = *(const f32x4*)&v[0];
        *(f32x4*)((float*)g.out + o + 4) = *(const f32x4*)&v[4];
      }
    }
    mt = mn;
  }
}

// ------------------------------------------------------------------------------------
// Row kernels.  A token row r = u L + pos is valid when pos < min(lens[u], L).
struct RowGeom { const int32_t* lens; int L, K, ntok; };

__device__ __forceinline__ int row_len(const RowGeom& q, int u) {
  int l = q.lens ? q.lens[u] : q.L;
  return l < 0 ? 0 : (l > q.L ? q.L : l);
}

// x0[r][:] = valid ? H[r][:] : 0   (fp32 copy of the raw tokens: the first block's input); four
// features per thread (d is a multiple of 4)
__global__ __launch_bounds__(256) void bw_load_x0_kernel(const __bf16* __restrict__ H, float* __restrict__ x0, RowGeom q, int d) {
  const size_t n = (size_t)q.ntok * d / 4;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) {
    const int r = (int)(i * 4 / d);
    const int u = r / q.L, pos = r - u * q.L;
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if (pos < row_len(q, u)) {
      const bf16x4 t = *(const bf16x4*)(H + i * 4);
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = (float)t[e];
    }
    *(f32x4*)(x0 + i * 4) = v;
  }
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// LayerNorm kernels: a row of width D = 4 LPR is held by LPR adjacent lanes, four consecutive
// features each (16-byte loads), so a wave works on 64 / LPR rows at a time.
template <int LPR>
__device__ __forceinline__ float row_sum(float v) {
#pragma unroll
  for (int o = LPR / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ f32x4 load_bf16x4(const __bf16* p) {
  const bf16x4 t = *(const bf16x4*)p;
  f32x4 o;
#pragma unroll
  for (int e = 0; e < 4; ++e) o[e] = (float)t[e];
  return o;
}
__device__ __forceinline__ void store_bf16x4(__bf16* p, f32x4 v) {
  bf16x4 t;
#pragma unroll
  for (int e = 0; e < 4; ++e) t[e] = (__bf16)v[e];
  *(bf16x4*)p = t;
}

// n[r][:] = bf16(LN(x[r][:]) g + b)
template <int LPR>
__global__ __launch_bounds__(256) void bw_ln_fwd_kernel(const float* __restrict__ x, const __bf16* __restrict__ gam,
                                                        const __bf16* __restrict__ bet, __bf16* __restrict__ out,
                                                        int ntok, float eps, RowsValid rows) {
  constexpr int RPW = 64 / LPR, D = 4 * LPR;
  const int lane = threadIdx.x & 63, sub = lane % LPR, rsub = lane / LPR;
  const int wave = blockIdx.x * 4 + (threadIdx.x >> 6), nw = gridDim.x * 4;
  const f32x4 gv = load_bf16x4(gam + 4 * sub), bv = load_bf16x4(bet + 4 * sub);
  const int ngroups = (ntok + RPW - 1) / RPW;
#pragma unroll 2
  for (int grp = wave; grp < ngroups; grp += nw) {
    const int r = grp * RPW + rsub;
    const bool ok = r < ntok;
    const bool live = ok && row_valid(rows, r);       // a padded row is written as zeros and not read
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if (live) v = *(const f32x4*)(x + (size_t)r * D + 4 * sub);
    const float mean = row_sum<LPR>(v[0] + v[1] + v[2] + v[3]) * (1.f / D);
    v -= mean;
    const float rstd = 1.f / sqrtf(row_sum<LPR>(v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3]) * (1.f / D) + eps);
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    if (ok) store_bf16x4(out + (size_t)r * D + 4 * sub, live ? v * rstd * gv + bv : zero);
  }
}

// LayerNorm backward for y = LN(x) g + b with upstream dn = dL/dy (bf16) and the gradient dres that
// reaches x through the residual connection (NULL: none): dx_out = dres + dLN, also stored as bf16 (dxb, may be
// NULL); the block's share of dg[e] = sum_r dn xhat and db[e] = sum_r dn goes to part[block][2][D]
// (bw_reduce_jobs_kernel sums the blocks).
template <int LPR>
__global__ __launch_bounds__(256) void bw_ln_bwd_kernel(const __bf16* __restrict__ dn, const float* __restrict__ x,
                                                        const __bf16* __restrict__ gam, const float* __restrict__ dres,
                                                        float* __restrict__ dx_out, __bf16* __restrict__ dxb,
                                                        float* __restrict__ part, int ntok, float eps, RowsValid rows) {
  constexpr int RPW = 64 / LPR, D = 4 * LPR;
  const int lane = threadIdx.x & 63, sub = lane % LPR, rsub = lane / LPR;
  const int wave = blockIdx.x * 4 + (threadIdx.x >> 6), nw = gridDim.x * 4;
  const f32x4 gv = load_bf16x4(gam + 4 * sub);
  f32x4 ag = {0.f, 0.f, 0.f, 0.f}, ab = {0.f, 0.f, 0.f, 0.f};
  const int ngroups = (ntok + RPW - 1) / RPW;
#pragma unroll 2
  for (int grp = wave; grp < ngroups; grp += nw) {
    const int r = grp * RPW + rsub;
    const bool ok = r < ntok;
    const bool live = ok && row_valid(rows, r);       // a padded row: zero gradient, nothing read
    const size_t o = (size_t)r * D + 4 * sub;
    f32x4 v = {0.f, 0.f, 0.f, 0.f}, t = v, res = v;
    if (live) {
      v = *(const f32x4*)(x + o);
      t = load_bf16x4(dn + o);
      if (dres) res = *(const f32x4*)(dres + o);
    }
    const float mean = row_sum<LPR>(v[0] + v[1] + v[2] + v[3]) * (1.f / D);
    v -= mean;
    const float rstd = 1.f / sqrtf(row_sum<LPR>(v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3]) * (1.f / D) + eps);
    v *= rstd;                                   // xhat
    ab += t;
    ag += t * v;
    t *= gv;                                     // dL/dxhat
    const float c1 = row_sum<LPR>(t[0] + t[1] + t[2] + t[3]) * (1.f / D);
    const float c2 = row_sum<LPR>(t[0] * v[0] + t[1] * v[1] + t[2] * v[2] + t[3] * v[3]) * (1.f / D);
    if (ok) {
      const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
      const f32x4 dx = live ? res + rstd * (t - c1 - v * c2) : zero;
      *(f32x4*)(dx_out + o) = dx;
      if (dxb) store_bf16x4(dxb + o, dx);
    }
  }
  // rows handled side by side in the wave, then the block's four waves (LDS)
#pragma unroll
  for (int e = 0; e < 4; ++e) {
#pragma unroll
    for (int o = LPR; o < 64; o <<= 1) {
      ag[e] += __shfl_xor(ag[e], o, 64);
      ab[e] += __shfl_xor(ab[e], o, 64);
    }
  }
  __shared__ f32x4 red[2][4][LPR];
  const int wv = threadIdx.x >> 6;
  if (rsub == 0) {
    red[0][wv][sub] = ag;
    red[1][wv][sub] = ab;
  }
  __syncthreads();
  if (threadIdx.x < 2 * LPR) {
    const int which = threadIdx.x / LPR, c = threadIdx.x % LPR;
    *(f32x4*)(part + (size_t)blockIdx.x * 2 * D + which * D + 4 * c) =
        red[which][0][c] + red[which][1][c] + red[which][2][c] + red[which][3][c];
  }
}

// Gradient of the merge (Section 3.4) into the last block's output rows:
//   mean:   dZ[r][:] = dM[u][t][:] / n_{u,t} for the group's n valid tokens;
//   concat: dZ[r][:] = dM[u][t][j d : (j + 1) d] for the token in slot j of its group;
// zeros for padded tokens.  Written as fp32 and as bf16.
__global__ __launch_bounds__(256) void bw_merge_bwd_kernel(const float* __restrict__ dM, float* __restrict__ dy,
                                                           __bf16* __restrict__ dyb, RowGeom q, int d, int T, int concat) {
  const size_t n = (size_t)q.ntok * d / 4;      // four features per thread
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) {
    const int r = (int)(i * 4 / d), e = (int)(i * 4 - (size_t)r * d);
    const int u = r / q.L, pos = r - u * q.L;
    const int len = row_len(q, u);
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if (pos < len) {
      const int t = pos / q.K, j = pos - t * q.K;
      if (concat) {
        v = *(const f32x4*)(dM + ((size_t)u * T + t) * ((size_t)q.K * d) + (size_t)j * d + e);
      } else {
        const int cnt = min(q.K, len - t * q.K);
        v = *(const f32x4*)(dM + ((size_t)u * T + t) * d + e) / (float)cnt;
      }
    }
    *(f32x4*)(dy + i * 4) = v;
    store_bf16x4(dyb + i * 4, v);
  }
}

// ------------------------------------------------------------------------------------
// Attention inside a group of K adjacent tokens (InnerTrans, Section 3.4): bidirectional, keys
// masked by validity.  qkv [ntok][3 d] = [q | k | v]; one thread per (row, head).
struct GroupOf {
  int first;      // first row of the group
  int n;          // valid tokens in it (they are its first n rows)
};
__device__ __forceinline__ bool group_of(const RowGeom& q, int r, GroupOf* g) {
  const int u = r / q.L, pos = r - u * q.L;
  const int len = row_len(q, u);
  const int t = pos / q.K;
  g->first = u * q.L + t * q.K;
  g->n = max(0, min(q.K, len - t * q.K));
  return pos < len;
}

// A head's DH features as stored (packed bf16): dot products take them two at a time
// (v_dot2_f32_bf16: fp32 sum of two bf16 products and the accumulator), sums weighted by a
// scalar widen them one by one.
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
template <int DH> struct HeadVec { bf16x8 c[DH / 8]; };
template <int DH>
__device__ __forceinline__ HeadVec<DH> load_head(const __bf16* p) {
  HeadVec<DH> v;
#pragma unroll
  for (int c = 0; c < DH / 8; ++c) v.c[c] = *(const bf16x8*)(p + 8 * c);
  return v;
}
template <int DH>
__device__ __forceinline__ void store_head(__bf16* p, const float* v) {
#pragma unroll
  for (int c = 0; c < DH; c += 8) {
    bf16x8 t;
#pragma unroll
    for (int e = 0; e < 8; ++e) t[e] = (__bf16)v[c + e];
    *(bf16x8*)(p + c) = t;
  }
}
template <int DH>
__device__ __forceinline__ float dot(const HeadVec<DH>& a, const HeadVec<DH>& b) {
  float s = 0.f;
#pragma unroll
  for (int c = 0; c < DH / 8; ++c) {
    s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(a.c[c], a.c[c], 0, 1), __builtin_shufflevector(b.c[c], b.c[c], 0, 1), s, false);
    s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(a.c[c], a.c[c], 2, 3), __builtin_shufflevector(b.c[c], b.c[c], 2, 3), s, false);
    s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(a.c[c], a.c[c], 4, 5), __builtin_shufflevector(b.c[c], b.c[c], 4, 5), s, false);
    s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(a.c[c], a.c[c], 6, 7), __builtin_shufflevector(b.c[c], b.c[c], 6, 7), s, false);
  }
  return s;
}
// acc[:] += w v[:]
template <int DH>
__device__ __forceinline__ void axpy(float* acc, float w, const HeadVec<DH>& v) {
#pragma unroll
  for (int c = 0; c < DH / 8; ++c)
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[8 * c + e] = fmaf(w, (float)v.c[c][e], acc[8 * c + e]);
}

// KG: the loops over a group's tokens are unrolled KG times (K <= KG) so that the per-token values
// stay in registers; tokens past the group's valid count are predicated off.
template <int DH, int KG>
__global__ __launch_bounds__(256) void bw_attn_fwd_kernel(const __bf16* qkv, __bf16* o, RowGeom q, int d, int heads) {
  const long long idx = (long long)blockIdx.x * 256 + threadIdx.x;
  if (idx >= (long long)q.ntok * heads) return;
  const int r = (int)(idx / heads), h = (int)(idx - (long long)r * heads);
  GroupOf g;
  float acc[DH];
#pragma unroll
  for (int c = 0; c < DH; ++c) acc[c] = 0.f;
  if (group_of(q, r, &g)) {
    const float scale = rsqrtf((float)DH);
    const HeadVec<DH> qv = load_head<DH>(qkv + (size_t)r * 3 * d + h * DH);
    const __bf16* kbase = qkv + (size_t)g.first * 3 * d + d + h * DH;
    float s[KG];
    float mx = -3.0e38f;
#pragma unroll
    for (int j = 0; j < KG; ++j) {
      s[j] = -3.0e38f;
      if (j < g.n) {
        s[j] = scale * dot<DH>(qv, load_head<DH>(kbase + (size_t)j * 3 * d));
        mx = fmaxf(mx, s[j]);
      }
    }
    float l = 0.f;
#pragma unroll
    for (int j = 0; j < KG; ++j) {
      s[j] = j < g.n ? __expf(s[j] - mx) : 0.f;
      l += s[j];
    }
    const float inv = 1.f / l;
#pragma unroll
    for (int j = 0; j < KG; ++j)
      if (j < g.n) axpy<DH>(acc, s[j] * inv, load_head<DH>(kbase + (size_t)j * 3 * d + d));
  }
  store_head<DH>(o + (size_t)r * d + h * DH, acc);
}

// Query side of the attention backward: for query row i, P_i. is recomputed, dP_ij = do_i . v_j,
// D_i = sum_j P_ij dP_ij, dS_ij = P_ij (dP_ij - D_i), dq_i = scale sum_j dS_ij k_j.  Writes dq into
// dqkv[:, 0:d) and the row's softmax statistics (log-sum-exp of the scaled scores, D_i) into stat.
template <int DH, int KG>
__global__ __launch_bounds__(256) void bw_attn_bwd_q_kernel(const __bf16* qkv, const __bf16* dob, __bf16* dqkv,
                                                            float2* stat, RowGeom q, int d, int heads) {
  const long long idx = (long long)blockIdx.x * 256 + threadIdx.x;
  if (idx >= (long long)q.ntok * heads) return;
  const int r = (int)(idx / heads), h = (int)(idx - (long long)r * heads);
  GroupOf g;
  float acc[DH];
#pragma unroll
  for (int c = 0; c < DH; ++c) acc[c] = 0.f;
  float2 st = make_float2(0.f, 0.f);
  if (group_of(q, r, &g)) {
    const float scale = rsqrtf((float)DH);
    const HeadVec<DH> qv = load_head<DH>(qkv + (size_t)r * 3 * d + h * DH);
    const HeadVec<DH> dov = load_head<DH>(dob + (size_t)r * d + h * DH);
    const __bf16* kbase = qkv + (size_t)g.first * 3 * d + d + h * DH;
    float s[KG], dp[KG];
    float mx = -3.0e38f;
#pragma unroll
    for (int j = 0; j < KG; ++j) {
      s[j] = -3.0e38f; dp[j] = 0.f;
      if (j < g.n) {
        s[j] = scale * dot<DH>(qv, load_head<DH>(kbase + (size_t)j * 3 * d));
        dp[j] = dot<DH>(dov, load_head<DH>(kbase + (size_t)j * 3 * d + d));
        mx = fmaxf(mx, s[j]);
      }
    }
    float l = 0.f, Dn = 0.f;
#pragma unroll
    for (int j = 0; j < KG; ++j) {
      s[j] = j < g.n ? __expf(s[j] - mx) : 0.f;
      l += s[j];
      Dn = fmaf(s[j], dp[j], Dn);
    }
    const float inv = 1.f / l;
    const float D = Dn * inv;
#pragma unroll
    for (int j = 0; j < KG; ++j)
      if (j < g.n) axpy<DH>(acc, scale * inv * s[j] * (dp[j] - D), load_head<DH>(kbase + (size_t)j * 3 * d));
    st = make_float2(mx + __logf(l), D);
  }
  store_head<DH>(dqkv + (size_t)r * 3 * d + h * DH, acc);
  stat[(size_t)r * heads + h] = st;
}

// Key side: for key row j, over the group's valid queries i: P_ij = exp(s_ij - lse_i),
// dv_j = sum_i P_ij do_i, dk_j = scale sum_i P_ij (do_i . v_j - D_i) q_i.  Writes dqkv[:, d:3d).
template <int DH, int KG>
__global__ __launch_bounds__(256) void bw_attn_bwd_kv_kernel(const __bf16* qkv, const __bf16* dob, __bf16* dqkv,
                                                             const float2* stat, RowGeom q, int d, int heads) {
  const long long idx = (long long)blockIdx.x * 256 + threadIdx.x;
  if (idx >= (long long)q.ntok * heads) return;
  const int r = (int)(idx / heads), h = (int)(idx - (long long)r * heads);
  GroupOf g;
  float dk[DH], dv[DH];
#pragma unroll
  for (int c = 0; c < DH; ++c) { dk[c] = 0.f; dv[c] = 0.f; }
  if (group_of(q, r, &g)) {
    const float scale = rsqrtf((float)DH);
    const HeadVec<DH> kv = load_head<DH>(qkv + (size_t)r * 3 * d + d + h * DH);
    const HeadVec<DH> vv = load_head<DH>(qkv + (size_t)r * 3 * d + 2 * d + h * DH);
#pragma unroll
    for (int i = 0; i < KG; ++i) {
      if (i < g.n) {
        const int ri = g.first + i;
        const HeadVec<DH> qi = load_head<DH>(qkv + (size_t)ri * 3 * d + h * DH);
        const HeadVec<DH> doi = load_head<DH>(dob + (size_t)ri * d + h * DH);
        const float2 st = stat[(size_t)ri * heads + h];
        const float p = __expf(scale * dot<DH>(qi, kv) - st.x);
        const float ds = scale * p * (dot<DH>(doi, vv) - st.y);
        axpy<DH>(dv, p, doi);
        axpy<DH>(dk, ds, qi);
      }
    }
  }
  store_head<DH>(dqkv + (size_t)r * 3 * d + d + h * DH, dk);
  store_head<DH>(dqkv + (size_t)r * 3 * d + 2 * d + h * DH, dv);
}

// Both sides in one launch, when every group lies inside one workgroup's rows (L a multiple of K, and K a divisor
// of the 256 / heads rows a workgroup holds): the query side first, its statistics to LDS, then the key side from
// there.  The second pass finds the group's rows in the cache that the first pass filled, so the pair reads
// q, k, v and the output gradient from memory once instead of twice.
template <int DH, int KG>
__global__ __launch_bounds__(256) void bw_attn_bwd_fused_kernel(const __bf16* qkv, const __bf16* dob, __bf16* dqkv,
                                                                RowGeom q, int d, int heads) {
  __shared__ float2 sst[256];
  const long long idx = (long long)blockIdx.x * 256 + threadIdx.x;
  const bool inside = idx < (long long)q.ntok * heads;
  const int r = inside ? (int)(idx / heads) : 0, h = inside ? (int)(idx - (long long)r * heads) : 0;
  const int r0 = (int)(((long long)blockIdx.x * 256) / heads);
  GroupOf g;
  const bool valid = inside && group_of(q, r, &g);
  const float scale = rsqrtf((float)DH);
  float2 st = make_float2(0.f, 0.f);
  {
    float acc[DH];
#pragma unroll
    for (int c = 0; c < DH; ++c) acc[c] = 0.f;
    if (valid) {
      const HeadVec<DH> qv = load_head<DH>(qkv + (size_t)r * 3 * d + h * DH);
      const HeadVec<DH> dov = load_head<DH>(dob + (size_t)r * d + h * DH);
      const __bf16* kbase = qkv + (size_t)g.first * 3 * d + d + h * DH;
      float s[KG], dp[KG];
      float mx = -3.0e38f;
#pragma unroll
      for (int j = 0; j < KG; ++j) {
        s[j] = -3.0e38f; dp[j] = 0.f;
        if (j < g.n) {
          s[j] = scale * dot<DH>(qv, load_head<DH>(kbase + (size_t)j * 3 * d));
          dp[j] = dot<DH>(dov, load_head<DH>(kbase + (size_t)j * 3 * d + d));
          mx = fmaxf(mx, s[j]);
        }
      }
      float l = 0.f, Dn = 0.f;
#pragma unroll
      for (int j = 0; j < KG; ++j) {
        s[j] = j < g.n ? __expf(s[j] - mx) : 0.f;
        l += s[j];
        Dn = fmaf(s[j], dp[j], Dn);
      }
      const float inv = 1.f / l;
      const float D = Dn * inv;
#pragma unroll
      for (int j = 0; j < KG; ++j)
        if (j < g.n) axpy<DH>(acc, scale * inv * s[j] * (dp[j] - D), load_head<DH>(kbase + (size_t)j * 3 * d));
      st = make_float2(mx + __logf(l), D);
    }
    if (inside) store_head<DH>(dqkv + (size_t)r * 3 * d + h * DH, acc);
  }
  sst[threadIdx.x] = st;
  __syncthreads();
  float dk[DH], dv[DH];
#pragma unroll
  for (int c = 0; c < DH; ++c) { dk[c] = 0.f; dv[c] = 0.f; }
  if (valid) {
    const HeadVec<DH> kv = load_head<DH>(qkv + (size_t)r * 3 * d + d + h * DH);
    const HeadVec<DH> vv = load_head<DH>(qkv + (size_t)r * 3 * d + 2 * d + h * DH);
#pragma unroll
    for (int i = 0; i < KG; ++i) {
      if (i < g.n) {
        const int ri = g.first + i;
        const HeadVec<DH> qi = load_head<DH>(qkv + (size_t)ri * 3 * d + h * DH);
        const HeadVec<DH> doi = load_head<DH>(dob + (size_t)ri * d + h * DH);
        const float2 si = sst[(ri - r0) * heads + h];
        const float p = __expf(scale * dot<DH>(qi, kv) - si.x);
        const float ds = scale * p * (dot<DH>(doi, vv) - si.y);
        axpy<DH>(dv, p, doi);
        axpy<DH>(dk, ds, qi);
      }
    }
  }
  if (inside) {
    store_head<DH>(dqkv + (size_t)r * 3 * d + d + h * DH, dk);
    store_head<DH>(dqkv + (size_t)r * 3 * d + 2 * d + h * DH, dv);
  }
}

// launchers by head width and group size
template <int DH, int KG>
static void attn_launch(int which, unsigned grid, hipStream_t st, const __bf16* qkv, const __bf16* dob, __bf16* out, float2* stat,
                        RowGeom q, int d, int heads) {
  if (which == 0) bw_attn_fwd_kernel<DH, KG><<<grid, 256, 0, st>>>(qkv, out, q, d, heads);
  else if (which == 3) bw_attn_bwd_fused_kernel<DH, KG><<<grid, 256, 0, st>>>(qkv, dob, out, q, d, heads);
  else if (which == 1) bw_attn_bwd_q_kernel<DH, KG><<<grid, 256, 0, st>>>(qkv, dob, out, stat, q, d, heads);
  else bw_attn_bwd_kv_kernel<DH, KG><<<grid, 256, 0, st>>>(qkv, dob, out, stat, q, d, heads);
}
// which: 0 forward (out = o), 1 backward, query side, 2 backward, key side (out = dqkv), 3 both sides in one launch
static void group_attn(int which, int dh, int K, unsigned grid, hipStream_t st, const __bf16* qkv, const __bf16* dob, __bf16* out,
                       float2* stat, RowGeom q, int d, int heads) {
#define LONGER_BW_ATTN(DH, KG) attn_launch<DH, KG>(which, grid, st, qkv, dob, out, stat, q, d, heads)
  if (dh == 16) {
    if (K <= 4) LONGER_BW_ATTN(16, 4); else if (K <= 8) LONGER_BW_ATTN(16, 8); else if (K <= 16) LONGER_BW_ATTN(16, 16); else LONGER_BW_ATTN(16, 32);
  } else {
    if (K <= 4) LONGER_BW_ATTN(32, 4); else if (K <= 8) LONGER_BW_ATTN(32, 8); else if (K <= 16) LONGER_BW_ATTN(32, 16); else LONGER_BW_ATTN(32, 32);
  }
#undef LONGER_BW_ATTN
}

// [wq | wk | wv] side by side: cat[i][j d + c] = w_j[i][c]; biases the same way
__global__ __launch_bounds__(256) void bw_concat_qkv_kernel(const __bf16* wq, const __bf16* wk, const __bf16* wv,
                                                            const __bf16* bq, const __bf16* bk, const __bf16* bv,
                                                            __bf16* cat, __bf16* bcat, int d) {
  const int n = d * 3 * d;
  for (int i = blockIdx.x * 256 + threadIdx.x; i < n + 3 * d; i += gridDim.x * 256) {
    if (i < n) {
      const int row = i / (3 * d), col = i - row * 3 * d;
      const int j = col / d, c = col - j * d;
      const __bf16* w = j == 0 ? wq : (j == 1 ? wk : wv);
      cat[i] = w[row * d + c];
    } else {
      const int col = i - n;
      const int j = col / d, c = col - j * d;
      const __bf16* b = j == 0 ? bq : (j == 1 ? bk : bv);
      bcat[col] = b[c];
    }
  }
}

// rows [B][T K][d] -> [B][L][d] (the first L rows of every user)
__global__ __launch_bounds__(256) void bw_take_rows_kernel(const float* __restrict__ src, float* __restrict__ dst, int B, int L,
                                                           int TK, int d) {
  const size_t per = (size_t)L * d / 4, total = per * B;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (size_t)gridDim.x * 256) {
    const size_t u = i / per, r = i - u * per;
    *(f32x4*)(dst + (u * L * d + r * 4)) = *(const f32x4*)(src + (u * TK * d + r * 4));
  }
}


// ------------------------------------------------------------------------------------
// The reduced stack (Section 3.5): cross-causal layer over R = [G; M] with the query set O of Eq. 5,
// self-causal layers over O's rows (descriptors and attention: bw_set_attn.h).

// merged index held by query slot i of a user with tu merged tokens (Section 3.5.1): the last
// k - k_uniform slots the most recent tokens, the first k_uniform spread evenly over the older ones
// (each the newest token of its share); negative: the slot is empty
__device__ __forceinline__ int slot_merged_index(int i, int k, int tu, int k_uniform) {
  if (tu <= k || i >= k_uniform) return tu - k + i;
  const int rest = tu - (k - k_uniform);
  return (int)(((long long)(i + 1) * rest) / k_uniform) - 1;
}

struct StackGeom { const int32_t* lens; int L, K, T, m, k, k_uniform, B, learn; };   // learn: the slots hold learnable query tokens

__device__ __forceinline__ int merged_len(const StackGeom& g, int u) {
  int l = g.lens ? g.lens[u] : g.L;
  l = l < 0 ? 0 : (l > g.L ? g.L : l);
  return (l + g.K - 1) / g.K;
}

// entry i of the descriptors of the query rows [B][m + k] and, behind them, of the cross layer's key rows [B][m + T]
__device__ __forceinline__ void write_descriptor(const StackGeom& g, int i, int* qdesc, int* kdesc) {
  const int n = g.m + g.k, nk = g.m + g.T;
  if (i < g.B * n) {
    const int u = i / n, r = i - u * n;
    int dsc = r;
    if (r >= g.m) {
      const int tu = merged_len(g, u);
      // a learnable query token stands after the user's newest token, in slot order (it sees every valid
      // merged token in the cross layer and the slots up to itself in the self layers); no token, no slot
      const int t = g.learn ? (tu > 0 ? tu + (r - g.m) : -1) : slot_merged_index(r - g.m, g.k, tu, g.k_uniform);
      dsc = t >= 0 ? kSeq + t : -1;
    }
    qdesc[i] = dsc;
  } else {
    const int j = i - g.B * n;
    const int u = j / nk, r = j - u * nk;
    kdesc[j] = r < g.m ? r : (r - g.m < merged_len(g, u) ? kSeq + (r - g.m) : -1);
  }
}

// Head and loss (Eq. 1-2) for one user per block: logit = <head_w, the m global rows of Y> + head_b,
// loss += (softplus form of the cross-entropy) / B, dlogit = (sigmoid(logit) - label) / B, and the
// gradients that follow: dY (global rows dlogit head_w; the other rows have none and are not written), head_w, head_b.
__global__ __launch_bounds__(256) void bw_head_kernel(const float* __restrict__ Y, const __bf16* __restrict__ hw,
                                                      const __bf16* __restrict__ hb, const float* __restrict__ labels,
                                                      int B, int n, int m, int d, float* __restrict__ logits,
                                                      float* loss, float* __restrict__ dY, float* dhw, float* dhb) {
  __shared__ float red[4];
  __shared__ float dl_s;
  const int u = blockIdx.x;
  const float* y = Y + (size_t)u * n * d;
  float s = 0.f;
  for (int j = threadIdx.x; j < m * d; j += 256) s += y[j] * (float)hw[j];
  s = wave_sum(s);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    const float z = red[0] + red[1] + red[2] + red[3] + (float)hb[0];
    const float lab = labels[u];
    const float e = __expf(-fabsf(z));
    const float sig = z >= 0.f ? 1.f / (1.f + e) : e / (1.f + e);
    const float dl = (sig - lab) / (float)B;
    if (logits) logits[u] = z;
    unsafeAtomicAdd(loss, (fmaxf(z, 0.f) - z * lab + log1pf(e)) / (float)B);
    unsafeAtomicAdd(dhb, dl);
    dl_s = dl;
  }
  __syncthreads();
  const float dl = dl_s;
  for (int j = threadIdx.x; j < m * d; j += 256) {
    dY[(size_t)u * n * d + j] = dl * (float)hw[j];
    unsafeAtomicAdd(dhw + j, dl * y[j]);
  }
}

// dG = the global rows of dO + the global rows of dR; dM[u][t] = dR's row of merged token t (zeros past T_u), plus dO's row of the
// slot that holds it (of other than the most recent tokens and learnable ones: bw_slot_grad_kernel)
__global__ __launch_bounds__(256) void bw_split_grad_kernel(StackGeom g, int d, const float* __restrict__ dO,
                                                            const float* __restrict__ dR, float* __restrict__ dG,
                                                            float* __restrict__ dM) {
  const int n = g.m + g.k, nk = g.m + g.T, d4 = d / 4;
  const size_t total = (size_t)g.B * nk * d4;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (size_t)gridDim.x * 256) {
    const int c = (int)(i % d4) * 4;
    const size_t row = i / d4;
    const int u = (int)(row / nk), r = (int)(row - (size_t)u * nk);
    const f32x4 v = *(const f32x4*)(dR + row * d + c);
    if (r < g.m) {
      *(f32x4*)(dG + ((size_t)u * g.m + r) * d + c) = v + *(const f32x4*)(dO + ((size_t)u * n + r) * d + c);
    } else {
      const int t = r - g.m;
      const int tu = merged_len(g, u), slot = t - tu + g.k;           // (the most recent k tokens fill the slots in order)
      f32x4 w = {0.f, 0.f, 0.f, 0.f};
      if (t < tu) {
        w = v;
        if (!g.k_uniform && !g.learn && slot >= 0) w += *(const f32x4*)(dO + ((size_t)u * n + g.m + slot) * d + c);
      }
      *(f32x4*)(dM + ((size_t)u * g.T + t) * d + c) = w;
    }
  }
}
// dM[u][t_i] += dO's row of query slot i (each slot of a user holds a different merged token)
// (learnable query tokens: the slot's gradient belongs to row sl of the parameter instead, summed over the users)
__global__ __launch_bounds__(256) void bw_slot_grad_kernel(StackGeom g, int d, const float* __restrict__ dO,
                                                           const int* __restrict__ qdesc, float* __restrict__ dM,
                                                           float* dql) {
  const int n = g.m + g.k, d4 = d / 4;
  const size_t total = (size_t)g.B * g.k * d4;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (size_t)gridDim.x * 256) {
    const int c = (int)(i % d4) * 4;
    const size_t s = i / d4;
    const int u = (int)(s / g.k), sl = (int)(s - (size_t)u * g.k);
    const int dsc = qdesc[(size_t)u * n + g.m + sl];
    if (dsc < kSeq) continue;
    const f32x4 v = *(const f32x4*)(dO + ((size_t)u * n + g.m + sl) * d + c);
    if (g.learn) {
#pragma unroll
      for (int e = 0; e < 4; ++e) unsafeAtomicAdd(dql + (size_t)sl * d + c + e, v[e]);
    } else {
      float* dst = dM + ((size_t)u * g.T + (dsc - kSeq)) * d + c;
      *(f32x4*)dst = *(const f32x4*)dst + v;
    }
  }
}


// ------------------------------------------------------------------------------------
// Input generation (Section 3.5.1): x = [E + pos ; tdiff] per valid token, H = act(x w1 + b1) w2 + b2.
// x[r][:] as bf16, zeros for padded tokens
__global__ __launch_bounds__(256) void bw_input_rows_kernel(const __bf16* __restrict__ E, const __bf16* __restrict__ pos,
                                                            const __bf16* __restrict__ td, __bf16* __restrict__ x,
                                                            RowGeom q, int d, int de) {
  const size_t n = (size_t)q.ntok * d / 4;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) {
    const int r = (int)(i * 4 / d), c = (int)(i * 4 - (size_t)r * d);
    const int u = r / q.L, p = r - u * q.L;
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if (p < row_len(q, u)) {
      if (c < de) v = load_bf16x4(E + (size_t)r * de + c) + load_bf16x4(pos + (size_t)p * de + c);
      else v = load_bf16x4(td + (size_t)r * (d - de) + (c - de));
    }
    store_bf16x4(x + i * 4, v);
  }
}
// the upstream gradient as bf16, zeros for padded tokens
__global__ __launch_bounds__(256) void bw_cast_rows_kernel(const float* __restrict__ g, __bf16* __restrict__ gb, RowGeom q, int d) {
  const size_t n = (size_t)q.ntok * d / 4;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) {
    const int r = (int)(i * 4 / d);
    const int u = r / q.L, p = r - u * q.L;
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if (p < row_len(q, u)) v = *(const f32x4*)(g + i * 4);
    store_bf16x4(gb + i * 4, v);
  }
}
// dx [ntok][d] -> dE [ntok][de] and dtdiff [ntok][d - de], zeros for padded tokens
__global__ __launch_bounds__(256) void bw_split_input_grad_kernel(const float* __restrict__ dx, float* __restrict__ dE,
                                                                  float* __restrict__ dtd, RowGeom q, int d, int de) {
  const size_t n = (size_t)q.ntok * d / 4;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) {
    const int r = (int)(i * 4 / d), c = (int)(i * 4 - (size_t)r * d);
    const int u = r / q.L, p = r - u * q.L;
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if (p < row_len(q, u)) v = *(const f32x4*)(dx + i * 4);
    if (c < de) *(f32x4*)(dE + (size_t)r * de + c) = v;
    else *(f32x4*)(dtd + (size_t)r * (d - de) + (c - de)) = v;
  }
}
// dpos[p][c] = sum over the users whose sequence reaches position p of dE[u L + p][c]: a workgroup sums 64 groups of four
// adjacent values, each of its waves every fourth user (eight requests on their way: with one thread per sum and one request
// at a time 90 users of 2500 positions took 33 us)
__global__ __launch_bounds__(256) void bw_pos_grad_kernel(const float* __restrict__ dE, float* __restrict__ dpos, RowGeom q, int B, int de) {
  __shared__ f32x4 red[4][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const size_t i = (size_t)blockIdx.x * 64 + lane, n = (size_t)q.L * de / 4;
  const int p = i < n ? (int)(i * 4 / de) : 0x7fffffff;
  f32x4 s = {0.f, 0.f, 0.f, 0.f};
  for (int u0 = w; u0 < B; u0 += 32) {
    f32x4 v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int u = u0 + 4 * k;
      v[k] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (u < B && p < row_len(q, u)) v[k] = *(const f32x4*)(dE + (size_t)u * q.L * de + i * 4);
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) s += v[k];
  }
  red[w][lane] = s;
  __syncthreads();
  if (w == 0 && i < n) *(f32x4*)(dpos + i * 4) = red[0][lane] + red[1][lane] + red[2][lane] + red[3][lane];
}

// out[c][r] = in[r][c]  (bf16, small parameter matrices; 32 x 32 tiles through LDS)
__global__ __launch_bounds__(256) void bw_transpose_kernel(const __bf16* __restrict__ in, __bf16* __restrict__ out, int rows, int cols) {
  __shared__ __bf16 t[32][33];
  const int r0 = blockIdx.y * 32, c0 = blockIdx.x * 32, x = threadIdx.x & 31, y = threadIdx.x >> 5;
  for (int i = y; i < 32; i += 8)
    if (r0 + i < rows && c0 + x < cols) t[i][x] = in[(size_t)(r0 + i) * cols + c0 + x];
  __syncthreads();
  for (int i = y; i < 32; i += 8)
    if (c0 + i < cols && r0 + x < rows) out[(size_t)(c0 + i) * rows + r0 + x] = t[x][i];
}

// ------------------------------------------------------------------------------------
// Weights for the tile kernels (bw_block.h, bw_stack.h), in the order a launch consumes them: segments of d / 16
// fragments of 64 lanes x 16 bytes.  Fragment = 32 rows of the product's result (lane % 32) x 16 contracted features in
// the order the lanes hold them (element e of lane half hi: 8 (e / 4) + 4 hi + e % 4).  A segment is either 32 result
// features over the whole width, or (spread) all result features over 32 contracted ones.
//
// A training step's launch also writes what else it needs ahead of everything: the rows' descriptors and the zeros that
// are added to with atomics (kPrepareRows rows of workgroups behind the jobs').  As launches of their own (two fills, descriptors,
// the stack's and the InnerTrans blocks' weights) they took 28 of the 316 us of the small model's step.
struct PackJob {
  const __bf16* w; __bf16* out; int sk, sm;        // element (contracted k, result m) at w[k sk + m sm]
  int d, spread, n, pos, stride;                   // n segments, the i-th at place pos + i stride of the stream `out`
};
constexpr int kPackJobs = 72, kPrepareRows = 8;
struct PackJobs { PackJob job[kPackJobs]; int n; };
struct Prepare { StackGeom geo; int *qdesc, *kdesc; float* zeros; size_t nzeros; float* loss; };
__global__ __launch_bounds__(256) void bw_pack_kernel(const PackJobs a, const Prepare q) {
  if ((int)blockIdx.y >= a.n) {
    const size_t rows = (size_t)q.geo.B * (2 * q.geo.m + q.geo.k + q.geo.T), total = rows + q.nzeros;
    const size_t first = ((size_t)(blockIdx.y - a.n) * gridDim.x + blockIdx.x) * 256 + threadIdx.x;
    if (first == 0) *q.loss = 0.f;
    for (size_t i = first; i < total; i += (size_t)kPrepareRows * gridDim.x * 256) {
      if (i < rows) write_descriptor(q.geo, (int)i, q.qdesc, q.kdesc);
      else q.zeros[i - rows] = 0.f;
    }
    return;
  }
  const PackJob& b = a.job[blockIdx.y];
  const int NG = b.d / 16, total = b.n * NG * 64;
  for (int i = blockIdx.x * 256 + threadIdx.x; i < total; i += gridDim.x * 256) {
    const int lane = i & 63, s = (i >> 6) % NG, seg = (i >> 6) / NG, m = lane & 31, hi = lane >> 5;
    const __bf16* src = b.w + (b.spread ? (size_t)(32 * seg + 16 * (s % 2)) * b.sk + (size_t)(32 * (s / 2) + m) * b.sm
                                        : (size_t)(16 * s) * b.sk + (size_t)(32 * seg + m) * b.sm);
    bf16x8 v;
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = src[(size_t)(8 * (e / 4) + 4 * hi + e % 4) * b.sk];
    *(bf16x8*)(b.out + (((size_t)(b.pos + seg * b.stride) * NG + s) * 64 + lane) * 8) = v;
  }
}

// The parameter gradients that the tile kernels leave in terms of the normalised rows xh (y = xh g + s in front
// of the products W): with X = xh^T dY and c = column sums of dY (bias gradients) both summed by now,
//   dW = diag(g) X + s c^T,   dg[e] = sum_c W[e][c] X[e][c],   ds[e] = sum_c W[e][c] c[c],
// so the LayerNorm gradients need no pass over the tokens.  One workgroup per row e and LayerNorm.
constexpr int kNormBlocks = 16;           // blocks per launch
struct NormJob { const __bf16 *w[3], *gain, *shift; float *dw, *dgain; int d, f; };
struct NormGrads { NormJob n[2 * kNormBlocks]; };
__global__ __launch_bounds__(256) void bw_norm_grads_kernel(const NormGrads a) {
  const auto& q = a.n[blockIdx.y];
  const int which = blockIdx.y & 1, e = blockIdx.x, d = q.d, n = which ? q.f : d, mats = which ? 1 : 3;     // ln1: Q, K, V; ln2: W1
  if (e >= d) return;
  const float gain = (float)q.gain[e], shift = (float)q.shift[e];
  float sg = 0.f, ss = 0.f;
  for (int i = threadIdx.x; i < mats * n; i += 256) {
    const int j = i / n, c = i - j * n;
    float* m = q.dw + (size_t)j * ((size_t)d * n + n);
    const float w = (float)q.w[j][(size_t)e * n + c], bias = m[(size_t)d * n + c], X = m[(size_t)e * n + c];
    sg = fmaf(w, X, sg);
    ss = fmaf(w, bias, ss);
    m[(size_t)e * n + c] = fmaf(gain, X, shift * bias);
  }
  __shared__ float red[2][4];
  sg = wave_sum(sg); ss = wave_sum(ss);
  if ((threadIdx.x & 63) == 0) { red[0][threadIdx.x >> 6] = sg; red[1][threadIdx.x >> 6] = ss; }
  __syncthreads();
  if (threadIdx.x < 2) {
    const float* r = red[threadIdx.x];
    q.dgain[threadIdx.x * d + e] = r[0] + r[1] + r[2] + r[3];
  }
}

// ------------------------------------------------------------------------------------ host side
static inline size_t up256(size_t v) { return (v + 255) & ~(size_t)255; }

// Parameter gradients of one block: fp32, in the order of the longer_block members.
struct GradLayout { size_t ln1_g, ln1_b, wq, bq, wk, bk, wv, bv, wo, bo, ln2_g, ln2_b, w1, b1, w2, b2, total; };
static GradLayout grad_layout(int d, int f) {
  GradLayout g;
  size_t o = 0;
  auto take = [&](size_t n) { size_t at = o; o += n; return at; };
  g.ln1_g = take(d); g.ln1_b = take(d);
  g.wq = take((size_t)d * d); g.bq = take(d);
  g.wk = take((size_t)d * d); g.bk = take(d);
  g.wv = take((size_t)d * d); g.bv = take(d);
  g.wo = take((size_t)d * d); g.bo = take(d);
  g.ln2_g = take(d); g.ln2_b = take(d);
  g.w1 = take((size_t)d * f); g.b1 = take(f);
  g.w2 = take((size_t)f * d); g.b2 = take(d);
  g.total = o;
  return g;      // ln*_b follows ln*_g directly: their partial sums are one vector
}

// most workgroups of a LayerNorm backward launch, each with a partial [2][d] of the gain / shift gradients
constexpr int kMaxLnBlocks = 2048;
static unsigned ln_blocks(size_t rows) { return (unsigned)((rows + 3) / 4 > kMaxLnBlocks ? kMaxLnBlocks : (rows + 3) / 4); }

struct Workspace {
  size_t wcat, bcat;                       // per layer: [d][3d] bf16, [3d] bf16
  size_t xin;                              // per layer: fp32 [ntok][d]
  size_t w1t, wcatt, wot;                  // per layer, transposed: W1 [f][d], [wq | wk | wv] [3d][d], W_O [d][d] (bf16)
  size_t n1, qkv, o, xmid, n2, a;          // one block's recomputed intermediates
  size_t dy, dyb, dh, dn, dxm, dxmb, dob, dqkv, stat;
  size_t part, lnpart;                     // partial parameter gradients of one block: matrices, LayerNorms (ln1, ln2)
  size_t fwd, fwd_bytes, ztmp;             // the fused forward kernel's scratch and output when it recomputes block inputs
  size_t stream, rec;                      // block kernel: packed weights per layer, tile records
  size_t total;
};
// The gradients of an InnerTrans block's four products (Q / K / V side by side), all over the raw token rows
static WgradBatch block_wgrads(int d, int f, size_t ntok, RowsValid rv, const __bf16* n1, const __bf16* dqkv, const __bf16* o,
                               const __bf16* dxmb, const __bf16* n2, const __bf16* dh, const __bf16* a, const __bf16* dyb, float* g) {
  const GradLayout gl = grad_layout(d, f);
  WgradBatch w(d, ntok);
  w.add(a, f, f, dyb, d, d, d, ntok, rv, g + gl.w2);
  w.add(n2, d, d, dh, f, f, f, ntok, rv, g + gl.w1);
  w.add(o, d, d, dxmb, d, d, d, ntok, rv, g + gl.wo);
  w.add(n1, d, d, dqkv, 3 * d, 3 * d, d, ntok, rv, g + gl.wq);
  return w;
}
// the same from the block kernel's tile records
// (the last block's W2 from its groups' operands, where they are kept: `groups` of K tokens)
struct GroupOperands { const __bf16 *x, *y; int groups, K; };
static WgradBatch block_wgrads_tiles(int d, int f, size_t slots, RowsValid rv, const __bf16* rec, float* g, const GroupOperands* go = nullptr) {
  const GradLayout gl = grad_layout(d, f);
  const BlockRecord r(d, f, go != nullptr);
  auto at = [&](int o) { return rec + (size_t)o * 512; };
  WgradBatch w(d, slots < 64 ? 64 : slots, true);      // (the groups' job has no more rows than that)
  if (go) w.add(go->x, f / 16, f, go->y, d / 16, d, d, 64 * group_tiles(slots, go->K), RowsValid{rv.lens, rv.L / go->K}, g + gl.w2, 1, 0, 0, 0, go->groups, go->K);
  else w.add(at(r.a), r.size, f, at(r.dyb), r.size, d, d, slots, rv, g + gl.w2);
  w.add(at(r.xh2), r.size, d, at(r.dh), r.size, f, f, slots, rv, g + gl.w1);
  w.add(at(r.o), r.size, d, at(r.dxmb), r.size, d, d, slots, rv, g + gl.wo);
  w.add(at(r.xh1), r.size, d, at(r.qkv), r.size, 3 * d, d, slots, rv, g + gl.wq);
  return w;
}
static int launch(WgradBatch& w, float* part, hipStream_t st) {
  w.place(part);
  const unsigned grid = (unsigned)((w.a.nslices + 7) / 8 * 8 * w.a.tiles);
  if (w.tiled) {
    if (w.a.job[0].groups) {             // (a job of groups is the first one)
      if (w.tb == 128) bw_wgrad_kernel<128, true, true><<<grid, 256, 0, st>>>(w.a);
      else bw_wgrad_kernel<64, true, true><<<grid, 256, 0, st>>>(w.a);
    } else if (w.tb == 128) bw_wgrad_kernel<128, true><<<grid, 256, 0, st>>>(w.a);
    else bw_wgrad_kernel<64, true><<<grid, 256, 0, st>>>(w.a);
  } else if (w.tb == 128) bw_wgrad_kernel<128, false><<<grid, 256, 0, st>>>(w.a);
  else bw_wgrad_kernel<64, false><<<grid, 256, 0, st>>>(w.a);
  return hipGetLastError() == hipSuccess ? 0 : api_error(LONGER_ERR_HIP, "parameter gradient launch failed");
}
static int launch(const ReduceBatch& r, hipStream_t st) {
  bw_reduce_jobs_kernel<<<(unsigned)r.blocks, 256, 0, st>>>(r.a);
  return hipGetLastError() == hipSuccess ? 0 : api_error(LONGER_ERR_HIP, "gradient reduction launch failed");
}

// Weights of one or several streams, packed in as few launches as their number allows
struct PackBatch {
  PackJobs a = {};
  int d; __bf16* out; hipStream_t st; int rc = 0;
  PackBatch(int d_, __bf16* out_, hipStream_t st_) : d(d_), out(out_), st(st_) {}
  void into(int d_, __bf16* out_) { d = d_; out = out_; }      // the following jobs' width and stream
  void add(const void* w, int sk, int sm, bool spread, int segs, int pos, int stride) {
    if (a.n == kPackJobs) flush();
    a.job[a.n++] = PackJob{(const __bf16*)w, out, sk, sm, d, spread, segs, pos, stride};
  }
  int flush(const Prepare* prepare = nullptr) {
    if ((a.n || prepare) && !rc) {
      bw_pack_kernel<<<dim3(64, a.n + (prepare ? kPrepareRows : 0)), 256, 0, st>>>(a, prepare ? *prepare : Prepare{});
      if (hipGetLastError() != hipSuccess) rc = api_error(LONGER_ERR_HIP, "weight packing launch failed");
    }
    a.n = 0;
    return rc;
  }
};
// Sums over partial results that wait for the next such launch (the results keep a place of their own), and the blocks whose LayerNorm
// gradients and dW = diag(g) X + s c^T (bw_norm_grads_kernel; blocks of one or several widths) are made of sums.  Nothing of the second
// part is launched but by finish(), behind all sums: with launches as they filled up, a model of sixteen self layers had
// its LayerNorm gradients taken ahead of the sums.
constexpr int kMaxBlocks = 64;            // (at most 32 InnerTrans blocks, 31 of the stack)
struct GradTail {
  ReduceBatch sums;
  NormJob norm[2 * kMaxBlocks];
  int blocks = 0; hipStream_t st;
  GradTail(hipStream_t st_) : st(st_) {}
  int add(int d, int f, const longer_block* blk, int count, float* g0, size_t stride) {      // grads of block i at g0 + i stride
    const GradLayout gl = grad_layout(d, f);
    if (blocks + count > kMaxBlocks) return api_error(LONGER_ERR_ARG, "more than %d blocks", kMaxBlocks);
    for (int i = 0; i < count; ++i, ++blocks) {
      const longer_block& b = blk[i];
      float* g = g0 + (size_t)i * stride;
      norm[2 * blocks] = {{(const __bf16*)b.wq, (const __bf16*)b.wk, (const __bf16*)b.wv}, (const __bf16*)b.ln1_g, (const __bf16*)b.ln1_b, g + gl.wq, g + gl.ln1_g, d, f};
      norm[2 * blocks + 1] = {{(const __bf16*)b.w1, nullptr, nullptr}, (const __bf16*)b.ln2_g, (const __bf16*)b.ln2_b, g + gl.w1, g + gl.ln2_g, d, f};
    }
    return 0;
  }
  int sum() {
    if (!sums.a.njobs) return 0;
    const int rc = launch(sums, st);
    sums = ReduceBatch{};
    return rc;
  }
  int finish() {
    int rc = sum();
    for (int first = 0; first < blocks && !rc; first += kNormBlocks) {
      NormGrads a = {};
      const int n = blocks - first < kNormBlocks ? blocks - first : kNormBlocks;
      int width = 0;
      for (int i = 0; i < 2 * n; ++i) { a.n[i] = norm[2 * first + i]; width = a.n[i].d > width ? a.n[i].d : width; }
      bw_norm_grads_kernel<<<dim3(width, 2 * n), 256, 0, st>>>(a);
      if (hipGetLastError() != hipSuccess) rc = api_error(LONGER_ERR_HIP, "LayerNorm gradient launch failed");
    }
    blocks = 0;
    return rc;
  }
};

static Workspace workspace(int layers, size_t ntok, int d, int f, int heads, size_t fwd_bytes, size_t ztmp_bytes) {
  Workspace w;
  size_t o = 0;
  auto take = [&](size_t bytes) { size_t at = o; o += up256(bytes); return at; };
  w.wcat = take((size_t)layers * d * 3 * d * 2);
  w.bcat = take((size_t)layers * up256((size_t)3 * d * 2));
  w.w1t = take((size_t)layers * d * f * 2);
  w.wcatt = take((size_t)layers * d * 3 * d * 2);
  w.wot = take((size_t)layers * d * d * 2);
  w.xin = take((size_t)layers * ntok * d * 4);
  w.n1 = take(ntok * d * 2);
  w.qkv = take(ntok * 3 * d * 2);
  w.o = take(ntok * d * 2);
  w.xmid = take(ntok * d * 4);
  w.n2 = take(ntok * d * 2);
  w.a = take(ntok * f * 2);
  w.dy = take(ntok * d * 4);
  w.dyb = take(ntok * d * 2);
  w.dh = take(ntok * f * 2);
  w.dn = take(ntok * d * 2);
  w.dxm = take(ntok * d * 4);
  w.dxmb = take(ntok * d * 2);
  w.dob = take(ntok * d * 2);
  w.dqkv = take(ntok * 3 * d * 2);
  w.stat = take(ntok * heads * 8);
  w.part = take(block_wgrads(d, f, ntok, RowsValid{}, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr).place(nullptr) * 4);
  w.lnpart = take((size_t)2 * kMaxLnBlocks * 2 * d * 4);
  w.fwd = take(fwd_bytes);
  w.fwd_bytes = fwd_bytes;
  w.ztmp = take(ztmp_bytes);
  w.total = o;
  return w;
}

// tiled: a block is one launch of the block kernel (bw_block.h); slots: B T K, padded: in whole workgroups of it
struct Dims { int d, f, heads, dh, layers, K, T; size_t ntok, slots, padded; bool tiled; };

// Workspace of the block kernel's form: tile blocks over the slots, block inputs [B][T K][d]
static Workspace tiled_workspace(const Dims& s, size_t fwd_bytes) {
  Workspace w = {};
  size_t o = 0;
  auto take = [&](size_t bytes) { size_t at = o; o += up256(bytes); return at; };
  const size_t n = s.padded, d = s.d, f = s.f;
  w.stream = take((size_t)s.layers * bw_block_segs_padded(s.d, s.f) * packed_seg_bytes(s.d, 2));
  w.xin = take((size_t)(s.layers - 1) * n * d * 4);
  w.rec = take(n / 32 * BlockRecord(s.d, s.f).size * 1024);
  w.dy = take(n * d * 4);
  w.part = take(block_wgrads_tiles(s.d, s.f, s.slots, RowsValid{}, nullptr, nullptr).place(nullptr) * 4);
  w.fwd = take(fwd_bytes);
  w.fwd_bytes = fwd_bytes;
  w.total = o;
  return w;
}

// the merge backward's workspace for a batch: with more than one block the fused forward kernel
// recomputes the block inputs (its scratch; a staging copy when L is not a multiple of K, whose rows
// then sit at [B, T K] instead of [B, L])
static Workspace merge_workspace(const longer_config* c, const Dims& s, int B, int L) {
  size_t fwd = 0, zt = 0;
  if (s.tiled) return tiled_workspace(s, s.layers > 1 ? least_workspace_bytes(c, B, L) : 0);
  if (s.layers > 1) {
    fwd = least_workspace_bytes(c, B, L);
    if (L % s.K) zt = (size_t)B * s.T * s.K * s.d * 4;
  }
  return workspace(s.layers, s.ntok, s.d, s.f, s.heads, fwd, zt);
}

static int check(const longer_config* c, int B, int L, Dims* s) {
  if (!c) return api_error(LONGER_ERR_ARG, "config is NULL");
  if (c->dtype != LONGER_BF16) return api_error(LONGER_ERR_ARG, "the backward pass is mixed precision: dtype must be LONGER_BF16");
  if (c->act != LONGER_ACT_GELU_ERF && c->act != LONGER_ACT_RELU) return api_error(LONGER_ERR_ARG, "act %d unknown", c->act);
  if (c->merge != LONGER_MERGE_MEAN && c->merge != LONGER_MERGE_CONCAT) return api_error(LONGER_ERR_ARG, "merge %d unknown", c->merge);
  if (c->K <= 0 || c->K > kMaxGroup || 32 % c->K) return api_error(LONGER_ERR_ARG, "K=%d must divide 32", c->K);
  if (c->d <= 0 || c->d % 32) return api_error(LONGER_ERR_ARG, "d=%d must be a positive multiple of 32", c->d);
  int d = c->d;
  if (c->merge == LONGER_MERGE_CONCAT) {
    if (d % c->K) return api_error(LONGER_ERR_ARG, "concat merge: K=%d must divide d=%d", c->K, d);
    d /= c->K;
  }
  if (d != 32 && d != 64 && d != 128 && d != 256) return api_error(LONGER_ERR_ARG, "InnerTrans width %d unsupported (32, 64, 128 or 256)", d);
  if (c->inner_layers <= 0 || c->inner_layers > 32) return api_error(LONGER_ERR_ARG, "inner_layers=%d out of range", c->inner_layers);
  if (c->inner_heads <= 0 || d % c->inner_heads) return api_error(LONGER_ERR_ARG, "inner_heads=%d must divide the InnerTrans width %d", c->inner_heads, d);
  const int dh = d / c->inner_heads;
  if (dh != 16 && dh != 32) return api_error(LONGER_ERR_ARG, "head width %d unsupported (16 or 32)", dh);
  if (c->ffn_mult <= 0 || c->ffn_mult * d > 2048) return api_error(LONGER_ERR_ARG, "ffn_mult=%d: the FFN hidden width must be at most 2048", c->ffn_mult);
  if (!(c->ln_eps > 0.f)) return api_error(LONGER_ERR_ARG, "ln_eps must be positive");
  if (B <= 0 || L <= 0) return api_error(LONGER_ERR_ARG, "B=%d, L=%d must be positive", B, L);
  const long long ntok = (long long)B * L;
  if (ntok * c->inner_heads >= (1ll << 31) - 256 || ntok * d * c->ffn_mult >= (1ll << 40))
    return api_error(LONGER_ERR_ARG, "B * L = %lld token rows are too many for one call; split the batch", ntok);
  s->d = d; s->f = c->ffn_mult * d; s->heads = c->inner_heads; s->dh = dh; s->layers = c->inner_layers;
  s->K = c->K; s->T = (L + c->K - 1) / c->K; s->ntok = (size_t)ntok;
  // The block kernel holds a tile's rows and two gradients of them in registers: 192 fp32 values per lane at width
  // 128, more than there are at 256.  It counts slots in 32 bits.
  s->slots = (size_t)B * s->T * s->K;
  s->padded = (s->slots + 32 * kBlkWaves - 1) / (32 * kBlkWaves) * (32 * kBlkWaves);
  s->tiled = d <= 128 && s->slots < ((size_t)1 << 31) - 256;
  return 0;
}

static bool aligned16(const void* p) { return ((uintptr_t)p & 15) == 0; }

static int launched(const char* what) {
  return hipGetLastError() == hipSuccess ? 0 : api_error(LONGER_ERR_HIP, "%s launch failed", what);
}

static int gemm(hipStream_t st, GemmArgs g) {
  if (!aligned16(g.A) || !aligned16(g.B) || g.lda % 8 || g.ldb % 8) return api_error(LONGER_ERR_ARG, "backward GEMM operand misaligned");
  const int ntm = (g.M + 127) / 128, ntn = (g.N + 127) / 128;
  dim3 grid((unsigned)(((ntm + 7) / 8) * 8 * ntn));            // see the tile order in the kernel
  if ((g.Kc == 32 || g.Kc == 64 || g.Kc == 128) &&
      (g.epi == EPI_FFN_MID || g.epi == EPI_BF16 || g.epi == EPI_RES_F32 || g.epi == EPI_F32)) {
    if (g.epi == EPI_FFN_MID && (!aligned16(g.A2) || !aligned16(g.B2) || g.lda2 % 8 || g.ldb2 % 8))
      return api_error(LONGER_ERR_ARG, "backward GEMM operand misaligned");
    // one workgroup per compute unit, each walking over row tiles for its 128 columns
    int P = (kComputeUnits / ntn) / 8 * 8;
    if (P < 8) P = 8;
    if (P > ((ntm + 7) / 8) * 8) P = ((ntm + 7) / 8) * 8;
    dim3 pg((unsigned)(P * ntn));
    const bool dual = g.epi == EPI_FFN_MID;
#define LONGER_ROWGEMM(KK) (dual ? bw_rowgemm_kernel<KK, true><<<pg, 512, 0, st>>>(g, P) : bw_rowgemm_kernel<KK, false><<<pg, 512, 0, st>>>(g, P))
    if (g.Kc == 128) LONGER_ROWGEMM(128); else if (g.Kc == 64) LONGER_ROWGEMM(64); else LONGER_ROWGEMM(32);
#undef LONGER_ROWGEMM
    return launched("backward row GEMM");
  }
  if (g.epi == EPI_FFN_MID) {
    if (!aligned16(g.A2) || !aligned16(g.B2) || g.lda2 % 8 || g.ldb2 % 8)
      return api_error(LONGER_ERR_ARG, "backward GEMM operand misaligned");
    bw_gemm_kernel<true><<<grid, 256, 0, st>>>(g);
  } else bw_gemm_kernel<false><<<grid, 256, 0, st>>>(g);
  return launched("backward GEMM");
}

// y = x W (+ epilogue) with W handed over transposed, wt [n][kc]: both operands contraction-contiguous
static int gemm_rows_wt(hipStream_t st, const __bf16* x, int kc, const __bf16* wt, int n, size_t ntok, int epi,
                        void* out, const __bf16* bias, const float* res, RowsValid rows) {
  GemmArgs g = {};
  g.rows = rows;
  g.A = x; g.lda = kc; g.B = wt; g.ldb = kc; g.M = (int)ntok; g.N = n; g.Kc = kc;
  g.epi = epi; g.out = out; g.ldo = n; g.bias = bias; g.res = res;
  return gemm(st, g);
}
// dx = dy W^T: dy [ntok][kc], W [n][kc] row-major (the forward's [in = n][out = kc])
static int gemm_rows_t(hipStream_t st, const __bf16* dy, int kc, const __bf16* W, int n, size_t ntok, int epi, void* out, RowsValid rows) {
  GemmArgs g = {};
  g.rows = rows;
  g.A = dy; g.lda = kc; g.B = W; g.ldb = kc; g.M = (int)ntok; g.N = n; g.Kc = kc;
  g.epi = epi; g.out = out; g.ldo = n;
  return gemm(st, g);
}
// The middle of the FFN's backward in one launch: v = x W1 + b1 (recomputed, not stored), g = dy W2^T,
// a_out = bf16(act(v)), dh_out = bf16(g act'(v)).  x, dy [ntok][d]; w1t = W1 transposed, [f][d]; w2 [f][d].
static int gemm_ffn_mid(hipStream_t st, const __bf16* x, const __bf16* dy, int d, const __bf16* w1t, const __bf16* w2, int f,
                        const __bf16* b1, size_t ntok, int act, __bf16* dh_out, __bf16* a_out, RowsValid rows) {
  GemmArgs g = {};
  g.rows = rows;
  g.A = x; g.lda = d; g.B = w1t; g.ldb = d; g.A2 = dy; g.lda2 = d; g.B2 = w2; g.ldb2 = d;
  g.M = (int)ntok; g.N = f; g.Kc = d;
  g.epi = EPI_FFN_MID; g.act = act; g.out = dh_out; g.out2 = a_out; g.ldo = f; g.bias = b1;
  return gemm(st, g);
}
static int transpose(hipStream_t st, const __bf16* in, __bf16* out, int rows, int cols) {
  bw_transpose_kernel<<<dim3((cols + 31) / 32, (rows + 31) / 32), 256, 0, st>>>(in, out, rows, cols);
  return launched("transpose");
}
static void ln_fwd(hipStream_t st, unsigned grid, int d, const float* x, const __bf16* g, const __bf16* b, __bf16* out,
                   int ntok, float eps, RowsValid rows = RowsValid{nullptr, 0}) {
  switch (d) {
    case 32: bw_ln_fwd_kernel<8><<<grid, 256, 0, st>>>(x, g, b, out, ntok, eps, rows); break;
    case 64: bw_ln_fwd_kernel<16><<<grid, 256, 0, st>>>(x, g, b, out, ntok, eps, rows); break;
    case 128: bw_ln_fwd_kernel<32><<<grid, 256, 0, st>>>(x, g, b, out, ntok, eps, rows); break;
    default: bw_ln_fwd_kernel<64><<<grid, 256, 0, st>>>(x, g, b, out, ntok, eps, rows); break;
  }
}
// part: the launch's partial gain / shift gradients, [grid][2 d]
static int ln_bwd(hipStream_t st, unsigned grid, int d, const __bf16* dn, const float* x, const __bf16* g, const float* dres,
                  float* dx, __bf16* dxb, float* part, int ntok, float eps, RowsValid rows = RowsValid{nullptr, 0}) {
  switch (d) {
    case 32: bw_ln_bwd_kernel<8><<<grid, 256, 0, st>>>(dn, x, g, dres, dx, dxb, part, ntok, eps, rows); break;
    case 64: bw_ln_bwd_kernel<16><<<grid, 256, 0, st>>>(dn, x, g, dres, dx, dxb, part, ntok, eps, rows); break;
    case 128: bw_ln_bwd_kernel<32><<<grid, 256, 0, st>>>(dn, x, g, dres, dx, dxb, part, ntok, eps, rows); break;
    default: bw_ln_bwd_kernel<64><<<grid, 256, 0, st>>>(dn, x, g, dres, dx, dxb, part, ntok, eps, rows); break;
  }
  return launched("LayerNorm backward");
}

static unsigned flat_grid(size_t n) {
  size_t b = (n + 255) / 256;
  return (unsigned)(b > 65536 ? 65536 : (b ? b : 1));
}

#define BW_TRY(x) do { int rc_ = (x); if (rc_) return rc_; } while (0)

// the block kernel's weights, all blocks' streams one after the other
static void pack_tiled(PackBatch& pk, const longer_block* inner, const Dims& s) {
  const int d = s.d, f = s.f;
  for (int l = 0; l < s.layers; ++l) {
    const longer_block& b = inner[l];
    const int NT = d / 32, NC = f / 32, o = l * bw_block_segs_padded(d, f), c = o + 4 * NT, k = c + 3 * NC;
    const void* qkv[3] = {b.wq, b.wk, b.wv};
    for (int i = 0; i < 3; ++i) pk.add(qkv[i], d, 1, false, NT, o + i, 3);
    pk.add(b.wo, d, 1, false, NT, o + 3 * NT, 1);
    pk.add(b.w1, f, 1, false, NC, c, 3);              // hidden values, their gradient, back through W1
    pk.add(b.w2, 1, d, false, NC, c + 1, 3);
    pk.add(b.w1, 1, f, true, NC, c + 2, 3);
    pk.add(b.wo, 1, d, false, NT, k, 4);              // back through W_O and, 32 features at a time, W_Q, W_K, W_V
    for (int i = 0; i < 3; ++i) pk.add(qkv[i], 1, d, true, NT, k + 1 + i, 4);
  }
}

static int run_tiled(const longer_config* c, const longer_block* inner, const void* H, const int32_t* lens, int B, int L,
                     const float* dM, float* dH, float* grads, char* ws, hipStream_t st, const Dims& s, bool inputs_kept, GradTail* tail) {
  const int d = s.d, f = s.f;
  const Workspace w = merge_workspace(c, s, B, L);
  const GradLayout gl = grad_layout(d, f);
  const RowsValid rv = {lens, s.T * s.K};
  const size_t stream_elems = (size_t)bw_block_segs_padded(d, f) * packed_seg_bytes(d, 2) / 2;
  auto at = [&](size_t o) { return (__bf16*)(ws + o); };
  if (!tail) {                                         // (a whole training step has packed them already)
    PackBatch pk(d, at(w.stream), st);
    pack_tiled(pk, inner, s);
    BW_TRY(pk.flush());
  }
  GradTail own(st);
  GradTail& t = tail ? *tail : own;
  // block inputs, by the fused forward kernel (its fp32 residual stream after l blocks is block l's input)
  auto xin = [&](int l) { return (float*)(ws + w.xin) + (size_t)(l - 1) * s.padded * d; };
  // unless the forward merge of the same call left them there
  for (int l = 1; l < s.layers && !inputs_kept; ++l) BW_TRY(inner_chain_f32(c, inner, l, H, lens, B, L, xin(l), ws + w.fwd, w.fwd_bytes, st));

  for (int l = s.layers - 1; l >= 0; --l) {
    const longer_block& b = inner[l];
    float* g = grads + (size_t)l * gl.total;
    BlockBwParams p = {};
    p.wstream = ws + w.stream + (size_t)l * stream_elems * 2;
    p.ln1_g = (const __bf16*)b.ln1_g; p.ln1_b = (const __bf16*)b.ln1_b; p.bq = (const __bf16*)b.bq; p.bv = (const __bf16*)b.bv;
    p.bo = (const __bf16*)b.bo; p.ln2_g = (const __bf16*)b.ln2_g; p.ln2_b = (const __bf16*)b.ln2_b; p.b1 = (const __bf16*)b.b1;
    p.lens = lens; p.B = B; p.L = L; p.K = s.K; p.T = s.T; p.f = f; p.act = c->act; p.eps = c->ln_eps;
    p.x = l ? (const void*)xin(l) : H; p.x_f32 = l != 0;
    p.dM = l == s.layers - 1 ? dM : nullptr; p.concat = c->merge == LONGER_MERGE_CONCAT;
    p.dy = (const float*)(ws + w.dy);
    p.rec = at(w.rec);
    p.dx = l ? (float*)(ws + w.dy) : dH; p.dx_rows = l == 0;      // (dy in place: a tile's values are read before they are replaced)
    // (the groups' operands behind the records, which are smaller by more than that)
    const bool grouped = l == s.layers - 1 && !p.concat && group_operands(d, s.K, lens != nullptr);
    GroupOperands go = {};
    if (grouped) {
      p.gx = p.rec + s.padded / 32 * BlockRecord(d, f, true).size * 512;
      p.gy = p.gx + group_tiles(s.padded, s.K) * (2 * f / 16) * 512;
      go = GroupOperands{p.gx, p.gy, B * s.T, s.K};
    }
    if (d == 32) bw_block_launch_32(s.dh, p, st);
    else if (d == 64) bw_block_launch_64(s.dh, p, st);
    else bw_block_launch_128(s.dh, p, st);
    BW_TRY(launched("block backward"));
    WgradBatch wg = block_wgrads_tiles(d, f, s.slots, rv, p.rec, g, grouped ? &go : nullptr);
    BW_TRY(launch(wg, (float*)(ws + w.part), st));
    t.sums.add(wg);
    BW_TRY(t.sum());
  }
  BW_TRY(t.add(d, f, inner, s.layers, grads, gl.total));
  return t.finish();
}

static int run(const longer_config* c, const longer_block* inner, const void* H, const int32_t* lens, int B, int L,
               const float* dM, float* dH, float* grads, char* ws, hipStream_t st, const Dims& s, bool inputs_kept = false,
               GradTail* tail = nullptr) {
  if (s.tiled) return run_tiled(c, inner, H, lens, B, L, dM, dH, grads, ws, st, s, inputs_kept, tail);
  if (tail) BW_TRY(tail->finish());
  const int d = s.d, f = s.f;
  const size_t nt = s.ntok;
  const Workspace w = merge_workspace(c, s, B, L);
  const GradLayout gl = grad_layout(d, f);
  const RowGeom q = {lens, L, s.K, (int)nt};
  const RowsValid rv = {lens, L};            // padded token rows are left out (lens NULL: there are none)
  auto xin = [&](int l) { return (float*)(ws + w.xin) + (size_t)l * nt * d; };
  auto wcat = [&](int l) { return (__bf16*)(ws + w.wcat) + (size_t)l * d * 3 * d; };
  auto bcat = [&](int l) { return (__bf16*)(ws + w.bcat + (size_t)l * up256((size_t)3 * d * 2)); };
  __bf16* n1 = (__bf16*)(ws + w.n1);   __bf16* qkv = (__bf16*)(ws + w.qkv); __bf16* o = (__bf16*)(ws + w.o);
  float* xmid = (float*)(ws + w.xmid); __bf16* n2 = (__bf16*)(ws + w.n2);
  auto w1t = [&](int l) { return (__bf16*)(ws + w.w1t) + (size_t)l * d * f; };
  auto wcatt = [&](int l) { return (__bf16*)(ws + w.wcatt) + (size_t)l * d * 3 * d; };
  auto wot = [&](int l) { return (__bf16*)(ws + w.wot) + (size_t)l * d * d; };
  __bf16* a = (__bf16*)(ws + w.a);     float* dy = (float*)(ws + w.dy);     __bf16* dyb = (__bf16*)(ws + w.dyb);
  __bf16* dh = (__bf16*)(ws + w.dh);   __bf16* dn = (__bf16*)(ws + w.dn);   float* dxm = (float*)(ws + w.dxm);
  __bf16* dxmb = (__bf16*)(ws + w.dxmb); __bf16* dob = (__bf16*)(ws + w.dob); __bf16* dqkv = (__bf16*)(ws + w.dqkv);
  float2* stat = (float2*)(ws + w.stat);
  float* part = (float*)(ws + w.part);
  float* lnpart[2] = {(float*)(ws + w.lnpart), (float*)(ws + w.lnpart) + (size_t)kMaxLnBlocks * 2 * d};
  const unsigned ln_grid = ln_blocks(nt);
  const unsigned ah_grid = (unsigned)((nt * s.heads + 255) / 256);

  for (int l = 0; l < s.layers; ++l) {
    const longer_block& b = inner[l];
    bw_concat_qkv_kernel<<<64, 256, 0, st>>>((const __bf16*)b.wq, (const __bf16*)b.wk, (const __bf16*)b.wv, (const __bf16*)b.bq,
                                             (const __bf16*)b.bk, (const __bf16*)b.bv, wcat(l), bcat(l), d);
    BW_TRY(launched("weight concatenation"));
    BW_TRY(transpose(st, (const __bf16*)b.w1, w1t(l), d, f));
    BW_TRY(transpose(st, wcat(l), wcatt(l), d, 3 * d));
    BW_TRY(transpose(st, (const __bf16*)b.wo, wot(l), d, d));
  }
  bw_load_x0_kernel<<<flat_grid(nt * d / 4), 256, 0, st>>>((const __bf16*)H, xin(0), q, d);
  BW_TRY(launched("input load"));

  // one block forward from its input x, up to the FFN's input: intermediates into the workspace
  auto forward = [&](int l) -> int {
    const longer_block& b = inner[l];
    const float* x = xin(l);
    ln_fwd(st, ln_grid, d, x, (const __bf16*)b.ln1_g, (const __bf16*)b.ln1_b, n1, (int)nt, c->ln_eps, rv);
    BW_TRY(launched("LayerNorm"));
    BW_TRY(gemm_rows_wt(st, n1, d, wcatt(l), 3 * d, nt, EPI_BF16, qkv, bcat(l), nullptr, rv));
    group_attn(0, s.dh, s.K, ah_grid, st, qkv, nullptr, o, nullptr, q, d, s.heads);
    BW_TRY(launched("group attention"));
    BW_TRY(gemm_rows_wt(st, o, d, wot(l), d, nt, EPI_RES_F32, xmid, (const __bf16*)b.bo, x, rv));
    ln_fwd(st, ln_grid, d, xmid, (const __bf16*)b.ln2_g, (const __bf16*)b.ln2_b, n2, (int)nt, c->ln_eps, rv);
    return launched("LayerNorm");
  };

  // the chain of block inputs (recomputed: nothing is kept from a forward call), by the fused forward
  // kernel: its fp32 residual stream after l + 1 blocks is block l + 1's input
  for (int l = 0; l + 1 < s.layers; ++l) {
    const bool direct = L % s.K == 0;
    float* z = direct ? xin(l + 1) : (float*)(ws + w.ztmp);
    BW_TRY(inner_chain_f32(c, inner, l + 1, H, lens, B, L, z, ws + w.fwd, w.fwd_bytes, st));
    if (!direct) {
      bw_take_rows_kernel<<<flat_grid(nt * d / 4), 256, 0, st>>>(z, xin(l + 1), B, L, s.T * s.K, d);
      BW_TRY(launched("row copy"));
    }
  }

  bw_merge_bwd_kernel<<<flat_grid(nt * d / 4), 256, 0, st>>>(dM, dy, dyb, q, d, s.T, c->merge == LONGER_MERGE_CONCAT);
  BW_TRY(launched("merge gradient"));

  for (int l = s.layers - 1; l >= 0; --l) {
    const longer_block& b = inner[l];
    float* g = grads + (size_t)l * gl.total;
    BW_TRY(forward(l));                          // this block's intermediates, from its input alone
    // FFN: y = xmid + act(n2 W1 + b1) W2 + b2; the hidden pre-activation is formed inside the launch
    // that takes its gradient, and only the activated values and the hidden gradient reach memory
    BW_TRY(gemm_ffn_mid(st, n2, dyb, d, w1t(l), (const __bf16*)b.w2, f, (const __bf16*)b.b1, nt, c->act, dh, a, rv));
    BW_TRY(gemm_rows_t(st, dh, f, (const __bf16*)b.w1, d, nt, EPI_BF16, dn, rv));
    BW_TRY(ln_bwd(st, ln_grid, d, dn, xmid, (const __bf16*)b.ln2_g, dy, dxm, dxmb, lnpart[1], (int)nt, c->ln_eps, rv));
    // attention: xmid = x + att W_O + b_O
    BW_TRY(gemm_rows_t(st, dxmb, d, (const __bf16*)b.wo, d, nt, EPI_BF16, dob, rv));
    if (L % s.K == 0 && 256 % s.heads == 0 && (256 / s.heads) % s.K == 0) {     // every group inside one workgroup's rows
      group_attn(3, s.dh, s.K, ah_grid, st, qkv, dob, dqkv, stat, q, d, s.heads);
    } else {
      group_attn(1, s.dh, s.K, ah_grid, st, qkv, dob, dqkv, stat, q, d, s.heads);
      group_attn(2, s.dh, s.K, ah_grid, st, qkv, dob, dqkv, stat, q, d, s.heads);
    }
    BW_TRY(launched("group attention backward"));
    // every matrix of the block at once, now that all operands are there (dyb goes to the next block's below)
    WgradBatch wg = block_wgrads(d, f, nt, rv, n1, dqkv, o, dxmb, n2, dh, a, dyb, g);
    BW_TRY(launch(wg, part, st));
    BW_TRY(gemm_rows_t(st, dqkv, 3 * d, wcat(l), d, nt, EPI_BF16, dn, rv));
    // the gradient of this block's input is the upstream gradient of the block before it
    float* dx = l ? dy : dH;
    BW_TRY(ln_bwd(st, ln_grid, d, dn, xin(l), (const __bf16*)b.ln1_g, dxm, dx, l ? dyb : nullptr, lnpart[0],
                  (int)nt, c->ln_eps, rv));
    ReduceBatch rb;
    rb.add(wg);
    rb.add_ln(lnpart[0], (int)ln_grid, d, g + gl.ln1_g);
    rb.add_ln(lnpart[1], (int)ln_grid, d, g + gl.ln2_g);
    BW_TRY(launch(rb, st));
  }
  return 0;
}


// ------------------------------------------------------------------------------------
// Whole model: loss and every gradient (longer_forward_backward)
struct StackDims { int d, f, heads, dh, m, k, n, T, B, layers; size_t rq, rk; };   // layers = 1 + n_self

struct StackWs {
  size_t fwd_ws, Mb, dM;                  // forward token merge: its scratch, M (bf16), and the gradient handed to the merge
  size_t qdesc, kdesc, stream;
  size_t xs;                              // the input rows of layers 1 .. and the last one's output ([layers][rq][d])
  size_t qkv, stat, xmid, rec, per_layer; // every layer's intermediates are kept (per_layer bytes apart): the reduced stack is
                                          // small, only the merge is recomputed
  size_t kv, krec, o, dy, dxm, dob, dqkv, dkv, dR, part;
  size_t rqp, rkp;                        // rows in whole tiles
  size_t total;
};
// records of the cross layer's key rows: normalised rows, gradients of K and V
static int key_record(int d) { return 3 * d / 16; }
// Where each launch's weights start (segments).  Forward: [Q of the cross layer] | [tail of 0, head of 1] | ... | [tail of the
// last]; backward: [head of the last] | [tail of it, head of the one before] | ... | [Q]; then K / V of the cross layer, both ways.
struct StackStreams {
  int NT, NC, layers, kv_f, kv_b, total;
  StackStreams(int d, int f, int n) : NT(d / 32), NC(f / 32), layers(n) {
    kv_f = bwd_tail(0) + NT; kv_b = kv_f + 2 * NT; total = kv_b + 2 * NT;
  }
  int fwd_head(int l) const { return l == 0 ? 0 : fwd_tail(l) - 3 * NT; }
  int fwd_tail(int l) const { return NT + l * (NT + 2 * NC + 3 * NT); }
  int fwd_end() const { return fwd_tail(layers - 1) + NT + 2 * NC; }
  int bwd_head(int l) const { return fwd_end() + (layers - 1 - l) * (3 * NC + NT + 3 * NT); }
  int bwd_tail(int l) const { return bwd_head(l) + 3 * NC + NT; }
};
// The gradients of every matrix of the stack in one batch: the self layers' (per_layer bytes and `per_main` floats
// apart), then the cross layer's, whose keys and values contract over the key rows
static WgradBatch stack_wgrads(const StackDims& s, const StackWs& w, const char* ws, float* grads, size_t cross, size_t self0, size_t per_main) {
  const int d = s.d, f = s.f;
  const GradLayout gl = grad_layout(d, f);
  const BlockRecord r(d, f);
  const RowsValid all = {nullptr, 0};
  WgradBatch b(d, s.rq, true);
  const long long ls = (long long)(w.per_layer / 2), os = (long long)per_main;
  auto at = [&](int o, int l) { return (const __bf16*)(ws + w.rec + (size_t)l * w.per_layer) + (size_t)o * 512; };
  auto side = [&](int l, int n, float* g, size_t rows) {
    b.add(at(r.a, l), r.size, f, at(r.dyb, l), r.size, d, d, rows, all, g + gl.w2, n, ls, ls, os);
    b.add(at(r.xh2, l), r.size, d, at(r.dh, l), r.size, f, f, rows, all, g + gl.w1, n, ls, ls, os);
    b.add(at(r.o, l), r.size, d, at(r.dxmb, l), r.size, d, d, rows, all, g + gl.wo, n, ls, ls, os);
  };
  const int last = s.layers - 1;          // (its records hold the global rows alone, but for those of Q, K and V)
  const size_t rg = (size_t)s.B * s.m;
  if (s.layers > 1) {
    float* g = grads + self0;
    if (last > 1) side(1, last - 1, g, s.rq);
    side(last, 1, g + (size_t)(last - 1) * os, rg);
    b.add(at(r.xh1, 1), r.size, d, at(r.qkv, 1), r.size, 3 * d, d, s.rq, all, g + gl.wq, s.layers - 1, ls, ls, os);
  }
  float* g = grads + cross;
  side(0, 1, g, last ? s.rq : rg);
  b.add(at(r.xh1, 0), r.size, d, at(r.qkv, 0), r.size, d, d, s.rq, all, g + gl.wq);
  const __bf16* kr = (const __bf16*)(ws + w.krec);
  b.add(kr, key_record(d), d, kr + (size_t)(d / 16) * 512, key_record(d), 2 * d, d, s.rk, all, g + gl.wk);
  return b;
}
static StackWs stack_ws(const StackDims& s, size_t fwd_bytes) {
  StackWs w;
  size_t o = 0;
  auto take = [&](size_t bytes) { size_t at = o; o += up256(bytes); return at; };
  const size_t rq = s.rq, rk = s.rk, d = s.d, f = s.f;
  w.rqp = (rq + 31) / 32 * 32;
  w.rkp = (rk + 31) / 32 * 32;
  w.fwd_ws = take(fwd_bytes);
  w.Mb = take((size_t)s.B * s.T * d * 2);
  w.dM = take((size_t)s.B * s.T * d * 4);
  w.qdesc = take(rq * 4);
  w.kdesc = take(rk * 4);
  w.stream = take((size_t)StackStreams(s.d, s.f, s.layers).total * packed_seg_bytes(s.d, 2));
  w.xs = take((size_t)s.layers * rq * d * 4);
  const size_t layer0 = o;
  w.qkv = take(rq * 3 * d * 2);
  w.stat = take(rq * s.heads * 8);
  w.xmid = take(w.rqp * d * 4);
  w.rec = take(w.rqp / 32 * BlockRecord(s.d, s.f).size * 1024);
  w.per_layer = o - layer0;
  o += (size_t)(s.layers - 1) * w.per_layer;
  w.kv = take(rk * 2 * d * 2);
  w.krec = take(w.rkp / 32 * key_record(s.d) * 1024);
  w.o = take(rq * d * 2);
  w.dy = take(rq * d * 4);
  w.dxm = take(w.rqp * d * 4);
  w.dob = take(rq * d * 2);
  w.dqkv = take(rq * 3 * d * 2);
  w.dkv = take(rk * 2 * d * 2);
  w.dR = take(rk * d * 4);
  w.part = take(stack_wgrads(s, w, nullptr, nullptr, 0, 0, 0).place(nullptr) * 4);
  w.total = o;
  return w;
}

static int check_stack(const longer_config* c, int B, int L, StackDims* s) {
  if (c->q_learn && (c->k_uniform || ((uintptr_t)c->q_learn & 15))) return api_error(LONGER_ERR_ARG, "q_learn needs k_uniform = 0 and 16-byte alignment");
  if (c->gmask != LONGER_GMASK_FULL && c->gmask != LONGER_GMASK_CAUSAL) return api_error(LONGER_ERR_ARG, "gmask %d unknown", c->gmask);
  const int d = c->d;
  if (d != 32 && d != 64 && d != 128 && d != 256) return api_error(LONGER_ERR_ARG, "width %d unsupported (32, 64, 128 or 256)", d);
  if (c->heads <= 0 || d % c->heads || (d / c->heads != 16 && d / c->heads != 32))
    return api_error(LONGER_ERR_ARG, "heads=%d: head width must be 16 or 32", c->heads);
  if (c->ffn_mult * d > 2048) return api_error(LONGER_ERR_ARG, "ffn_mult=%d: the FFN hidden width must be at most 2048", c->ffn_mult);
  if (c->m <= 0 || c->k_recent <= 0 || c->n_self < 0 || c->n_self > 30) return api_error(LONGER_ERR_ARG, "m, k_recent, n_self out of range");
  if (c->k_uniform < 0 || c->k_uniform > c->k_recent) return api_error(LONGER_ERR_ARG, "k_uniform=%d must lie in [0, k_recent]", c->k_uniform);
  s->d = d; s->f = c->ffn_mult * d; s->heads = c->heads; s->dh = d / c->heads; s->m = c->m; s->k = c->k_recent;
  s->n = c->m + c->k_recent; s->T = (L + c->K - 1) / c->K; s->B = B; s->layers = 1 + c->n_self;
  s->rq = (size_t)B * s->n; s->rk = (size_t)B * (c->m + s->T);
  if (s->rk * (size_t)s->heads >= ((size_t)1 << 31) - 256) return api_error(LONGER_ERR_ARG, "too many key rows for one call; split the batch");
  return 0;
}

// layout of the gradient buffer: [InnerTrans blocks][cross block][self blocks][head_w (m d)][head_b (1), padded to 4]
// [learnable query tokens (k d), if the configuration has them]
struct ModelGrads { size_t inner, cross, self0, head_w, head_b, q_learn, total, per_main; };
static ModelGrads model_grads(const Dims& mi, const StackDims& s, bool learn) {
  ModelGrads g;
  g.inner = 0;
  g.cross = (size_t)mi.layers * grad_layout(mi.d, mi.f).total;
  g.per_main = grad_layout(s.d, s.f).total;
  g.self0 = g.cross + g.per_main;
  g.head_w = g.self0 + (size_t)(s.layers - 1) * g.per_main;
  g.head_b = g.head_w + (size_t)s.m * s.d;
  g.q_learn = (g.head_b + 1 + 3) & ~(size_t)3;
  g.total = g.q_learn + (learn ? (size_t)s.k * s.d : 0);
  return g;
}

static int run_model(const longer_config* c, const longer_weights* wts, const void* H, const void* G, const int32_t* lens,
                     int B, int L, const float* labels, float* loss, float* logits, float* dH, float* dG, float* grads,
                     char* ws, size_t fwd_bytes, hipStream_t st, const Dims& mi, const StackDims& s, float* block_inputs,
                     __bf16* block_stream, GradTail& tail) {
  const int d = s.d, f = s.f;
  const size_t rq = s.rq, rk = s.rk;
  const StackWs w = stack_ws(s, fwd_bytes);
  const ModelGrads mg = model_grads(mi, s, c->q_learn != nullptr);
  const GradLayout gl = grad_layout(d, f);
  const StackGeom geo = {lens, L, c->K, s.T, s.m, s.k, c->k_uniform, B, c->q_learn != nullptr};
  int* qdesc = (int*)(ws + w.qdesc);   int* kdesc = (int*)(ws + w.kdesc);
  __bf16* Mb = (__bf16*)(ws + w.Mb);   float* dM = (float*)(ws + w.dM);
  auto xs = [&](int l) { return (float*)(ws + w.xs) + (size_t)(l - 1) * rq * d; };
  auto blk = [&](int l) -> const longer_block& { return l == 0 ? wts->cross[0] : wts->self[l - 1]; };
  auto of = [&](size_t o, int l) { return ws + o + (size_t)l * w.per_layer; };      // a layer's own buffers
  auto bf = [](const void* q) { return (const __bf16*)q; };
  __bf16* kv = (__bf16*)(ws + w.kv);   __bf16* krec = (__bf16*)(ws + w.krec); __bf16* o = (__bf16*)(ws + w.o);
  float* dy = (float*)(ws + w.dy);     float* dxm = (float*)(ws + w.dxm);     __bf16* dob = (__bf16*)(ws + w.dob);
  __bf16* dqkv = (__bf16*)(ws + w.dqkv); __bf16* dkv = (__bf16*)(ws + w.dkv); float* dR = (float*)(ws + w.dR);
  const BlockRecord r(d, f);
  const StackStreams sg(d, f, s.layers);
  const int NT = d / 32, NC = f / 32, last = s.layers - 1;
  auto stream_at = [&](int seg) { return ws + w.stream + (size_t)seg * packed_seg_bytes(d, 2); };

  // ---- weights in the launches' order, row descriptors, zeros
  PackBatch pk(d, (__bf16*)(ws + w.stream), st);
  for (int l = 0; l < s.layers; ++l) {
    const longer_block& b = blk(l);
    const void* qkv[3] = {b.wq, b.wk, b.wv};
    const int mats = l ? 3 : 1, t = sg.fwd_tail(l) + NT, h = sg.bwd_head(l);
    for (int i = 0; i < mats; ++i) {
      pk.add(qkv[i], d, 1, false, NT, sg.fwd_head(l) + i, mats);
      pk.add(qkv[i], 1, d, true, NT, sg.bwd_tail(l) + i, mats);
    }
    for (int i = mats; i < 3; ++i) {
      pk.add(qkv[i], d, 1, false, NT, sg.kv_f + i - 1, 2);
      pk.add(qkv[i], 1, d, true, NT, sg.kv_b + i - 1, 2);
    }
    pk.add(b.wo, d, 1, false, NT, sg.fwd_tail(l), 1);
    pk.add(b.w1, f, 1, false, NC, t, 2);
    pk.add(b.w2, d, 1, true, NC, t + 1, 2);
    pk.add(b.w1, f, 1, false, NC, h, 3);              // hidden values, their gradient, back through W1
    pk.add(b.w2, 1, d, false, NC, h + 1, 3);
    pk.add(b.w1, 1, f, true, NC, h + 2, 3);
    pk.add(b.wo, 1, d, false, NT, h + 3 * NC, 1);
  }
  if (block_stream) {
    pk.into(mi.d, block_stream);
    pack_tiled(pk, wts->inner, mi);
  }
  // (added to with atomics: the head's gradients, the learnable query tokens', the loss)
  const Prepare prepare = {geo, qdesc, kdesc, grads + mg.head_w, mg.total - mg.head_w, loss};
  BW_TRY(pk.flush(&prepare));

  // ---- forward from the inputs: merged tokens (the fused forward kernel; the merge's intermediates are
  // recomputed later by its own backward pass), then the stack, keeping every layer's intermediates
  int rc = block_inputs ? merge_keep_f32(c, wts->inner, H, lens, B, L, Mb, block_inputs, mi.padded * mi.d, ws + w.fwd_ws, fwd_bytes, st)
                        : longer_token_merge(c, wts->inner, H, lens, B, L, Mb, ws + w.fwd_ws, fwd_bytes, st);
  if (rc) return rc;
  // the cross layer's rows: R = [G; M] (merged tokens past T_u are zeros) and O = [G; the slots' merged tokens]
  const StackSource key_rows = {(const __bf16*)G, Mb, nullptr, nullptr, s.m + s.T, s.m, s.T};
  const StackSource query_rows = {(const __bf16*)G, Mb, (const __bf16*)c->q_learn, qdesc, s.n, s.m, s.T};
  auto attn = [&](int l) {
    SetAttn t;
    const __bf16* qkv = (const __bf16*)of(w.qkv, l);
    t.qdesc = qdesc; t.nq = l == last ? s.m : s.n; t.qrows = s.n; t.B = B; t.heads = s.heads; t.gmask = c->gmask;
    if (l == 0) { t.q = qkv; t.qpitch = d; t.k = kv; t.v = kv + d; t.kvpitch = 2 * d; t.kdesc = kdesc; t.nk = s.m + s.T; }
    else { t.q = qkv; t.qpitch = 3 * d; t.k = qkv + d; t.v = qkv + 2 * d; t.kvpitch = 3 * d; t.kdesc = qdesc; t.nk = s.n; }
    return t;
  };
  auto attn_forward = [&](int l) -> int {
    float2* stat = (float2*)of(w.stat, l);
    if (s.dh == 16) set_attn_forward<16>(st, attn(l), o, d, stat); else set_attn_forward<32>(st, attn(l), o, d, stat);
    return launched("attention");
  };
  auto attn_backward = [&](int l, int dqpitch, __bf16* dk, __bf16* dv, int dkvpitch) -> int {
    float2* stat = (float2*)of(w.stat, l);
    if (s.dh == 16) set_attn_backward<16>(st, attn(l), dob, d, dqkv, dqpitch, dk, dv, dkvpitch, stat);
    else set_attn_backward<32>(st, attn(l), dob, d, dqkv, dqpitch, dk, dv, dkvpitch, stat);
    return launched("attention backward");
  };
  auto fwd = [&](const StackFwd& p, const StackFwd& k) -> int {
    if (d == 32) bw_stack_fwd_32(p, k, st); else if (d == 64) bw_stack_fwd_64(p, k, st);
    else if (d == 128) bw_stack_fwd_128(p, k, st); else bw_stack_fwd_256(p, k, st);
    return launched("stack forward");
  };
  auto bwd = [&](const StackBwd& p, const StackBwd& k) -> int {
    if (d == 32) bw_stack_bwd_32(p, k, st); else if (d == 64) bw_stack_bwd_64(p, k, st);
    else if (d == 128) bw_stack_bwd_128(p, k, st); else bw_stack_bwd_256(p, k, st);
    return launched("stack backward");
  };
  const StackRows globals = {s.m, s.n};
  // forward: [head of 0 (and its keys)], attention, [tail of l, head of l + 1], ...
  for (int l = -1; l <= last; ++l) {
    StackFwd p = {};
    p.rows = (int)rq; p.f = f; p.act = c->act; p.eps = c->ln_eps;
    if (l >= 0) {
      const longer_block& b = blk(l);
      BW_TRY(attn_forward(l));
      p.wstream = stream_at(sg.fwd_tail(l));
      if (l) p.x = xs(l); else p.from = query_rows;
      p.o = o; p.bo = bf(b.bo); p.ln2_g = bf(b.ln2_g); p.ln2_b = bf(b.ln2_b); p.b1 = bf(b.b1); p.b2 = bf(b.b2);
      p.desc = qdesc; p.xmid = (float*)of(w.xmid, l); p.y = xs(l + 1); p.rec = (__bf16*)of(w.rec, l);
      if (l == last) { p.only = globals; p.rows = (int)((size_t)B * s.m); }
    } else {
      p.wstream = stream_at(sg.fwd_head(0)); p.from = query_rows;
    }
    if (l < last) {
      const longer_block& b = blk(l + 1);
      p.mats = l < 0 ? 1 : 3;
      p.ln1_g = bf(b.ln1_g); p.ln1_b = bf(b.ln1_b); p.bias[0] = bf(b.bq); p.bias[1] = bf(b.bk); p.bias[2] = bf(b.bv);
      p.out = (__bf16*)of(w.qkv, l + 1); p.ldo = p.mats * d; p.rec1 = (__bf16*)of(w.rec, l + 1); p.rec1_size = r.size; p.rec1_xh = r.xh1;
    }
    StackFwd k = {};
    if (l < 0) {
      const longer_block& b = blk(0);
      k.rows = (int)rk; k.f = f; k.eps = c->ln_eps; k.wstream = stream_at(sg.kv_f); k.from = key_rows;
      k.ln1_g = bf(b.ln1_g); k.ln1_b = bf(b.ln1_b); k.bias[0] = bf(b.bk); k.bias[1] = bf(b.bv);
      k.mats = 2; k.out = kv; k.ldo = 2 * d; k.rec1 = krec; k.rec1_size = key_record(d); k.rec1_xh = 0;
    }
    BW_TRY(fwd(p, k));
  }

  // ---- head and loss (Eq. 1-2), and the gradient of the stack's output
  bw_head_kernel<<<B, 256, 0, st>>>(xs(s.layers), bf(wts->head_w), bf(wts->head_b), labels, B, s.n, s.m, d,
                                    logits, loss, dy, grads + mg.head_w, grads + mg.head_b);
  BW_TRY(launched("head"));

  // ---- back: [head of the last], attention backward, [tail of l, head of l - 1], ..., [tail of 0 (and its keys)]
  for (int l = last + 1; l >= 0; --l) {
    StackBwd p = {};
    p.rows = (int)rq; p.f = f; p.act = c->act; p.eps = c->ln_eps;
    if (l <= last) {
      // (the cross layer's keys are rows of their own; a self layer's dq, dk, dv lie side by side)
      BW_TRY(l ? attn_backward(l, 3 * d, dqkv + d, dqkv + 2 * d, 3 * d) : attn_backward(l, d, dkv, dkv + d, 2 * d));
      p.mats = l ? 3 : 1; p.wstream = stream_at(sg.bwd_tail(l));
      if (l) p.x = xs(l); else p.from = query_rows;
      p.dqkv = dqkv; p.ldq = p.mats * d; p.ln1_g = bf(blk(l).ln1_g); p.dxm_in = l == last ? (const float*)of(w.xmid, last) : dxm;
      p.rec1 = (__bf16*)of(w.rec, l); p.rec1_size = r.size; p.rec1_dqkv = r.qkv; p.dx = dy;
      if (l == last) p.head = globals;
    } else {
      p.wstream = stream_at(sg.bwd_head(last)); p.dy = dy; p.only = globals; p.rows = (int)((size_t)B * s.m);
    }
    if (l > 0) {
      const longer_block& b = blk(l - 1);
      p.desc = qdesc; p.xmid = (const float*)of(w.xmid, l - 1); p.ln2_g = bf(b.ln2_g); p.ln2_b = bf(b.ln2_b); p.b1 = bf(b.b1);
      // (the last layer's takes the place of its rows, tile by tile: the launch that reads it writes dxm in tiles of all rows)
      p.dxm = l > last ? (float*)of(w.xmid, last) : dxm; p.dob = dob; p.rec = (__bf16*)of(w.rec, l - 1);
    }
    StackBwd k = {};
    if (l == 0) {
      k.rows = (int)rk; k.f = f; k.eps = c->ln_eps; k.wstream = stream_at(sg.kv_b); k.mats = 2;
      k.dqkv = dkv; k.ldq = 2 * d; k.from = key_rows; k.ln1_g = bf(blk(0).ln1_g); k.rec1 = krec; k.rec1_size = key_record(d);
      k.rec1_dqkv = d / 16; k.dx = dR;
    }
    BW_TRY(bwd(p, k));
  }
  // ---- parameter gradients of all layers: one launch; the sums of its partial results and the LayerNorms' from those go with the merge's
  WgradBatch wg = stack_wgrads(s, w, ws, grads, mg.cross, mg.self0, mg.per_main);
  BW_TRY(launch(wg, (float*)(ws + w.part), st));
  tail.sums.add(wg);
  BW_TRY(tail.add(d, f, wts->cross, 1, grads + mg.cross, mg.per_main));
  if (s.layers > 1) BW_TRY(tail.add(d, f, wts->self, s.layers - 1, grads + mg.self0, mg.per_main));
  // ---- gradients of the stack's inputs: global tokens (query rows and key rows), merged tokens (key
  // rows, plus the query slots that hold them)
  bw_split_grad_kernel<<<flat_grid(rk * d / 4), 256, 0, st>>>(geo, d, dy, dR, dG, dM);
  if (geo.k_uniform || geo.learn)
    bw_slot_grad_kernel<<<flat_grid((size_t)B * s.k * d / 4), 256, 0, st>>>(geo, d, dy, qdesc, dM, grads + mg.q_learn);
  BW_TRY(launched("gradient routing"));
  return 0;
}


// ------------------------------------------------------------------------------------
// Input generation backward (longer_input_generation_backward)
// Widths 64 and 128: one launch over tiles (bw_input.h); others: kernels over row-major [token, feature] tensors.
static bool input_tiled(int d) { return d == 64 || d == 128; }
struct InputWs { size_t w1t, x, a, dyb, dh, dx, rec, part, total; };      // tiled: w1t holds the weight stream, rec the records
static WgradBatch input_wgrads(int d, int f, size_t ntok, RowsValid rv, const __bf16* x, const __bf16* dh, const __bf16* a,
                               const __bf16* dyb, float* gw1, float* gw2) {
  WgradBatch w(d, ntok);
  w.add(a, f, f, dyb, d, d, d, ntok, rv, gw2);          // H = a w2 + b2
  w.add(x, d, d, dh, f, f, f, ntok, rv, gw1);
  return w;
}
static WgradBatch input_wgrads_tiles(int d, int f, size_t ntok, RowsValid rv, const __bf16* rec, float* gw1, float* gw2) {
  const InputRecord r(d, f);
  auto at = [&](int o) { return rec + (size_t)o * 512; };
  WgradBatch w(d, ntok, true);
  w.add(at(r.a), r.size, f, at(r.dyb), r.size, d, d, ntok, rv, gw2);
  w.add(at(r.x), r.size, d, at(r.dh), r.size, f, f, ntok, rv, gw1);
  return w;
}
static InputWs input_ws(size_t ntok, int d, int f) {
  InputWs w = {};
  size_t o = 0;
  auto take = [&](size_t bytes) { size_t at = o; o += up256(bytes); return at; };
  if (input_tiled(d)) {
    const size_t tiles = (ntok + 32 * kBlkWaves - 1) / (32 * kBlkWaves) * kBlkWaves;      // whole workgroups
    w.w1t = take((size_t)bw_input_segs_padded(f) * d * 64);
    w.rec = take(tiles * InputRecord(d, f).size * 1024);
    w.part = take(input_wgrads_tiles(d, f, ntok, RowsValid{}, nullptr, nullptr, nullptr).place(nullptr) * 4);
  } else {
    w.w1t = take((size_t)d * f * 2);
    w.x = take(ntok * d * 2);
    w.a = take(ntok * f * 2);
    w.dyb = take(ntok * d * 2);
    w.dh = take(ntok * f * 2);
    w.dx = take(ntok * d * 4);
    w.part = take(input_wgrads(d, f, ntok, RowsValid{}, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr).place(nullptr) * 4);
  }
  w.total = o;
  return w;
}
// gradient buffer: [pos L de][w1 d f][b1 f][w2 f d][b2 d]
struct InputGrads { size_t pos, w1, b1, w2, b2, total; };
static InputGrads input_grads(int L, int d, int f, int de) {
  InputGrads g;
  g.pos = 0; g.w1 = (size_t)L * de; g.b1 = g.w1 + (size_t)d * f; g.w2 = g.b1 + f; g.b2 = g.w2 + (size_t)f * d;
  g.total = g.b2 + d;
  return g;
}
static int check_input_bw(const longer_config* c, int B, int L, int de, int* d, int* f) {
  if (!c) return api_error(LONGER_ERR_ARG, "config is NULL");
  if (c->dtype != LONGER_BF16) return api_error(LONGER_ERR_ARG, "the backward pass is mixed precision: dtype must be LONGER_BF16");
  if (c->merge != LONGER_MERGE_MEAN) return api_error(LONGER_ERR_ARG, "input generation feeds the mean merge (H of width d)");
  if (c->act != LONGER_ACT_GELU_ERF && c->act != LONGER_ACT_RELU) return api_error(LONGER_ERR_ARG, "act %d unknown", c->act);
  if (c->d <= 0 || c->d % 32 || c->d > 512) return api_error(LONGER_ERR_ARG, "d=%d must be a multiple of 32, at most 512", c->d);
  if (c->ffn_mult <= 0 || c->ffn_mult * c->d > 2048) return api_error(LONGER_ERR_ARG, "ffn_mult=%d: the hidden width must be at most 2048", c->ffn_mult);
  if (de <= 0 || de >= c->d || de % 32) return api_error(LONGER_ERR_ARG, "d_e=%d must be a multiple of 32 below d=%d", de, c->d);
  if (B <= 0 || L <= 0 || (long long)B * L >= (1ll << 31) / 8) return api_error(LONGER_ERR_ARG, "B=%d, L=%d out of range", B, L);
  *d = c->d; *f = c->ffn_mult * c->d;
  return 0;
}

}  // namespace bw
}  // namespace longer

using namespace longer;

extern "C" {

size_t longer_backward_workspace_bytes(const longer_config* cfg, int B, int L) {
  bw::Dims s;
  if (bw::check(cfg, B, L, &s)) return 0;
  return bw::merge_workspace(cfg, s, B, L).total;
}

size_t longer_block_grad_floats(const longer_config* cfg) {
  bw::Dims s;
  if (bw::check(cfg, 1, 1, &s)) return 0;
  return bw::grad_layout(s.d, s.f).total;
}

int longer_token_merge_backward(const longer_config* cfg, const longer_block* inner, const void* H,
                                const int32_t* lens, int B, int L, const float* dM,
                                float* dH_out, float* grads_out,
                                void* ws, size_t ws_bytes, void* stream) {
  bw::Dims s;
  int rc = bw::check(cfg, B, L, &s);
  if (rc) return rc;
  if (!inner || !H || !dM || !dH_out || !grads_out || !ws) return api_error(LONGER_ERR_ARG, "null pointer argument");
  if (!bw::aligned16(H) || !bw::aligned16(dM) || !bw::aligned16(dH_out) || !bw::aligned16(grads_out) || ((uintptr_t)ws & 255))
    return api_error(LONGER_ERR_ARG, "H, dM, dH_out, grads_out must be 16-byte aligned and ws 256-byte aligned");
  for (int l = 0; l < s.layers; ++l) {
    const void* const* p = (const void* const*)&inner[l];
    for (int i = 0; i < 16; ++i)
      if (!p[i] || !bw::aligned16(p[i])) return api_error(LONGER_ERR_ARG, "InnerTrans block %d: parameter %d is NULL or not 16-byte aligned", l, i);
  }
  const size_t need = bw::merge_workspace(cfg, s, B, L).total;
  if (ws_bytes < need) return api_error(LONGER_ERR_WS, "workspace too small: %zu < %zu bytes", ws_bytes, need);
  return bw::run(cfg, inner, H, lens, B, L, dM, dH_out, grads_out, (char*)ws, (hipStream_t)stream, s);
}

size_t longer_model_grad_floats(const longer_config* cfg) {
  bw::Dims mi;
  bw::StackDims s;
  if (bw::check(cfg, 1, 1, &mi) || bw::check_stack(cfg, 1, 1, &s)) return 0;
  return bw::model_grads(mi, s, cfg->q_learn != nullptr).total;
}

size_t longer_forward_backward_workspace_bytes(const longer_config* cfg, int B, int L) {
  bw::Dims mi;
  bw::StackDims s;
  if (bw::check(cfg, B, L, &mi) || bw::check_stack(cfg, B, L, &s)) return 0;
  const size_t fwd = least_workspace_bytes(cfg, B, L);
  if (fwd == 0) return 0;
  return bw::stack_ws(s, fwd).total + bw::merge_workspace(cfg, mi, B, L).total;
}

int longer_forward_backward(const longer_config* cfg, const longer_weights* w, const void* H, const void* G,
                            const int32_t* lens, int B, int L, const float* labels,
                            float* loss_out, float* logits_out, float* dH_out, float* dG_out, float* grads_out,
                            void* ws, size_t ws_bytes, void* stream) {
  bw::Dims mi;
  bw::StackDims s;
  int rc = bw::check(cfg, B, L, &mi);
  if (rc) return rc;
  rc = bw::check_stack(cfg, B, L, &s);
  if (rc) return rc;
  if (!w || !w->inner || !w->cross || (cfg->n_self && !w->self) || !w->head_w || !w->head_b || !H || !G || !labels || !loss_out ||
      !dH_out || !dG_out || !grads_out || !ws)
    return api_error(LONGER_ERR_ARG, "null pointer argument");
  const void* ptrs[] = {H, G, labels, loss_out, dH_out, dG_out, grads_out, w->head_w};
  for (const void* p : ptrs)
    if (!bw::aligned16(p)) return api_error(LONGER_ERR_ARG, "H, G, labels, loss_out, dH_out, dG_out, grads_out, head_w must be 16-byte aligned");
  if ((uintptr_t)ws & 255) return api_error(LONGER_ERR_ARG, "ws must be 256-byte aligned");
  for (int l = 0; l < mi.layers + s.layers; ++l) {
    const longer_block* b = l < mi.layers ? &w->inner[l] : (l == mi.layers ? &w->cross[0] : &w->self[l - mi.layers - 1]);
    const void* const* p = (const void* const*)b;
    for (int i = 0; i < 16; ++i)
      if (!p[i] || !bw::aligned16(p[i])) return api_error(LONGER_ERR_ARG, "block %d: parameter %d is NULL or not 16-byte aligned", l, i);
  }
  const size_t fwd = least_workspace_bytes(cfg, B, L);
  if (fwd == 0) return LONGER_ERR_ARG;
  const size_t stack_bytes = bw::stack_ws(s, fwd).total;
  const size_t need = stack_bytes + bw::merge_workspace(cfg, mi, B, L).total;
  if (ws_bytes < need) return api_error(LONGER_ERR_WS, "workspace too small: %zu < %zu bytes", ws_bytes, need);
  hipStream_t st = (hipStream_t)stream;
  // with several blocks the forward merge writes the later ones' input rows where the merge's backward pass expects them
  const bool keep = mi.tiled && mi.layers > 1;
  float* block_inputs = keep ? (float*)((char*)ws + stack_bytes + bw::merge_workspace(cfg, mi, B, L).xin) : nullptr;
  bw::GradTail tail(st);
  __bf16* block_stream = mi.tiled ? (__bf16*)((char*)ws + stack_bytes + bw::merge_workspace(cfg, mi, B, L).stream) : nullptr;
  rc = bw::run_model(cfg, w, H, G, lens, B, L, labels, loss_out, logits_out, dH_out, dG_out, grads_out, (char*)ws, fwd, st, mi, s, block_inputs,
                     block_stream, tail);
  if (rc) return rc;
  // the merge's gradients: dM was left in the stack's workspace; the InnerTrans blocks come first in grads_out
  const float* dM = (const float*)((char*)ws + bw::stack_ws(s, fwd).dM);
  return bw::run(cfg, w->inner, H, lens, B, L, dM, dH_out, grads_out, (char*)ws + stack_bytes, st, mi, keep, &tail);
}

size_t longer_input_backward_workspace_bytes(const longer_config* cfg, int B, int L, int d_e) {
  int d, f;
  if (bw::check_input_bw(cfg, B, L, d_e, &d, &f)) return 0;
  return bw::input_ws((size_t)B * L, d, f).total;
}

size_t longer_input_grad_floats(const longer_config* cfg, int L, int d_e) {
  int d, f;
  if (bw::check_input_bw(cfg, 1, L, d_e, &d, &f)) return 0;
  return bw::input_grads(L, d, f, d_e).total;
}

int longer_input_generation_backward(const longer_config* cfg, const longer_input_weights* w, const void* E,
                                     const void* tdiff, const int32_t* lens, int B, int L, int d_e, const float* dH,
                                     float* dE_out, float* dtdiff_out, float* grads_out,
                                     void* ws, size_t ws_bytes, void* stream) {
  int d, f;
  int rc = bw::check_input_bw(cfg, B, L, d_e, &d, &f);
  if (rc) return rc;
  if (!w || !w->pos || !w->w1 || !w->b1 || !w->w2 || !w->b2 || !E || !tdiff || !dH || !dE_out || !dtdiff_out || !grads_out || !ws)
    return api_error(LONGER_ERR_ARG, "null pointer argument");
  const void* ptrs[] = {w->pos, w->w1, w->b1, w->w2, w->b2, E, tdiff, dH, dE_out, dtdiff_out, grads_out};
  for (const void* p : ptrs)
    if (!bw::aligned16(p)) return api_error(LONGER_ERR_ARG, "every pointer must be 16-byte aligned");
  if ((uintptr_t)ws & 255) return api_error(LONGER_ERR_ARG, "ws must be 256-byte aligned");
  const size_t nt = (size_t)B * L;
  const bw::InputWs l = bw::input_ws(nt, d, f);
  if (ws_bytes < l.total) return api_error(LONGER_ERR_WS, "workspace too small: %zu < %zu bytes", ws_bytes, l.total);
  const bw::InputGrads gl = bw::input_grads(L, d, f, d_e);
  hipStream_t st = (hipStream_t)stream;
  char* w8 = (char*)ws;
  const bw::RowGeom q = {lens, L, 1, (int)nt};
  const bw::RowsValid rv = {lens, L};
  float* part = (float*)(w8 + l.part);
  bw::ReduceBatch rb;
  if (bw::input_tiled(d)) {
    __bf16* stream_w = (__bf16*)(w8 + l.w1t);
    __bf16* rec = (__bf16*)(w8 + l.rec);
    bw::PackBatch pk(d, stream_w, st);
    pk.add(w->w1, f, 1, false, f / 32, 0, 3);           // hidden values, their gradient, back through W1
    pk.add(w->w2, 1, d, false, f / 32, 1, 3);
    pk.add(w->w1, 1, f, true, f / 32, 2, 3);
    if ((rc = pk.flush())) return rc;
    const bw::InputBwParams p = {(const char*)stream_w, (const __bf16*)E, (const __bf16*)w->pos, (const __bf16*)tdiff, (const __bf16*)w->b1,
                                 lens, B, L, d_e, f, cfg->act, dH, dE_out, dtdiff_out, rec};
    if (d == 128) bw::bw_input_launch_128(p, st); else bw::bw_input_launch_64(p, st);
    if ((rc = bw::launched("input gradient"))) return rc;
    bw::WgradBatch wg = bw::input_wgrads_tiles(d, f, nt, rv, rec, grads_out + gl.w1, grads_out + gl.w2);
    if ((rc = bw::launch(wg, part, st))) return rc;
    rb.add(wg);
    if ((rc = bw::launch(rb, st))) return rc;
  } else {
    __bf16* x = (__bf16*)(w8 + l.x);   __bf16* w1t = (__bf16*)(w8 + l.w1t); __bf16* a = (__bf16*)(w8 + l.a);
    __bf16* dyb = (__bf16*)(w8 + l.dyb); __bf16* dh = (__bf16*)(w8 + l.dh); float* dx = (float*)(w8 + l.dx);
    const unsigned eg = bw::flat_grid(nt * d / 4);
    bw::bw_input_rows_kernel<<<eg, 256, 0, st>>>((const __bf16*)E, (const __bf16*)w->pos, (const __bf16*)tdiff, x, q, d, d_e);
    bw::bw_cast_rows_kernel<<<eg, 256, 0, st>>>(dH, dyb, q, d);
    if ((rc = bw::launched("input rows"))) return rc;
    // the hidden pre-activation is formed again inside the launch that takes its gradient (as in the merge's FFN)
    if ((rc = bw::transpose(st, (const __bf16*)w->w1, w1t, d, f))) return rc;
    if ((rc = bw::gemm_ffn_mid(st, x, dyb, d, w1t, (const __bf16*)w->w2, f, (const __bf16*)w->b1, nt, cfg->act, dh, a, rv))) return rc;
    bw::WgradBatch wg = bw::input_wgrads(d, f, nt, rv, x, dh, a, dyb, grads_out + gl.w1, grads_out + gl.w2);
    if ((rc = bw::launch(wg, part, st))) return rc;
    rb.add(wg);
    if ((rc = bw::launch(rb, st))) return rc;
    if ((rc = bw::gemm_rows_t(st, dh, f, (const __bf16*)w->w1, d, nt, bw::EPI_F32, dx, rv))) return rc;
    bw::bw_split_input_grad_kernel<<<eg, 256, 0, st>>>(dx, dE_out, dtdiff_out, q, d, d_e);
  }
  bw::bw_pos_grad_kernel<<<(unsigned)(((size_t)L * d_e / 4 + 63) / 64), 256, 0, st>>>(dE_out, grads_out + gl.pos, q, B, d_e);
  return bw::launched("input gradient");
}

}  // extern "C"
