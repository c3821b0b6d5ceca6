// One InnerTrans block's recomputation and backward pass in one launch, a tile of 32 tokens per wave.
//
// Everything between the block's input rows and the operands of its parameter gradients stays in the wave's
// registers, in the layout of the forward kernels (device.h: lane = token, registers = features; an accumulator
// tile rounded to bf16 is the next product's operand): LayerNorm, Q / K / V, the attention inside the groups,
// output projection, LayerNorm, the FFN's hidden values and their gradient chunk by chunk, and back through all
// of them.  What reaches memory is what the parameter gradients contract over the whole batch, and q, k, v, which
// wait there for the way back.
//
// What bounds it: as thirteen launches over [token, feature] tensors (two LayerNorms, three products, attention,
// the FFN's middle, three products back, attention back, two LayerNorms back) a block of the headline batch
// (512 000 rows of width 128) moved 18.8 KB per token beside its parameter gradients in 2.1 ms; here it is 8.0 KB (4.1 GB)
// in 0.80 ms (to 0.84 by card): 5 TB/s, what a large copy reaches; the last block 6.7 KB (3.4 GB) in 0.79 (to 0.82), 4.3 TB/s, the groups' sums beside it.  Memory and the vector unit add up: with a third of its stores
// left out it took 0.80 instead of 0.90 ms, and with 9 650 instead of 10 800 vector instructions per tile (beside 808 products) 0.84.  The stream's waits
// waited for the records' stores with it (step of the headline model 4169 -> 4100 us without that), a segment's fragments came out of LDS two at a time
// (four: 4079), and q, k, v, which the tile reads again, passed by the caches (now not: 0.2 % there, 1 % of a step of 128 short users).
//
// Tile blocks.  A tensor of F features that the parameter gradients read is stored as [F / 16][1 KiB] per tile: 16
// features of 32 tokens, 32 bytes per token, as the lanes hold them (lane half hi: features 4 hi .. + 3 and
// 8 + 4 hi .. + 3 of the sixteen), so a store or load of a wave is 1 KiB without gaps and the transposing LDS
// read finds four consecutive features in every 8 bytes.  In odd sixteens the tokens' 128-byte quarters are
// swapped pairwise, so that the two sixteens of a fragment lie in different LDS banks.
// Tiles count slots [B][T K] (a user's groups, the last one filled up), so a group never spans two tiles.
#pragma once
#include "block_kernel.h"
#include "bw_common.h"

namespace longer {
namespace bw {

struct BlockBwParams {
  const char* wstream;                      // packed weights of the block (bw_pack_block_kernel)
  const __bf16 *ln1_g, *ln1_b, *bq, *bv, *bo, *ln2_g, *ln2_b, *b1;
  const int32_t* lens;
  int B, L, K, T, f, act;
  float eps;
  const void* x; int x_f32;                 // the block's input rows: raw tokens [B][L][D] bf16, or [B][T K][D] fp32
  const float* dM; int concat;              // gradient of the block's output: from the merged tokens' gradient,
  const float* dy;                          // or (dM NULL) the fp32 tile blocks the block after this one wrote
  __bf16* rec;                              // tile records (BlockRecord)
  float* dx; int dx_rows;                   // gradient of the input: fp32 tile blocks, or [B][L][D] (zeros for padded tokens)
  __bf16* gx; __bf16* gy;                   // NULL, or where the operands of W2's gradient go group by group (GroupOperands)
};

// The last block's output gradient is the same for all tokens of a group (the merge takes their mean), so W2's gradient contracts over groups: the
// mean of a group's activated hidden values, in two bf16 parts (the value and what its rounding left), times the merged token's gradient.  At K = 8
// these are 288 instead of 1280 bytes a token, written here and read by the gradients: step of the headline model 3725 -> 3610 us (the block 826 -> 788, its
// gradients 388 -> 348), from the raw inputs 1108 -> 1073, of the small model 249 -> 244; W2's gradient comes out 2 to 4 % closer to double precision.  Tile blocks of 32 groups: x [2 t + part][f / 16], y [t][d / 16].
// For K = 8, and 16 at width 128: below, two parts of few tokens save little; at 32 a group is a whole tile; below width 128 a token's W2 operands are a smaller
// share of its record, and at K = 16 the readers' masks cost as much (a step with them / without, 65 536 tokens of width 64: K = 8 241 / 246 us, K = 16 294 / 291; width 32,
// steps of 16 x 200, 128 x 2000 and 400 x 3000 tokens: K = 8 110 / 109, 272 / 273, 853 / 876, K = 16 111 / 110, 250 / 259, 808 / 827: there only large ones gain).  Nor below
// width 128 for users of different length: the readers look for tokens row by row, with a loop that knows groups for the other matrices too, and what either block
// writes finds fewer lines of the other one's records in the last-level cache (width 64, 256 users of at most 512 tokens, two blocks 457 / 444 us, 128 of them, one block 243 / 241,
// 60 of at most 4000 390 / 385; width 32, 500 of at most 1000 358 / 352).
__host__ __device__ constexpr bool group_operands(int d, int K) { return K == 8 || (K == 16 && d >= 128); }
inline bool group_operands(int d, int K, bool ragged) { return group_operands(d, K) && (d >= 128 || !ragged); }
__host__ __device__ inline size_t group_tiles(size_t slots, int K) { return (slots / K + 31) / 32; }

// A tile's record: all of its tile blocks side by side (xh: normalised rows before gain and shift; the gradients of q, k,
// v take the place of q, k, v).  Offsets and size in sixteens of features (1 KiB).
struct BlockRecord {
  int qkv, xh1, o, xh2, dyb, dxmb, a, dh, size;
  // grouped: dyb and a are not there (GroupOperands take their place)
  __host__ __device__ BlockRecord(int d, int f, bool grouped = false)
      : qkv(0), xh1(3 * d / 16), o(4 * d / 16), xh2(5 * d / 16), dyb(6 * d / 16), dxmb(grouped ? dyb : 7 * d / 16), a(dxmb + d / 16),
        dh(grouped ? a : a + f / 16), size(dh + f / 16) {}
};

constexpr int kBlkWaves = 4;
__host__ __device__ inline int bw_block_segs(int d, int f) { return 8 * (d / 32) + 3 * (f / 32); }
constexpr int kBlkPanel = 2;                // segments per panel of the weight stream (4 below width 128)
// segments that are readable: the stream is read in whole panels
__host__ __device__ inline int bw_block_segs_padded(int d, int f) { return (bw_block_segs(d, f) + 3) / 4 * 4; }
// floats of the block's vectors in LDS: ln1 gain and shift, b_Q, b_V, b_O, ln2 gain and shift, b_1
__host__ __device__ inline int bw_block_vec_floats(int d, int f) { return 7 * d + f; }

void bw_block_launch_32(int dh, const BlockBwParams& p, hipStream_t st);
void bw_block_launch_64(int dh, const BlockBwParams& p, hipStream_t st);
void bw_block_launch_128(int dh, const BlockBwParams& p, hipStream_t st);

// the lane's 16 bytes of a sixteen whose index has parity `odd`
__device__ __forceinline__ int tile_lane_offset(int lane, int odd) { return ((lane & 31) ^ (4 * odd)) * 32 + (lane >> 5) * 16; }

// A tile's stretch of memory (wave-uniform base, `bytes` long) as a buffer: offset = the lane's part + a uniform one.  Loads take
// the uniform part from a scalar register, stores do not: a store reads its data for two more cycles after its issue, and the
// compiler keeps the registers for that long unless the store has a scalar offset.  With one, the vector instruction
// right behind a store replaced its data now and then (one 1 KiB piece of a few tiles in a pass of 16 000).  Their uniform part goes into the
// buffer's base instead: as part of the lane's offset each was a vector addition, whose results the compiler kept, and spilled, from one place to another.
struct TileBuffer {
  __amdgpu_buffer_rsrc_t r;
  char* b; int n;
  __device__ __forceinline__ TileBuffer(const void* base, int bytes) : r(__builtin_amdgcn_make_buffer_rsrc((void*)base, 0, bytes, 0x00027000)), b((char*)base), n(bytes) {}
  __device__ __forceinline__ __amdgpu_buffer_rsrc_t at(int off) const { return __builtin_amdgcn_make_buffer_rsrc(b + (off & ~4095), 0, n - (off & ~4095), 0x00027000); }
  __device__ __forceinline__ u32x4 get(unsigned lane_off, int off) const { return __builtin_amdgcn_raw_buffer_load_b128(r, (int)lane_off, off, 0); }
  __device__ __forceinline__ void put(unsigned lane_off, int off, u32x4 v) const { __builtin_amdgcn_raw_buffer_store_b128(v, at(off), (int)lane_off + (off & 4095), 0, 0); }
  __device__ __forceinline__ void put4(unsigned lane_off, int off, uint32_t v) const { __builtin_amdgcn_raw_buffer_store_b32(v, at(off), (int)lane_off + (off & 4095), 0, 2); }
  __device__ __forceinline__ void put2(unsigned lane_off, int off, uint16_t v) const { __builtin_amdgcn_raw_buffer_store_b16(v, at(off), (int)lane_off + (off & 4095), 0, 2); }
  __device__ __forceinline__ void put_once(unsigned lane_off, int off, u32x4 v) const { __builtin_amdgcn_raw_buffer_store_b128(v, at(off), (int)lane_off + (off & 4095), 0, 2); }      // (streaming: `nt`)
};

typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
__device__ __forceinline__ bf16x8 join_tr(s16x4 lo, s16x4 up) {
  typedef short s16x8 __attribute__((ext_vector_type(8)));
  const s16x8 v = __builtin_shufflevector(lo, up, 0, 1, 2, 3, 4, 5, 6, 7);
  return __builtin_bit_cast(bf16x8, v);
}
// byte offset, inside a 2 KiB piece (32 features = two sixteens) of a tile block, that this lane hands to the
// transposing read: 16 lanes cover four tokens from `token` on and sixteen features
__device__ __forceinline__ int tile_tr_offset(int lane, int token) {
  const int i = lane & 15, c = i & 3, fg = (lane >> 4) & 1;
  return fg * 1024 + (((token + (i >> 2)) ^ (4 * fg)) * 32) + (c & 1) * 16 + (c >> 1) * 8;
}

// The W registers of a score tile that a lane's group can occupy, and probabilities back into an operand
// (block_kernel.h, softmax_window, explains the windows).
template <int W>
__device__ __forceinline__ void pick_window(const f32x16& S, int widx, float (&x)[W]) {
  const bool b0 = widx & 1, b1 = widx & 2;
  float sv[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) { float t = S[r]; asm("" : "+v"(t)); sv[r] = t; }
#pragma unroll
  for (int c = 0; c < W; ++c) {
    const float a0 = sv[c], a1 = sv[(16 / W > 2 ? 4 : 8) % 16 + c % 8];      // (values, not elements: no indexed register)
    if (W == 16) x[c] = a0;
    else if (W == 8) x[c] = b0 ? a1 : a0;
    else {
      const float a2 = sv[8 + c % 4], a3 = sv[12 + c % 4];
      const float lo = b0 ? a1 : a0, up = b0 ? a3 : a2;
      x[c] = b1 ? up : lo;
    }
  }
}
template <int W>
__device__ __forceinline__ void place_window(const float (&x)[W], const uint32_t (&wmask)[16 / W], bf16x8 (&op)[2]) {
  uint32_t pk[W / 2];
#pragma unroll
  for (int c = 0; c < W / 2; ++c) {
    const longer::bf16x2 t2 = {(__bf16)x[2 * c], (__bf16)x[2 * c + 1]};
    pk[c] = __builtin_bit_cast(uint32_t, t2);
  }
#pragma unroll
  for (int g = 0; g < 2; ++g) {
    u32x4 v;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int ps = 4 * g + i;
      v[i] = W == 16 ? pk[ps % (W / 2)] : pk[ps % (W / 2)] & wmask[ps / (W / 2)];
    }
    op[g] = __builtin_bit_cast(bf16x8, v);
  }
}

// Probabilities and score gradients go into their products as two bf16 operands, the value and what its rounding left
// (16 significant bits between them): the second pair of products costs less than the rounding did in accuracy.
template <int W>
__device__ __forceinline__ void place_split(const float (&x)[W], const uint32_t (&wmask)[16 / W], bf16x8 (&op)[2], bf16x8 (&rest)[2]) {
  float lo[W];
#pragma unroll
  for (int c = 0; c < W; ++c) lo[c] = x[c] - (float)(__bf16)x[c];
  place_window<W>(x, wmask, op);
  place_window<W>(lo, wmask, rest);
}

// CENTRE: the mean is taken from the rows as well
template <int NT, bool CENTRE = false>
__device__ __forceinline__ void row_stats(f32x16 (&x)[NT], float eps, float& mean, float& rstd) {
  float s = 0.f, v = 0.f;
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) s += x[t][r];
  mean = sum_halves(s) * (1.f / (32 * NT));
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) { const float q = x[t][r] - mean; v = fmaf(q, q, v); if (CENTRE) x[t][r] = q; }
  rstd = 1.f / sqrtf(sum_halves(v) * (1.f / (32 * NT)) + eps);
}

// dx = res + LayerNorm backward of dn at the rows x; result in x.  (Normalised rows are formed by subtraction, here and on the way forward: in
// x rstd - mean rstd, one instruction, the second product is rounded ahead of the difference, and rows whose mean is large
// against their deviation lose digits: rows of equal features 1000 came out as up to 0.016 instead of 0.)
template <int NT>
__device__ __forceinline__ void norm_backward(f32x16 (&x)[NT], f32x16 (&dn)[NT], const float* gain, float mean, float rstd, int hi) {
  float c1 = 0.f, c2 = 0.f;
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    dn[t] *= bias_tile(gain, t, hi);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      x[t][r] = (x[t][r] - mean) * rstd;
      c1 += dn[t][r];
      c2 = fmaf(dn[t][r], x[t][r], c2);
    }
  }
  c1 = sum_halves(c1) * (1.f / (32 * NT));
  c2 = sum_halves(c2) * (1.f / (32 * NT));
  c1 *= -rstd; c2 *= -rstd;
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) x[t][r] = fmaf(x[t][r], c2, fmaf(dn[t][r], rstd, c1));      // rstd (dn - mean(dn) - x mean(dn x))
}

// use(s, fragment s) for the stream's current segment, four fragments on their way out of LDS (the compiler keeps two, and each pair of
// products waited out the latency)
template <int NG, typename WS, typename F>
__device__ __forceinline__ void segment_fragments(const WS& ws, const F& use) {
  constexpr int AH = NG < 4 ? NG : 4;
  bf16x8 fr[AH];
#pragma unroll
  for (int s = 0; s < AH; ++s) fr[s] = ws.template frag<bf16x8>(s);
#pragma unroll
  for (int s = 0; s < NG; ++s) {
    __builtin_amdgcn_sched_barrier(0x6);
    use(s, fr[s % AH]);
    if (s + AH < NG) fr[s % AH] = ws.template frag<bf16x8>(s + AH);
  }
  __builtin_amdgcn_sched_barrier(0x6);
}

// W: registers of a score tile that one group can occupy (K <= 2 W)
// GROUPED: W2's operands are kept group by group
template <int D, int DH, int W, bool GROUPED>
__global__ __launch_bounds__(64 * kBlkWaves, 2) void bw_block_kernel(const BlockBwParams p) {
  constexpr int NT = D / 32, NG = D / 16, SEGV = NG * 64, HPT = 32 / DH, GPH = DH / 16;
  constexpr int PSEG = D >= 128 ? kBlkPanel : 4, NB = 3;
  using E = ET<__bf16>;
  __shared__ uint4 ring[NB * PSEG * SEGV];
  __shared__ uint4 turn[kBlkWaves][3][128];        // a wave's K, Q and dO (V on the way forward) pieces of 32 features
  __shared__ f32x4 stat[kBlkWaves][2][8];          // its queries' log-sum-exp and sum of P dP
  __shared__ uint8_t lefts[kBlkWaves][32];         // valid tokens of its tokens' groups
  __shared__ float2 norm1[kBlkWaves][32];          // its tokens' first LayerNorm: mean, 1 / standard deviation
  extern __shared__ f32x4 vec4[];
  float* vec = (float*)vec4;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), j = lane & 31, hi = lane >> 5;
  const int NC = p.f / 32;
  const BlockRecord rc(D, p.f, GROUPED);

  // ---- the lane's token
  const int tile = blockIdx.x * kBlkWaves + wave;
  char* rec = (char*)p.rec + (size_t)tile * rc.size * 1024;       // (wave-uniform: a scalar base, the lane's part an offset)
  const unsigned lane0 = tile_lane_offset(lane, 0), lane1 = tile_lane_offset(lane, 1);
  // records and tile blocks are addressed as buffers: with 64-bit addresses every access cost the vector unit two or three instructions
  const TileBuffer recb(rec, rc.size * 1024);
  auto put_rec = [&](int base, int g, bf16x8 v) { recb.put_once(g & 1 ? lane1 : lane0, (base + g) * 1024, __builtin_bit_cast(u32x4, v)); };      // (base is even)
  // (q, k and v are read again by this tile; everything else by a later launch only)
  auto keep_rec = [&](int base, int g, bf16x8 v) { recb.put(g & 1 ? lane1 : lane0, (base + g) * 1024, __builtin_bit_cast(u32x4, v)); };
  auto get_rec = [&](int base, int g) -> bf16x8 { return __builtin_bit_cast(bf16x8, recb.get(g & 1 ? lane1 : lane0, (base + g) * 1024)); };
  struct Token { uint32_t slot; int u, tg, jj; bool stored; long long row; };
  auto locate = [&](uint32_t first) {
    Token k;
    k.slot = first + (uint32_t)j;
    const uint32_t gidx = k.slot >> __builtin_ctz(p.K);
    k.jj = (int)(k.slot & (uint32_t)(p.K - 1));
    k.u = (int)(gidx / (uint32_t)p.T); k.tg = (int)(gidx - (uint32_t)k.u * (uint32_t)p.T);
    const int pos = k.tg * p.K + k.jj;
    k.stored = k.u < p.B && pos < p.L;             // the token has a row in the [B][L] tensors
    k.row = (long long)k.u * p.L + pos;
    return k;
  };
  const Token tk = locate((uint32_t)tile * 32u);
  int left = 0;                                    // valid tokens of the lane's group
  if (tk.u < p.B) {
    int len = p.lens ? p.lens[tk.u] : p.L;
    left = min(max(min(max(len, 0), p.L) - tk.tg * p.K, 0), p.K);
  }
  if (hi == 0) lefts[wave][j] = (uint8_t)left;
  const bool valid = tk.jj < left;
  if (!__syncthreads_or(valid ? 1 : 0)) {
    if (p.dx_rows && tk.stored) {
      const f32x4 z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q) *(f32x4*)(p.dx + tk.row * D + 32 * t + 8 * q + 4 * hi) = z;
    }
    return;
  }
  const int widx = W == 16 ? 0 : j / (2 * W);
  constexpr int KG = 2 * W;                        // tokens of a group where its operands are kept group by group
  const int gfirst = tile * (32 / KG);             // and the tile's first group
  uint32_t wmask[16 / W];
#pragma unroll
  for (int w = 0; w < 16 / W; ++w) { wmask[w] = widx == w ? 0xffffffffu : 0u; asm("" : "+v"(wmask[w])); }
  uint32_t vb = (uint32_t)__ballot(valid);
  const uint32_t gb = (p.K >= 32 ? 0xffffffffu : ((1u << p.K) - 1u)) << (p.K * (j / p.K));
  uint32_t seen = ((gb & vb) >> (4 * hi)) >> (2 * W * widx);     // window bits: the group's valid tokens

  // ---- vectors to LDS, weight stream
  const int oG1 = 0, oB1n = D, oBq = 2 * D, oBv = 3 * D, oBo = 4 * D, oG2 = 5 * D, oB2n = 6 * D, oBf = 7 * D;
  // Everything that is read before the first product is requested at once (a trip to memory takes several thousand
  // cycles under this kernel's stores): rows, vectors into registers, the stream's first panels.
  f32x16 x[NT];
  load_rows<__bf16, NT>(x, p.x, p.x_f32, (p.x_f32 ? (long long)tk.slot : tk.row) * D, valid, hi);
  constexpr int VB = 2048 / (64 * kBlkWaves);
  __bf16 vd[7], vf[VB];
  {
    const int i = tid < D ? tid : 0;
    vd[0] = p.ln1_g[i]; vd[1] = p.ln1_b[i]; vd[2] = p.bq[i]; vd[3] = p.bv[i]; vd[4] = p.bo[i]; vd[5] = p.ln2_g[i]; vd[6] = p.ln2_b[i];
#pragma unroll
    for (int k = 0; k < VB; ++k) {
      const int c = tid + 64 * kBlkWaves * k;
      vf[k] = p.b1[c < p.f ? c : 0];
    }
  }
  WStream<SEGV, PSEG, NB, false, 64 * kBlkWaves> ws;
  ws.init(ring, p.wstream, bw_block_segs(D, p.f));
  if (tid < D) {
#pragma unroll
    for (int k = 0; k < 7; ++k) vec[k * D + tid] = (float)vd[k];
  }
#pragma unroll
  for (int k = 0; k < VB; ++k) {
    const int c = tid + 64 * kBlkWaves * k;
    if (c < p.f) vec[oBf + c] = (float)vf[k];
  }
  __syncthreads();
  // The stream's waits leave the records' stores alone: of those issued since the panel due was requested, two panels ago, at least
  // these many may still be on their way (in the order of the stream: Q, K, V of a feature tile with two stores behind each and two
  // of o; the output projection, the last of which has four stores in two panels of two segments; a hidden chunk's four; two in front of
  // each product that takes dq, dk, dv back).  Waiting for them as well, a chunk could not end before its stores had.
  typedef std::integral_constant<int, 8> Attn;
  typedef std::integral_constant<int, PSEG == 2 ? 4 : D == 64 ? 8 : 0> Hidden;
  typedef std::integral_constant<int, 6> Back;
  auto fragments = [&](auto&& use) { segment_fragments<NG>(ws, use); };
  auto product = [&](f32x16& acc, const bf16x8 (&b)[NG], auto younger) {      // acc += (this segment's 32 output features) b
    fragments([&](int s, const bf16x8 w) { acc = E::mma(w, b[s], acc); });
    ws.template advance<D >= 64 ? decltype(younger)::value : 0>();
    settle(acc);
  };
  auto spread = [&](f32x16 (&acc)[NT], const bf16x8 (&b)[2], auto younger) {  // acc += (all output features of 32 contracted ones) b
    fragments([&](int s, const bf16x8 w) { acc[s / 2] = E::mma(w, b[s & 1], acc[s / 2]); });
    ws.template advance<D >= 64 ? decltype(younger)::value : 0>();
  };
  // pieces of 32 features through LDS: in as the lanes hold them, out with lane = feature (tokens 16 g ..)
  const int put = j * 32 + hi * 16, put1 = 1024 + (j ^ 4) * 32 + hi * 16, get = tile_tr_offset(lane, 4 * hi);
  auto turn_in = [&](int which, const bf16x8 (&v)[2]) {
    char* s = (char*)turn[wave][which];
    *(bf16x8*)(s + put) = v[0];
    *(bf16x8*)(s + put1) = v[1];
  };
  auto turn_out = [&](int which, int g) -> bf16x8 {
    const char* s = (const char*)turn[wave][which] + get + 16 * g * 32;
    return join_tr(__builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)s),
                   __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(s + 8 * 32)));
  };

  // ---- first LayerNorm
  float mean1, rstd1;
  row_stats<NT>(x, p.eps, mean1, rstd1);
  if (hi == 0) norm1[wave][j] = make_float2(mean1, rstd1);
  bf16x8 nop[NG];
  auto normalise = [&](float mean, float rstd, int og, int ob, int dump) {
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const f32x16 g = bias_tile(vec + og, t, hi), b = bias_tile(vec + ob, t, hi);
      f32x16 h, y;
#pragma unroll
      for (int r = 0; r < 16; ++r) { h[r] = (x[t][r] - mean) * rstd; y[r] = fmaf(h[r], g[r], b[r]); }
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        put_rec(dump, 2 * t + q, E::pack(h, q));
        nop[2 * t + q] = E::pack(y, q);
      }
    }
  };
  normalise(mean1, rstd1, oG1, oB1n, rc.xh1);

  // ---- attention inside the groups.  Q carries log2(e) / sqrt(head width): scores come out ready for exp2.  The
  // key bias adds a constant to a query's scores and is left out.
  const float scale = 1.f / sqrtf((float)DH), qscale = scale * 1.44269504088896341f;
  auto probabilities = [&](const f32x16& S, float (&x_)[W], float& m, float& l) {   // lane = query; unnormalised
    pick_window<W>(S, widx, x_);
    m = kNegBig;
#pragma unroll
    for (int c = 0; c < W; ++c) {
      x_[c] = ((seen >> (8 * (c / 4) + (c % 4))) & 1u) ? x_[c] : -__builtin_inff();
      m = fmaxf(m, x_[c]);
    }
    m = max_halves(m);
    l = 0.f;
#pragma unroll
    for (int c = 0; c < W; ++c) { x_[c] = __builtin_amdgcn_exp2f(x_[c] - m); l += x_[c]; }
    l = sum_halves(l);
  };
  // Gradient of the block's output: requested all at once, a product or more ahead of its use (a request waits for every store
  // in front of it).  The tile blocks of the block after this one and the merged tokens' gradient both go on in equal steps.
  f32x4 up[4 * NT];
  auto request_upstream = [&](const Token& k, bool there) {
    if (!p.dM) {
      const TileBuffer b(p.dy + (size_t)tile * (32 * D), 128 * D);
#pragma unroll
      for (int i = 0; i < 4 * NT; ++i) up[i] = __builtin_bit_cast(f32x4, b.get(16u * (unsigned)lane, 1024 * i));
    } else {                                           // (a padded token reads the first merged token's and drops it)
      typedef __attribute__((address_space(1))) const f32x4 gcf32x4;
      const float* base = p.dM + (there ? ((size_t)k.u * p.T + k.tg) * (size_t)(p.concat ? p.K * D : D) + (p.concat ? k.jj * D : 0) : 0) + 4 * hi;
#pragma unroll
      for (int i = 0; i < 4 * NT; ++i) up[i] = *(gcf32x4*)(base + 8 * i);
    }
  };
  auto take_upstream = [&](int n, bool there) {
    if (p.dM) {
      const float share = !there ? 0.f : p.concat ? 1.f : 1.f / (float)n;
#pragma unroll
      for (int i = 0; i < 4 * NT; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) { const float one = up[i][e]; up[i][e] = there ? one * share : 0.f; }
    }
  };
  auto upstream = [&](int t) -> f32x16 {
    f32x16 v;
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e) { const float one = up[4 * t + q][e]; v[4 * q + e] = one; }
    return v;
  };
  bf16x8 dyop[NG];
  {
    bf16x8 oop[NG];
#pragma unroll
    for (int ft = 0; ft < NT; ++ft) {
      bf16x8 qop[2], kop[2];
      {
        f32x16 q = bias_tile(vec + oBq, ft, hi);
        product(q, nop, Attn{});
        q *= qscale;
#pragma unroll
        for (int g = 0; g < 2; ++g) { qop[g] = E::pack(q, g); keep_rec(rc.qkv, 2 * ft + g, qop[g]); }
      }
      {
        f32x16 k = splat16(0.f);
        product(k, nop, Attn{});
#pragma unroll
        for (int g = 0; g < 2; ++g) { kop[g] = E::pack(k, g); keep_rec(rc.qkv, NG + 2 * ft + g, kop[g]); }
      }
      {
        f32x16 v = bias_tile(vec + oBv, ft, hi);
        product(v, nop, Attn{});
        bf16x8 vop[2];
#pragma unroll
        for (int g = 0; g < 2; ++g) { vop[g] = E::pack(v, g); keep_rec(rc.qkv, 2 * NG + 2 * ft + g, vop[g]); }
        turn_in(2, vop);
      }
      __builtin_amdgcn_wave_barrier();
      f32x16 o;
#pragma unroll
      for (int hh = 0; hh < HPT; ++hh) {
        f32x16 S = splat16(0.f);
#pragma unroll
        for (int g = 0; g < GPH; ++g) S = E::mma(kop[hh * GPH + g], qop[hh * GPH + g], S);
        float pr[W], m, l;
        probabilities(S, pr, m, l);
        const float inv = l > 0.f ? 1.f / l : 0.f;
        bf16x8 pop[2], plo[2];
        place_split<W>(pr, wmask, pop, plo);
        f32x16 acc = splat16(0.f);
#pragma unroll
        for (int g = 0; g < 2; ++g) {
          const bf16x8 vt = turn_out(2, g);
          acc = E::mma(vt, plo[g], acc);
          acc = E::mma(vt, pop[g], acc);
        }
#pragma unroll
        for (int r = 0; r < 16 / HPT; ++r) o[16 / HPT * hh + r] = acc[16 / HPT * hh + r] * inv;
      }
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int g = 0; g < 2; ++g) { oop[2 * ft + g] = E::pack(o, g); put_rec(rc.o, 2 * ft + g, oop[2 * ft + g]); }
    }
    // output projection + residual, second LayerNorm
    request_upstream(tk, valid);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      x[t] += bias_tile(vec + oBo, t, hi);
      if (t + 1 < NT) product(x[t], oop, Attn{}); else product(x[t], oop, Hidden{});
    }
    if constexpr (GROUPED) {   // the merged token's gradient, from the lanes of its group's first token (of an empty group: any, the reader drops it)
      const TileBuffer yb(p.gy + (size_t)(gfirst / 32) * (NG * 512), NG * 1024);
      const int q = gfirst % 32 + j / KG;
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const f32x16 v = upstream(t);
#pragma unroll
        for (int g = 0; g < 2; ++g) {
          const bf16x8 b = E::pack(v, g);
          if (j % KG == 0) yb.put_once((q ^ (4 * g)) * 32 + hi * 16, (2 * t + g) * 1024, __builtin_bit_cast(u32x4, b));
        }
      }
      if (hi == 0) ((float*)stat[wave][0])[j] = left > 0 ? 1.f / (float)left : 0.f;
    }
    take_upstream(left, valid);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const f32x16 v = upstream(t);
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        dyop[2 * t + g] = E::pack(v, g);
        if (!GROUPED) put_rec(rc.dyb, 2 * t + g, dyop[2 * t + g]);
      }
    }
  }
  float mean2, rstd2;
  row_stats<NT, true>(x, p.eps, mean2, rstd2);       // (the rows themselves are not needed any more)
  normalise(0.f, rstd2, oG2, oB2n, rc.xh2);

  f32x16 dn[NT];
  {
    // (at width 128 the LDS pieces of the attention, idle here, hold six of the operand's eight groups)
    constexpr int PARK = NG == 8 ? 6 : 0;
    char* park = (char*)turn[wave] + lane * 16;
#pragma unroll
    for (int t = 0; t < NT; ++t) dn[t] = splat16(0.f);
#pragma unroll
    for (int g = 0; g < PARK; ++g) *(bf16x8*)(park + g * 1024) = dyop[g];
    // (K = 8: the lane ends with registers 8 b2 + 4 b0 + 2 b1, + 1 of its group's mean, one 4-byte piece of a row; K = 16: with 8 b3 + 4 b2 + 2 b0 + b1,
    // two bytes, where b0 .. b3 are the bits of its token)
    const int b0 = j & 1, b1 = (j >> 1) & 1, b2 = (j >> 2) & 1, b3 = (j >> 3) & 1;
    const int gg = KG == 8 ? b2 : b3, ge = KG == 8 ? 4 * b0 + 2 * b1 : 4 * b2 + 2 * b0 + b1;
    const unsigned goff = gg * 1024 + (((gfirst % 32 + j / KG) ^ (4 * gg)) * 32) + hi * 16 + 2 * ge;
    const TileBuffer xb(p.gx + (size_t)(gfirst / 32) * (2 * p.f * 32), 2 * p.f * 64);
    const bool some_padding = (uint32_t)__ballot(valid) != 0xffffffffu;
    auto put_group = [&](int c, f32x16& v) {
      if (some_padding) {
#pragma unroll
        for (int r = 0; r < 16; ++r) v[r] = valid ? v[r] : 0.f;
      }
      const float share = ((const float*)stat[wave][0])[j];
      // sums over a group's lanes, halving the registers a lane is left with at each step
      float a[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) a[r] = v[r];
      auto both = [](float x, auto ctrl) {
        return x + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), decltype(ctrl)::value, 0xF, 0xF, true));
      };
      auto step = [&](auto n, auto ctrl, int bit) {
        constexpr int N = decltype(n)::value;
#pragma unroll
        for (int i = 0; i < N; ++i) a[i] = both(a[i], ctrl);
#pragma unroll
        for (int i = 0; i < N / 2; ++i) a[i] = bit ? a[i + N / 2] : a[i];
      };
      using std::integral_constant;
      typedef integral_constant<int, 0x140> Mirror16; typedef integral_constant<int, 0x141> Mirror8;
      typedef integral_constant<int, 0xB1> Swap1; typedef integral_constant<int, 0x4E> Swap2;
      if constexpr (KG == 8) {
        step(integral_constant<int, 16>{}, Mirror8{}, b2); step(integral_constant<int, 8>{}, Swap1{}, b0); step(integral_constant<int, 4>{}, Swap2{}, b1);
      } else {
        step(integral_constant<int, 16>{}, Mirror16{}, b3); step(integral_constant<int, 8>{}, Mirror8{}, b2);
        step(integral_constant<int, 4>{}, Swap1{}, b0); step(integral_constant<int, 2>{}, Swap2{}, b1);
      }
      const float m0 = a[0] * share, m1 = a[1] * share;
      // what the rounding to u left, below 2^119; where u is infinite (a NaN, or an infinity, is left) a finite number, which the infinity outweighs
      auto rest = [](float m, __bf16 u) { return fmaxf(m - (float)u, -0x1p120f); };
      if constexpr (KG == 8) {
        const longer::bf16x2 up2 = {(__bf16)m0, (__bf16)m1}, lo2 = {(__bf16)rest(m0, up2[0]), (__bf16)rest(m1, up2[1])};
        xb.put4(goff, c * 2048, __builtin_bit_cast(uint32_t, up2));
        xb.put4(goff, c * 2048 + p.f * 64, __builtin_bit_cast(uint32_t, lo2));
      } else {
        const __bf16 up1 = (__bf16)m0;
        xb.put2(goff, c * 2048, __builtin_bit_cast(uint16_t, up1));
        xb.put2(goff, c * 2048 + p.f * 64, __builtin_bit_cast(uint16_t, (__bf16)rest(m0, up1)));
      }
    };
    // FFN, 32 hidden features at a time: values and gradient formed, used and written out
    for (int c = 0; c < NC; ++c) {
      f32x16 v = bias_tile(vec + oBf, c, hi), g = splat16(0.f);
      product(v, nop, Hidden{});
      fragments([&](int s, const bf16x8 w) { g = E::mma(w, s < PARK ? *(const bf16x8*)(park + s * 1024) : dyop[s], g); });
      ws.template advance<Hidden::value>();
      settle(g);
      if (p.act == LONGER_ACT_RELU) {
#pragma unroll
        for (int r = 0; r < 16; ++r) { float a_, d_; act_both(v[r], LONGER_ACT_RELU, &a_, &d_, g[r]); v[r] = a_; g[r] = d_; }
      } else {
#pragma unroll
        for (int r = 0; r < 16; ++r) { float a_, d_; act_both(v[r], LONGER_ACT_GELU_ERF, &a_, &d_, g[r]); v[r] = a_; g[r] = d_; }
      }
      bf16x8 hop[2];
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        hop[q] = E::pack(g, q);
        put_rec(rc.dh, 2 * c + q, hop[q]);
        if (!GROUPED) put_rec(rc.a, 2 * c + q, E::pack(v, q));
      }
      if constexpr (GROUPED) put_group(c, v);
      spread(dn, hop, Hidden{});
    }
  }
#pragma unroll
  for (int t = 0; t < NT; ++t) settle(dn[t]);
  // (where the lane's token sits is worked out again, so that nothing of it is kept through the FFN)
  uint32_t again = (uint32_t)tile * 32u;
  asm volatile("" : "+s"(again));
  const Token tk2 = locate(again);
  const int left2 = lefts[wave][j];
  const bool valid2 = tk2.jj < left2;
  request_upstream(tk2, valid2);
  norm_backward<NT>(x, dn, vec + oG2, 0.f, rstd2, hi);
  vb = (uint32_t)__ballot(valid2);
  seen = ((gb & vb) >> (4 * hi)) >> (2 * W * widx);
  take_upstream(left2, valid2);
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    x[t] += upstream(t);                          // gradient of the rows between attention and FFN
#pragma unroll
    for (int g = 0; g < 2; ++g) { nop[2 * t + g] = E::pack(x[t], g); put_rec(rc.dxmb, 2 * t + g, nop[2 * t + g]); }
    dn[t] = splat16(0.f);
  }

  // ---- back through the attention, 32 features (one or two heads) at a time
  const uint32_t keyseen = valid2 ? seen : 0u;
#pragma unroll
  for (int ft = 0; ft < NT; ++ft) {
    bf16x8 qop[2], kop[2], vop[2], dop[2];
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      qop[g] = get_rec(rc.qkv, 2 * ft + g);
      kop[g] = get_rec(rc.qkv, NG + 2 * ft + g);
      vop[g] = get_rec(rc.qkv, 2 * NG + 2 * ft + g);
    }
    {
      f32x16 d = splat16(0.f);
      product(d, nop, Back{});
#pragma unroll
      for (int g = 0; g < 2; ++g) dop[g] = E::pack(d, g);
    }
    turn_in(0, kop);
    turn_in(1, qop);
    turn_in(2, dop);
    __builtin_amdgcn_wave_barrier();
    f32x16 dq, dk, dv;
#pragma unroll
    for (int hh = 0; hh < HPT; ++hh) {
      constexpr int RH = 16 / HPT;
      {   // lane = query: probabilities, dP, D = sum P dP, dS = P (dP - D); dq^T = K^T dS^T
        f32x16 S = splat16(0.f), dP = splat16(0.f);
#pragma unroll
        for (int g = 0; g < GPH; ++g) {
          S = E::mma(kop[hh * GPH + g], qop[hh * GPH + g], S);
          dP = E::mma(vop[hh * GPH + g], dop[hh * GPH + g], dP);
        }
        float pr[W], dp[W], m, l;
        probabilities(S, pr, m, l);
        pick_window<W>(dP, widx, dp);
        const float inv = l > 0.f ? 1.f / l : 0.f;
        float dsum = 0.f;
#pragma unroll
        for (int c = 0; c < W; ++c) { pr[c] *= inv; dsum = fmaf(pr[c], dp[c], dsum); }
        dsum = sum_halves(dsum);
        if (hi == 0) {
          ((float*)stat[wave][0])[j] = m + __builtin_amdgcn_logf(l);
          ((float*)stat[wave][1])[j] = dsum;
        }
#pragma unroll
        for (int c = 0; c < W; ++c) pr[c] *= dp[c] - dsum;
        bf16x8 sop[2], slo[2];
        place_split<W>(pr, wmask, sop, slo);
        f32x16 acc = splat16(0.f);
#pragma unroll
        for (int g = 0; g < 2; ++g) {
          const bf16x8 kt = turn_out(0, g);
          acc = E::mma(kt, slo[g], acc);
          acc = E::mma(kt, sop[g], acc);
        }
#pragma unroll
        for (int r = 0; r < RH; ++r) dq[RH * hh + r] = acc[RH * hh + r] * scale;
      }
      __builtin_amdgcn_wave_barrier();
      {   // lane = key: the same with queries in the registers; dv^T = dO^T P, dk^T = Q^T dS
        f32x16 S = splat16(0.f), dP = splat16(0.f);
#pragma unroll
        for (int g = 0; g < GPH; ++g) {
          S = E::mma(qop[hh * GPH + g], kop[hh * GPH + g], S);
          dP = E::mma(dop[hh * GPH + g], vop[hh * GPH + g], dP);
        }
        float pr[W], dp[W];
        pick_window<W>(S, widx, pr);
        pick_window<W>(dP, widx, dp);
#pragma unroll
        for (int q = 0; q < W / 4; ++q) {
          const f32x4 lse = stat[wave][0][(W / 2) * widx + 2 * q + hi], ds = stat[wave][1][(W / 2) * widx + 2 * q + hi];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int c = 4 * q + e;
            const float s = ((keyseen >> (8 * q + e)) & 1u) ? pr[c] - lse[e] : -__builtin_inff();
            pr[c] = __builtin_amdgcn_exp2f(s);
            dp[c] = pr[c] * (dp[c] - ds[e]);
          }
        }
        f32x16 accv = splat16(0.f), acck = splat16(0.f);
        {
          bf16x8 pop[2], plo[2];
          place_split<W>(pr, wmask, pop, plo);
#pragma unroll
          for (int g = 0; g < 2; ++g) {
            const bf16x8 dt = turn_out(2, g);
            accv = E::mma(dt, plo[g], accv);
            accv = E::mma(dt, pop[g], accv);
          }
        }
        {
          bf16x8 sop[2], slo[2];
          place_split<W>(dp, wmask, sop, slo);
#pragma unroll
          for (int g = 0; g < 2; ++g) {
            const bf16x8 qt = turn_out(1, g);
            acck = E::mma(qt, slo[g], acck);
            acck = E::mma(qt, sop[g], acck);
          }
        }
#pragma unroll
        for (int r = 0; r < RH; ++r) {
          dv[RH * hh + r] = accv[RH * hh + r];
          dk[RH * hh + r] = acck[RH * hh + r] * 0.69314718055994531f;       // (Q carries scale log2 e)
        }
      }
      __builtin_amdgcn_wave_barrier();
    }
#pragma unroll
    for (int m = 0; m < 3; ++m) {
      bf16x8 op[2];
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        op[g] = E::pack(m == 0 ? dq : m == 1 ? dk : dv, g);
        put_rec(rc.qkv, m * NG + 2 * ft + g, op[g]);
      }
      spread(dn, op, Back{});
    }
  }

  // ---- first LayerNorm's backward: x holds the gradient that reaches the input through the residual connection
  f32x16 xin[NT];
  asm volatile("" : "+s"(again));
  const Token tk3 = locate(again);
  const bool valid3 = tk3.jj < lefts[wave][j];
  load_rows<__bf16, NT>(xin, p.x, p.x_f32, (p.x_f32 ? (long long)tk3.slot : tk3.row) * D, valid3, hi);
  { const float2 st = norm1[wave][j]; mean1 = st.x; rstd1 = st.y; }
  const TileBuffer dxb(p.dx + (p.dx_rows ? 0 : (size_t)tile * (32 * D)), p.dx_rows ? 0 : 128 * D);
#pragma unroll
  for (int t = 0; t < NT; ++t) settle(dn[t]);
  norm_backward<NT>(xin, dn, vec + oG1, mean1, rstd1, hi);
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    x[t] += xin[t];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      f32x4 v;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = valid3 ? x[t][4 * q + e] : 0.f;
      if (!p.dx_rows) dxb.put(16u * (unsigned)lane, 1024 * (4 * t + q), __builtin_bit_cast(u32x4, v));
      else if (tk3.stored) *(f32x4*)(p.dx + tk3.row * D + 32 * t + 8 * q + 4 * hi) = v;
    }
  }
}

template <int D>
inline void bw_block_launch_d(int dh, const BlockBwParams& p, hipStream_t st) {
  const size_t tiles = ((size_t)p.B * p.T * p.K + 31) / 32;
  const unsigned grid = (unsigned)((tiles + kBlkWaves - 1) / kBlkWaves);
  const size_t lds = (size_t)bw_block_vec_floats(D, p.f) * 4;
#define LONGER_BW_BLOCK(DH, W)                                                                                    \
  do {                                                                                                            \
    if constexpr (group_operands(D, 2 * W)) { if (p.gx) { bw_block_kernel<D, DH, W, true><<<grid, 64 * kBlkWaves, lds, st>>>(p); break; } } \
    bw_block_kernel<D, DH, W, false><<<grid, 64 * kBlkWaves, lds, st>>>(p);                                       \
  } while (0)
  if (dh == 16) { if (p.K <= 8) LONGER_BW_BLOCK(16, 4); else if (p.K == 16) LONGER_BW_BLOCK(16, 8); else LONGER_BW_BLOCK(16, 16); }
  else { if (p.K <= 8) LONGER_BW_BLOCK(32, 4); else if (p.K == 16) LONGER_BW_BLOCK(32, 8); else LONGER_BW_BLOCK(32, 16); }
#undef LONGER_BW_BLOCK
}

}  // namespace bw
}  // namespace longer
