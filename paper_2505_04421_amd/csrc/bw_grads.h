// Parameter gradients of the backward pass: dW = x^T dy for every matrix of a launch at once, and the
// sums of the partial results.
//
// A parameter gradient is a contraction over the token rows, so its parallelism comes from cutting the
// rows into slices.  One launch takes all matrices (of all layers) whose operands are ready: the reduced
// stack's gradients, 24-48 tiles of 128 x 128 with 100-1000 row steps each, were 24 launches of 12-16 us and
// as many reductions before (512 us of a 1091 us step of the small model: B = 128, L = 512, d = 64), each too
// small for the chip; see the figures at bw_wgrad_kernel.
#pragma once
#include "bw_block.h"

namespace longer {
namespace bw {

// One matrix (or one per layer): dW [m][n] = X^T Y over `rows` token rows, and db [n] = column sums of Y.
struct WgradJob {
  RowsValid rv;                       // padded rows read as zeros; row steps that hold nothing else are passed over
  const __bf16* X; const __bf16* Y;   // [rows][..], pitches ldx, ldy
  long long xstride, ystride;         // elements from one layer's operand to the next layer's
  float* part;                        // partial results: [layer][slice][m n + n]
  int ldx, ldy, m, n, rows;
  int tiles_m, tiles_n, layers;
  int nsub;                           // slices of this job per slice of the launch (a job with more rows than the others)
  int first;                          // its first tile inside a slice's tiles
  int groups, unit;                   // 0, or the operands are of that many groups of `unit` tokens (bw_block.h, GroupOperands): X's tile 2 t + part goes with Y's tile t,
                                      // rows without a token, which nobody wrote, count as zeros, and db, twice what it should be, is halved
};
constexpr int kMaxWgradJobs = 12;
struct WgradArgs { WgradJob job[kMaxWgradJobs]; int njobs, tiles, nslices; };

// TB: output tile TB x TB, four waves in 2 x 2.  Both operands are stored with the contraction (token) index
// strided: a step's 32 rows go to LDS as they are, and the fragments (lane = column, eight tokens per lane)
// come back through the transposing LDS read, two per fragment.  The six launches that this one replaces, with
// eight 2-byte LDS reads per fragment, took 595 us for a block of the headline batch (512 000 rows, width 128), this
// one 392 us (5.3 TB/s of the 4.1 KB per row below); at 4608 rows of width 64 and three layers (the small model's
// reduced stack) 18 launches of 12-16 us became one of 13 us.  The row pitch of 2 TB + 32 bytes puts the four rows
// that 16 lanes read together into different banks.
// Memory bound at scale: at the headline batch one block's gradients read 4.1 KB per token, 2.1 GB.  Slices take
// every nslices-th step, so that each samples long and short users alike; the tiles of a slice, which share
// their operands' rows, run on one accelerator die (one L2).
// TILES: the operands are tile blocks in records (bw_block.h: rows are slots; ldx, ldy: sixteens of features from one tile to the next).  A step's
// tile is then contiguous in memory and goes to LDS as it is (a block of the headline batch 392 -> 370 us).
// GROUPED: a job may be of groups (with that read from the job in every launch's steps, those without one were slower too: 110 -> 115 us and 70 -> 75 us at
// width 64, 187 000 rows; both kinds' loops in one kernel 188 and 118)
template <int TB, bool TILES, bool GROUPED = false>
__global__ __launch_bounds__(256, TB == 128 ? 2 : 3) void bw_wgrad_kernel(const WgradArgs a) {
  constexpr int PITCH = TB + 16, TT = TB / 64, NCH = TB / 64;     // NCH: 16-byte chunks per thread, operand and step
  constexpr int CPR = TB / 8;                                     // chunks per row
  __shared__ __attribute__((aligned(16))) __bf16 sm[4 * 32 * PITCH];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int wm = w & 1, wn = w >> 1, hi = lane >> 5, l32 = lane & 31;
  const int slot = blockIdx.x >> 3, slice = (slot / a.tiles) * 8 + (blockIdx.x & 7);
  if (slice >= a.nslices) return;
  int t = slot % a.tiles;
  // (static offsets into the kernel arguments and scalar selects: no run-time index into a by-value argument)
  WgradJob jb = a.job[0];
#pragma unroll
  for (int i = 1; i < kMaxWgradJobs; ++i)
    if (i < a.njobs && t >= a.job[i].first) jb = a.job[i];
  t -= jb.first;
  const int sub = t % jb.nsub; t /= jb.nsub;
  const int tn = t % jb.tiles_n; t /= jb.tiles_n;
  const int tm = t % jb.tiles_m, layer = t / jb.tiles_m;
  const __bf16* X = jb.X + layer * jb.xstride;
  const __bf16* Y = jb.Y + layer * jb.ystride;
  const int m0 = tm * TB, n0 = tn * TB;
  const int kfirst = slice * jb.nsub + sub, kstride = a.nslices * jb.nsub;
  const int steps = (jb.rows + 31) / 32;
  const int nk = steps > kfirst ? (steps - kfirst + kstride - 1) / kstride : 0;

  f32x16 acc[TT][TT], accb[TT];
#pragma unroll
  for (int i = 0; i < TT; ++i) {
#pragma unroll
    for (int r = 0; r < 16; ++r) accb[i][r] = 0.f;
#pragma unroll
    for (int j = 0; j < TT; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  }
  // column sums of Y: one more product, ones [32, rows] Y, by the waves of the first row half of the first row tile
  const bool bias_sum = tm == 0 && wm == 0;
  bf16x8 ones;
#pragma unroll
  for (int e = 0; e < 8; ++e) ones[e] = (__bf16)(GROUPED && jb.groups ? 0.5f : 1.f);

  // Steps on their way from memory (registers: 16 a step at TB = 128, 8 at 64).  One, three workgroups a compute unit: steps of the headline, small
  // and raw-inputs models 4392 / 315 / 1291 us; two at the same occupancy, with spills at TB = 128: 4536 / 313 / 1317; this, two workgroups
  // of width 128 a compute unit and as many slices: 4390 / 312 / 1275.
  constexpr int PD = TB == 128 ? 3 : 4;
  bf16x8 rx[PD][NCH], ry[PD][NCH];
  bool there[PD][NCH];                       // (groups)
  const int two = GROUPED && jb.groups ? 1 : 0, row_end = two ? jb.groups : jb.rows, unit = GROUPED ? jb.unit : 1;
  auto first_row = [&](int kt) { return (kfirst + kt * kstride) >> two << 5; };
  auto gload = [&](int p, int kt) {
    const int k0 = (kfirst + kt * kstride) * 32;
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      const int c = tid + 256 * i, row = k0 + c / CPR, col = 8 * (c % CPR);
      if constexpr (TILES) {                 // (past the last column: any other one, its results are dropped)
        const size_t tile = (size_t)(k0 >> 5);
        const int gx = min(m0 / 16 + (c >> 6), jb.m / 16 - 1), gy = min(n0 / 16 + (c >> 6), jb.n / 16 - 1);
        rx[p][i] = *(const bf16x8*)(X + (tile * jb.ldx + gx) * 512 + 8 * (c & 63));
        ry[p][i] = *(const bf16x8*)(Y + ((tile >> two) * jb.ldy + gy) * 512 + 8 * (c & 63));
        if (GROUPED && two) {
          const int r = first_row(kt) + (((c & 63) >> 1) ^ (4 * ((c >> 6) & 1)));
          there[p][i] = r < row_end && row_valid(jb.rv, r, unit);
        }
      } else {
        bf16x8 z;
#pragma unroll
        for (int e = 0; e < 8; ++e) z[e] = (__bf16)0.f;
        rx[p][i] = z; ry[p][i] = z;
        if (row < jb.rows && row_valid(jb.rv, row)) {
          if (m0 + col < jb.m) rx[p][i] = *(const bf16x8*)(X + (size_t)row * jb.ldx + m0 + col);
          if (n0 + col < jb.n) ry[p][i] = *(const bf16x8*)(Y + (size_t)row * jb.ldy + n0 + col);
        }
      }
    }
  };
  auto next_step = [&](int kt) {
    while (kt < nk) {
      const int k0 = first_row(kt);
      if (rows_any_valid(jb.rv, k0, min(row_end, k0 + 32), unit)) break;
      ++kt;
    }
    return kt;
  };
  const int foff = TILES ? tile_tr_offset(lane, 8 * hi) : frag_t_offset<PITCH>(lane);
  // 32 columns from x on, contraction rows 16 ks ..: eight rows per lane half
  auto frag = [&](const __bf16* s, int x, int ks) -> bf16x8 {
    if constexpr (TILES) {
      const char* q = (const char*)s + x * 64 + 512 * ks;
      return join_tr(__builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(q + foff)),
                     __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(q + (foff ^ 128))));
    } else {
      return frag_t<PITCH>(s + foff + 16 * ks * PITCH + x);
    }
  };
  int buf = 0, kn = next_step(0);            // kn: the next step to request
  bool have[PD];
  auto request = [&](int p) {
    have[p] = kn < nk;
    if (!have[p]) return;
    gload(p, kn);
    kn = next_step(kn + 1);
  };
#pragma unroll
  for (int p = 0; p < PD; ++p) request(p);
  while (have[0]) {
#pragma unroll
    for (int p = 0; p < PD; ++p) {
      if (p > 0 && !have[p]) { have[0] = false; break; }      // (requests are made in order: nothing comes after one that is missing)
      __bf16* sx = sm + buf * (2 * 32 * PITCH);
      __bf16* sy = sx + 32 * PITCH;
#pragma unroll
      for (int i = 0; i < NCH; ++i) {
        const int c = tid + 256 * i, o = TILES ? 8 * c : (c / CPR) * PITCH + 8 * (c % CPR);
        if (GROUPED && two) { rx[p][i] = keep_if(rx[p][i], there[p][i]); ry[p][i] = keep_if(ry[p][i], there[p][i]); }
        *(bf16x8*)&sx[o] = rx[p][i];
        *(bf16x8*)&sy[o] = ry[p][i];
      }
      request(p);
      __syncthreads();       // (the other buffer was last read two steps ago, ahead of the previous barrier)
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        bf16x8 fx[TT], fy[TT];
#pragma unroll
        for (int i = 0; i < TT; ++i) {
          fx[i] = frag(sx, (TB / 2) * wm + 32 * i, ks);
          fy[i] = frag(sy, (TB / 2) * wn + 32 * i, ks);
        }
#pragma unroll
        for (int i = 0; i < TT; ++i)
#pragma unroll
          for (int j = 0; j < TT; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fx[i], fy[j], acc[i][j], 0, 0, 0);
        if (bias_sum) {
#pragma unroll
          for (int j = 0; j < TT; ++j) accb[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ones, fy[j], accb[j], 0, 0, 0);
        }
      }
      buf ^= 1;
    }
  }
  float* out = jb.part + ((size_t)layer * kstride + kfirst) * ((size_t)jb.m * jb.n + jb.n);
#pragma unroll
  for (int i = 0; i < TT; ++i)
#pragma unroll
    for (int j = 0; j < TT; ++j) {
      const int n = n0 + (TB / 2) * wn + 32 * j + l32, mb = m0 + (TB / 2) * wm + 32 * i;
      if (n >= jb.n || mb >= jb.m) continue;               // (m and n are multiples of 32)
#pragma unroll
      for (int r = 0; r < 16; ++r) out[(size_t)(mb + tile_row(r, hi)) * jb.n + n] = acc[i][j][r];
    }
  if (bias_sum && hi == 0) {
#pragma unroll
    for (int j = 0; j < TT; ++j) {
      const int n = n0 + (TB / 2) * wn + 32 * j + l32;
      if (n < jb.n) out[(size_t)jb.m * jb.n + n] = accb[j][0];
    }
  }
}

// Sums of partial results: out = sum over the slices of part[slice][m n + n], for every job (and layer) of a
// launch.  Columns come in blocks of nb (the three matrices of [W_Q | W_K | W_V] are one job): column block j, its
// m rows and then its n-vector, goes to out + j (m nb + nb).  m = 0: a plain vector of n (the LayerNorms' [gain | shift]).
// A workgroup sums 4 CX adjacent outputs, its 256 / CX rows of threads each every (256 / CX)-th slice.  CX = 64 for the matrices, 128 up to 16 slices: a thread
// has about ten slices to ask for at once (with 16 it was one or two, and 15 000 workgroups came and went: 28.8 -> 16.8 us for the 56 MB of a step of the headline
// model; steps of 8 x 100 and 32 x 400 tokens of width 128, which have few slices, 392 and 460 us, with 64 throughout 393 and 462, with 16 409 and 473).  16 for matrices of at most
// 16 384 elements and more slices than that, where 64 leaves too few workgroups (64 x 256 of 40 slices 14.0 -> 10.6 us; a step of 128 x 2000 tokens of
// width 32 267 us, with 64 throughout 271, with 128 278; of 64 x 3000 tokens of width 64 425, 427, 430).  4 for the
// vectors (hundreds of slices).  Every sum is taken in a fixed order.
struct ReduceJob {
  const float* part; float* out;
  long long sstride, plstride, olstride;    // floats from slice to slice, from layer to layer (partial, output)
  int nslices, m, n, nb, layers, cxlog, blocks, first;   // blocks: workgroups per layer; first: its first workgroup
};
constexpr int kMaxReduceJobs = 18;
struct ReduceArgs { ReduceJob job[kMaxReduceJobs]; int njobs; };

__global__ __launch_bounds__(256) void bw_reduce_jobs_kernel(const ReduceArgs a) {
  __shared__ f32x4 red[256];
  int b = blockIdx.x;
  ReduceJob jb = a.job[0];
#pragma unroll
  for (int i = 1; i < kMaxReduceJobs; ++i)
    if (i < a.njobs && b >= a.job[i].first) jb = a.job[i];
  b -= jb.first;
  const int layer = b / jb.blocks, blk = b - layer * jb.blocks;
  const int cx = 1 << jb.cxlog, ny = 256 >> jb.cxlog;
  const int x = threadIdx.x & (cx - 1), y = threadIdx.x >> jb.cxlog;
  const long long i4 = 4ll * ((long long)blk * cx + x), count = (long long)jb.m * jb.n + jb.n;
  f32x4 s = {0.f, 0.f, 0.f, 0.f};
  if (i4 < count) {
    const float* p = jb.part + layer * jb.plstride + i4;
#pragma unroll 4
    for (int sl = y; sl < jb.nslices; sl += ny) s += *(const f32x4*)(p + sl * jb.sstride);
  }
  red[threadIdx.x] = s;
  __syncthreads();
  for (int h = ny >> 1; h > 0; h >>= 1) {
    if (y < h) red[threadIdx.x] += red[threadIdx.x + (h << jb.cxlog)];
    __syncthreads();
  }
  if (y == 0 && i4 < count) {
    const int row = (int)(i4 / jb.n), col = (int)(i4 - (long long)row * jb.n);
    const int cb = col / jb.nb, cc = col - cb * jb.nb;
    float* o = jb.out + layer * jb.olstride + (size_t)cb * ((size_t)jb.m * jb.nb + jb.nb) + (size_t)row * jb.nb + cc;
    *(f32x4*)o = red[x];
  }
}

// ------------------------------------------------------------------------------------ host side
// Slices of a launch with `tiles` output tiles over `rows` rows: enough workgroups to fill the chip two deep
// (what fits a compute unit at width 128), but at least four row steps (128 rows) each.  A job with fewer rows than the launch's (groups, the last
// layer's global rows) has as many slices, shorter ones; those beyond its last step are zeros in its sum.
static inline int wgrad_slices(int tiles, size_t rows) {
  const int steps = (int)((rows + 31) / 32);
  int s = 2 * kComputeUnits / (tiles > 0 ? tiles : 1);
  if (s > steps / 4) s = steps / 4;
  if (s > 8) s = s / 8 * 8;                 // (slices are dealt to the 8 dies)
  return s < 1 ? 1 : s;
}
static inline int wgrad_tile(int d) { return d >= 128 ? 128 : 64; }

// The matrices of a launch, then their reductions.  Used twice with the same calls: without a base pointer
// to learn how many floats of partial results the launch needs, and with one to launch it.
struct WgradBatch {
  WgradArgs a = {};
  bool tiled;                               // the operands are tile blocks
  int tb; size_t rows;                      // rows: of the jobs with nsub = 1 (sets the number of slices)
  struct Out { float* out; long long olstride; int nb; } outs[kMaxWgradJobs];
  WgradBatch(int d, size_t rows_, bool tiled_ = false) : tiled(tiled_), tb(wgrad_tile(d)), rows(rows_) {}
  void add(const __bf16* X, int ldx, int m, const __bf16* Y, int ldy, int n, int nb, size_t nrows, RowsValid rv, float* out,
           int layers = 1, long long xstride = 0, long long ystride = 0, long long olstride = 0, int groups = 0, int unit = 1) {
    WgradJob& j = a.job[a.njobs];
    j.groups = groups; j.unit = unit;
    j.X = X; j.Y = Y; j.ldx = ldx; j.ldy = ldy; j.m = m; j.n = n; j.rows = (int)nrows; j.rv = rv;
    j.tiles_m = (m + tb - 1) / tb; j.tiles_n = (n + tb - 1) / tb; j.layers = layers;
    j.nsub = nrows > rows ? (int)((nrows + rows - 1) / rows) : 1;
    j.xstride = xstride; j.ystride = ystride; j.first = a.tiles;
    a.tiles += j.tiles_m * j.tiles_n * layers * j.nsub;
    outs[a.njobs] = Out{out, olstride, nb};
    ++a.njobs;
  }
  // floats of partial results, and where each job's start
  size_t place(float* base) {
    a.nslices = wgrad_slices(a.tiles, rows);
    size_t o = 0;
    for (int i = 0; i < a.njobs; ++i) {
      WgradJob& j = a.job[i];
      j.part = base ? base + o : nullptr;
      o += (size_t)j.layers * a.nslices * j.nsub * ((size_t)j.m * j.n + j.n);
    }
    return o;
  }
};

struct ReduceBatch {
  ReduceArgs a = {};
  int blocks = 0;
  void add(const float* part, long long sstride, int nslices, int m, int n, int nb, float* out, int layers, long long plstride,
           long long olstride) {
    ReduceJob& j = a.job[a.njobs++];
    j.part = part; j.out = out; j.sstride = sstride; j.nslices = nslices; j.m = m; j.n = n; j.nb = nb; j.layers = layers;
    j.plstride = plstride; j.olstride = olstride; j.cxlog = !m ? 2 : nslices > 16 ? (m * n <= 16384 ? 4 : 6) : 7;
    const long long groups = ((long long)m * n + n) / 4;
    j.blocks = (int)((groups + (1 << j.cxlog) - 1) >> j.cxlog);
    j.first = blocks;
    blocks += j.blocks * layers;
  }
  // the LayerNorm partials [nslices][2 d] of a launch (per layer plstride floats apart)
  void add_ln(const float* part, int nslices, int d, float* out, int layers = 1, long long plstride = 0, long long olstride = 0) {
    add(part, 2 * d, nslices, 0, 2 * d, 2 * d, out, layers, plstride, olstride);
  }
  void add(const WgradBatch& w) {
    for (int i = 0; i < w.a.njobs; ++i) {
      const WgradJob& j = w.a.job[i];
      const long long per = (long long)j.m * j.n + j.n;
      add(j.part, per, w.a.nslices * j.nsub, j.m, j.n, w.outs[i].nb, w.outs[i].out, j.layers, per * w.a.nslices * j.nsub, w.outs[i].olstride);
    }
  }
};

}  // namespace bw
}  // namespace longer
