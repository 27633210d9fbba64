// fp32 kernels of the GTA pass for gfx950: fp32 operands, fp32 MFMA (v_mfma_f32_32x32x2 / 16x16x4: products
// and sums in fp32, twice the rate of the vector ALU), for the shapes the conditions at the end of this file
// name; everything else stays on the shape-generic kernels.
//
// The fp32 matrix instructions are slow next to everything that feeds them (64 cycles for 2048 products), so
// the kernels here need no elaborate schedule: what decides is that every SIMD has work and that operands are
// requested early.  The contraction index of an MFMA step is only a label: as long as both operands use the
// same assignment of k to (step, lane half), any assignment computes the same sum.  Operands that are
// contiguous along k are therefore read 16 bytes per lane, and lane half h covers k = 4h .. 4h+3 of every
// eight, one k per step.
#include <math.h>

#include <algorithm>

#include "gta_epilogues.h"
#include "gta_tuned.h"

namespace gta {
namespace {

typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ void zero16(f32x16 &v) {
#pragma unroll
  for (int r = 0; r < 16; ++r) v[r] = 0.f;
}
// value of the lane pair's other half (lanes l and l + 32) combined by max / sum
__device__ __forceinline__ float pair_max(float v) {
  const u32x2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float pair_sum(float v) {
  const u32x2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// ------------------------------------------------------------------------------ operands
// Both operands for the columns from `col` on: the segment they lie in (projection), or the head they belong to
// (decoder: the left operand then starts at the head's map group).
struct GemmOperands {
  const float *A; int lda, M, K;
  const float *B[4]; int ldb[4], seg_cols[4];   // segments side by side (unused ones have 0 columns)
  int heads_per_group, a_group_stride;          // decoder: > 0; B[0] is [n_h, K, seg_cols[0]]
  int tiles;                                    // of the launch (few rows)
};
__device__ __forceinline__ void operand_at(const GemmOperands &g, int col, const float *&A, const float *&B, int &ldb) {
  A = g.A;
  if (g.heads_per_group) {
    const int head = col / g.seg_cols[0];
    A += (int64_t)(head / g.heads_per_group) * g.a_group_stride;
    B = g.B[0] + (int64_t)head * g.K * g.seg_cols[0] + col % g.seg_cols[0];
    ldb = g.seg_cols[0];
    return;
  }
  int seg = 0;
  while (seg < 3 && col >= g.seg_cols[seg]) { col -= g.seg_cols[seg]; ++seg; }
  B = g.B[seg] + col;
  ldb = g.ldb[seg];
}

// ------------------------------------------------------------------------------ few rows: K split over waves
// Tile of 32 rows x BN columns (or 16 x 16); the W waves of the workgroup each take every W-th group of KG k and read
// their operand fragments straight from memory (nothing is shared between the waves, so LDS would only add a round
// trip), U groups in flight; the W partial tiles are summed through LDS in a fixed order.  For a decode step's
// rows and short prompts: what bounds these is the latency of a few loads and how many workgroups pull on the
// weights, not arithmetic.  A tile that is rotated must hold both halves of its heads: with heads wider than the tile it
// takes half its columns of one half and those they pair with, otherwise (whole heads fit) columns in a row.
constexpr int kRowsInFlight = 5;   // U
template <int W, int BM, int BN, bool LONG, class Epi>
__global__ __launch_bounds__(64 * W) void gemm_rows_f32_kernel(GemmOperands g, Epi epi) {
  constexpr int MT = BN == 32 ? 32 : 16, NSUB = BM / MT;   // MFMA tile, tiles of rows
  constexpr int U = kRowsInFlight, PITCH = BN + 4, KG = 256 / MT, HB = BN / 2, GR = BN / 4;   // GR: groups of four columns a row
  extern __shared__ __attribute__((aligned(16))) float red[];   // [W][BM][PITCH]
  const int tid = threadIdx.x, lane = tid & 63, h = lane / MT, ln = lane % MT;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // consecutive workgroup ids go to different XCDs; each XCD takes a contiguous eighth of the tiles, row tiles
  // fastest: neighbouring tiles share the 128-byte lines of the weights, which should reach one L2 only
  const int id = blockIdx.x, per = g.tiles / 8, at = id < per * 8 ? (id % 8) * per + id / 8 : id;
  if (id >= g.tiles) { epi.commit((id - g.tiles) * W + wave); return; }
  const int ntm = (g.M + BM - 1) / BM, nt = at / ntm, m0 = at % ntm * BM;
  const bool rot = epi.rotates(nt * BN);
  const RowTile ct = row_tile<BN>(nt, rot, epi.head_dim());
  const int col0 = ct.col0, step = ct.step;
  const float *A, *B;
  int ldb;
  operand_at(g, col0, A, B, ldb);
  const float *ap[NSUB];
#pragma unroll
  for (int i = 0; i < NSUB; ++i) ap[i] = A + (int64_t)min(m0 + i * MT + ln, g.M - 1) * g.lda + h * 4;
  const float *bp = B + (int64_t)(h * 4) * ldb + ln % HB + ln / HB * step;
  typedef float accvec __attribute__((ext_vector_type(MT * MT / 64)));
  accvec acc[NSUB];
#pragma unroll
  for (int i = 0; i < NSUB; ++i)
#pragma unroll
    for (int r = 0; r < MT * MT / 64; ++r) acc[i][r] = 0.f;
  const int ng = g.K / KG;
  f32x4 a[U][NSUB], b[U];
  // groups past the end re-read the last one; they are not used (a branch around the loads instead: 64 rows of the paper's
  // layer 54 us a step, not 50)
  auto load = [&](int u, int c) {
    const int k = min(c, ng - 1) * KG;
#pragma unroll
    for (int i = 0; i < NSUB; ++i) a[u][i] = *reinterpret_cast<const f32x4 *>(ap[i] + k);
#pragma unroll
    for (int j = 0; j < 4; ++j) b[u][j] = bp[(int64_t)(k + j) * ldb];
  };
  const int row = tid / GR, c = tid % GR * 4, fcol = col0 + c % HB + c / HB * step;   // what this thread finishes
  const bool finisher = tid < BM * GR && m0 + row < g.M;
  typename Epi::Early early{};
  if (finisher) early = epi.early(m0 + row, fcol, rot);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int u = 0; u < U; ++u) load(u, wave + u * W);
  __builtin_amdgcn_sched_barrier(0);
  typename Epi::Ctx ctx{};
  if (finisher) ctx = epi.prepare(early, m0 + row, fcol, rot);
  auto multiply = [&](int u) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int i = 0; i < NSUB; ++i) {
        if constexpr (MT == 32) acc[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[u][i][j], b[u][j], acc[i], 0, 0, 0);
        else acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u][i][j], b[u][j], acc[i], 0, 0, 0);
      }
  };
  // Requests behind the last round are left out (they took 3 to 6 us of 40 to 90 at K = 1280).  A branch around each in the loop
  // costs a contraction of more than one round (LONG) more than that: 32 x 32 tiles at K = 4096, 60 heads, 128 rows 128 us,
  // unconditional 124, last round apart 111; K = 8192, 200 rows 148, 138, 123; 16-column tiles, 20 rows 43.8, 44.0, 41.6.  Of a single
  // round it is the faster form: 64 x 2048 rows of the paper's layer 49.3 us, last round apart 51.8; K = 640, 256 rows 31.5, 32.8.
  int c0 = wave;
  if constexpr (LONG) {
    for (; c0 + U * W < ng; c0 += U * W) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        multiply(u);
        load(u, c0 + (u + U) * W);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (c0 + u * W < ng) multiply(u);
  } else {
    for (; c0 < ng; c0 += U * W) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (c0 + u * W < ng) multiply(u);
        if (c0 + U * W < ng) load(u, c0 + (u + U) * W);
      }
    }
  }
  float *mine = red + wave * BM * PITCH;
#pragma unroll
  for (int i = 0; i < NSUB; ++i)
#pragma unroll
    for (int r = 0; r < MT * MT / 64; ++r)
      mine[(i * MT + 256 / MT * (r >> 2) + 4 * h + (r & 3)) * PITCH + ln] = acc[i][r];
  __syncthreads();
  auto sum4 = [&](int row, int col) {
    const float *p = red + row * PITCH + col;
    f32x4 v = *reinterpret_cast<const f32x4 *>(p);
#pragma unroll
    for (int w = 1; w < W; ++w) v += *reinterpret_cast<const f32x4 *>(p + w * BM * PITCH);
    return v;
  };
  if (!finisher) return;
  epi.store(ctx, m0 + row, sum4(row, c), [&](int off) { return sum4(row, c + (ct.pair ? (off > 0 ? HB : -HB) : off)); });
}

// ------------------------------------------------------------------------------ many rows: LDS tiles
// Tile 64 x 64 x 16, four waves of 32 x 32, two LDS stages, 19 KiB of LDS, so that up to five workgroups share a CU
// and cover each other's loads and barriers.  Bound by the fp32 MFMA rate (153 TFLOP/s measured for a large library
// GEMM).  Small tiles because they divide evenly over the CUs: 4096 rows of the paper's layer are 7 (projection) and
// 5 (W_O) tiles a CU; 128 x 64 tiles are 3.5 and 2.5, and that call takes 374 us instead of 361 (512 rows: 138
// instead of 88).  The finished tile is parked in LDS and handed to the epilogue in groups of four columns.
template <class Epi>
__global__ __launch_bounds__(256) void gemm_tiles_f32_kernel(GemmOperands g, int ntn, Epi epi) {
  constexpr int BM = 64, BN = 64, BK = 16, TM = BM / 64;
  constexpr int AP = BK + 4, BP = BN + 4, OP = BN + 4;   // pitches in floats; AP = 4 * odd: conflict-free b128 reads
  constexpr int STAGE = BM * AP + BK * BP;
  __shared__ __attribute__((aligned(16))) float sm[2 * STAGE > BM * OP ? 2 * STAGE : BM * OP];
  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, ln = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave >> 1, wn = wave & 1;
  // consecutive workgroup ids go to different XCDs; each XCD takes a contiguous eighth of the tiles, columns
  // fastest, so that the workgroups of an XCD share row strips in its L2
  const int id = blockIdx.x, per = gridDim.x / 8;
  const int at = id < per * 8 ? (id % 8) * per + id / 8 : id;
  const int nt = at % ntn, m0 = (at / ntn) * BM;
  const float *A, *B;
  int ldb;
  operand_at(g, nt * BN, A, B, ldb);
  // A: BK/4 chunks of 16 bytes per row, AR rows a pass; B: row tid/16 + 16 i, chunk tid%16
  constexpr int AC = BK / 4, AR = 256 / AC, AL = BM / AR, BL = BK / 16;
  const int ar = tid / AC, ac = tid % AC * 4, br = tid >> 4, bc = (tid & 15) * 4;
  const float *ap[AL];
#pragma unroll
  for (int i = 0; i < AL; ++i) ap[i] = A + (int64_t)min(m0 + ar + AR * i, g.M - 1) * g.lda + ac;
  const float *bp = B + (int64_t)br * ldb + bc;
  struct Regs { f32x4 a[AL], b[BL]; };
  const int nk = g.K / BK;
  auto gload = [&](Regs &r, int kt) {   // tiles past the end re-read the last one; they are not used
    kt = min(kt, nk - 1);
#pragma unroll
    for (int i = 0; i < AL; ++i) r.a[i] = *reinterpret_cast<const f32x4 *>(ap[i] + kt * BK);
#pragma unroll
    for (int i = 0; i < BL; ++i) r.b[i] = *reinterpret_cast<const f32x4 *>(bp + (int64_t)(kt * BK + 16 * i) * ldb);
  };
  auto sstore = [&](float *st, const Regs &r) {
#pragma unroll
    for (int i = 0; i < AL; ++i) *reinterpret_cast<f32x4 *>(st + (ar + AR * i) * AP + ac) = r.a[i];
#pragma unroll
    for (int i = 0; i < BL; ++i) *reinterpret_cast<f32x4 *>(st + BM * AP + (br + 16 * i) * BP + bc) = r.b[i];
  };
  f32x16 acc[TM];
#pragma unroll
  for (int t = 0; t < TM; ++t) zero16(acc[t]);
  auto compute = [&](const float *st) {
#pragma unroll
    for (int c = 0; c < BK / 8; ++c) {
      f32x4 xa[TM];
      float xb[4];
#pragma unroll
      for (int t = 0; t < TM; ++t)
        xa[t] = *reinterpret_cast<const f32x4 *>(st + (wm * (BM / 2) + t * 32 + ln) * AP + c * 8 + h * 4);
#pragma unroll
      for (int j = 0; j < 4; ++j) xb[j] = st[BM * AP + (c * 8 + h * 4 + j) * BP + wn * 32 + ln];
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int t = 0; t < TM; ++t) acc[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(xa[t][j], xb[j], acc[t], 0, 0, 0);
    }
  };
  // loads run two tiles ahead of the LDS writes: a tile's 512 cycles of MFMA do not cover a trip to memory
  Regs r0, r1;
  gload(r0, 0);
  gload(r1, 1);
  sstore(sm, r0);
  gload(r0, 2);
  __syncthreads();
  for (int kt = 0; kt + 1 < nk; kt += 2) {
    compute(sm);
    sstore(sm + STAGE, r1);
    gload(r1, kt + 3);
    __syncthreads();
    compute(sm + STAGE);
    sstore(sm, r0);
    gload(r0, kt + 4);
    __syncthreads();
  }
  if (nk & 1) {
    compute(sm);
    __syncthreads();
  }
#pragma unroll
  for (int t = 0; t < TM; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r)
      sm[(wm * (BM / 2) + t * 32 + 8 * (r >> 2) + 4 * h + (r & 3)) * OP + wn * 32 + ln] = acc[t][r];
  __syncthreads();
  const bool rot = epi.rotates(nt * BN);
#pragma unroll 4
  for (int i = tid; i < BM * (BN / 4); i += 256) {
    const int row = i / (BN / 4), col = (i % (BN / 4)) * 4;
    if (m0 + row >= g.M) continue;
    const float *p = sm + row * OP + col;
    epi.store(epi.prepare(epi.early(m0 + row, nt * BN + col, rot), m0 + row, nt * BN + col, rot), m0 + row, *reinterpret_cast<const f32x4 *>(p),
              [&](int off) { return *reinterpret_cast<const f32x4 *>(p + off); });
  }
}

// ------------------------------------------------------------------------------ prefill attention
// L_g = Softmax(Q_g K^T / sqrt(d_h)) C for 32 queries of one (sequence, map group) and one slice of DLW latent
// columns.  The four waves of the workgroup take the 32-key blocks of the causal range in turn (block w, w + 4,
// ..), each with its own online softmax, and merge at the end: the longest chain of blocks is a quarter of the
// sequence, and 32-query tiles leave enough workgroups to fill the chip at a few thousand tokens.  Both products
// are transposed (S^T = K Q^T, L^T += C^T P^T), so a lane holds one query: the statistics are per lane pair, and
// the probabilities are the second product's operand as they stand.  Operands come straight from memory: a key
// row is read 16 bytes per lane, a latent row as 32 lanes x 16 (or 8) bytes, each requested one block ahead into the
// registers its predecessor has just left.  Later tokens never reach earlier rows, whatever they hold: in the block on
// the diagonal their probability of 0 turns a latent that is not finite into NaN, so a wave whose sums over that block
// are not finite forms its part again key by key.  (Looked at behind the loop: a test of the block's latents
// inside it keeps softmax and products from overlapping, 61 us instead of 57 at 4 x 1024 tokens of the paper's layer.)
struct AttnF32 {
  const float *q, *k, *c; float *L;
  const int32_t *cu; int per_seq, max_len;
  int nq, qpk, qpc, wq_w, wk_w, wc_w, dl, n_qtiles, nslice, batch;
  int back;   // PAIR: workgroups i < 256 take tile i, the others tile back - i
  float scale_log2e;
};

template <int DH, int DLW, bool PAIR>
__global__ __launch_bounds__(256, DH + DLW < 256 ? 2 : 1) void attn_prefill_f32_kernel(AttnF32 a) {
  constexpr int NT = DLW / 32, OP = DLW + 4;
  typedef float cvec __attribute__((ext_vector_type(NT)));
  extern __shared__ __attribute__((aligned(16))) float dyn[];
  float (*lacc)[32][OP] = reinterpret_cast<float (*)[32][OP]>(dyn);   // [4][32][OP]
  __shared__ float sm[4][32], sl[4][32];
  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, ln = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // longest query tiles first; inside a level the maps of one sequence side by side (they share keys and latents)
  // A CU holds two workgroups (DH + DLW < 256; heads of 32 and latent tiles of 64: three, but is given a second one only when all have
  // one).  Where the chip holds all of them, those behind the first 256 go backwards, so that the longest shares its CU with the
  // shortest of them: paper's layer 2 x 1500 tokens (470 workgroups) 306 -> 293 us, 768 wide layer 4 x 1000 (384) 173 -> 168, 16 heads of
  // 32, 4 maps, 9 x 400 (468) 61.2 -> 59.3.  A few behind the first 256 lose more than they gain: 768 wide layer 3 x 1000 (288) 149.9 -> 150.7,
  // 5 x 600 (285) 112.7 -> 113.1, paper's layer 2 x 896 (280) 200.9 -> 201.5, but 2 x 928 (290) 206.8 -> 204.3.  Larger launches even
  // it out by themselves (4 x 1024, 640: 357, backwards 360) and are kernels of their own: the choice alone, made at run time, took
  // 0.6 of their 360 us.
  const int per_qt = a.batch * a.nq * a.nslice, id = !PAIR || blockIdx.x < 256 ? (int)blockIdx.x : a.back - (int)blockIdx.x;
  const int lvl = id / per_qt, rest = id % per_qt;
  const int qt = a.n_qtiles - 1 - lvl;
  const int sl_i = rest % a.nslice, g = rest / a.nslice % a.nq, b = rest / (a.nslice * a.nq);
  const int64_t start = a.cu ? a.cu[b] : (int64_t)b * a.per_seq;
  const int Tb = min(a.cu ? a.cu[b + 1] - a.cu[b] : a.per_seq, a.max_len);
  const int q0 = qt * 32;
  if (q0 >= Tb) return;
  const int nkeys = min(q0 + 32, Tb), nblk = (nkeys + 31) / 32;
  const float *K = a.k + start * a.wk_w + (g / a.qpk) * DH + h * 4;
  const float *C = a.c + start * a.wc_w + (g / a.qpc) * a.dl + sl_i * DLW + ln * NT;

  f32x4 qf[DH / 8];
  {
    const float *qp = a.q + (start + min(q0 + ln, Tb - 1)) * a.wq_w + g * DH + h * 4;
#pragma unroll
    for (int c = 0; c < DH / 8; ++c) qf[c] = *reinterpret_cast<const f32x4 *>(qp + c * 8);
  }
  f32x16 acc[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) zero16(acc[t]);
  float m = -INFINITY, l = 0.f;
  f32x4 kf[DH / 8];
  cvec cf[16];
  // rows past the visible keys (and blocks past the last) re-read the last row; they are masked or not used
  auto kload = [&](int blk) {
    const float *p = K + (int64_t)min(blk * 32 + ln, nkeys - 1) * a.wk_w;
#pragma unroll
    for (int c = 0; c < DH / 8; ++c) kf[c] = *reinterpret_cast<const f32x4 *>(p + c * 8);
  };
  auto cload = [&](int blk, int r) {   // key of register r in lane half h: 8 (r / 4) + 4 h + r % 4
    cf[r] = *reinterpret_cast<const cvec *>(C + (int64_t)min(blk * 32 + 8 * (r >> 2) + 4 * h + (r & 3), nkeys - 1) * a.wc_w);
  };
  if (wave < nblk) {
    kload(wave);
#pragma unroll
    for (int r = 0; r < 16; ++r) cload(wave, r);
  }
  for (int blk = wave; blk < nblk; blk += 4) {
    f32x16 s;
    zero16(s);
#pragma unroll
    for (int c = 0; c < DH / 8; ++c)
#pragma unroll
      for (int j = 0; j < 4; ++j) s = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[c][j], qf[c][j], s, 0, 0, 0);
    kload(blk + 4);
    if (blk * 32 + 31 > q0) {   // the block on the diagonal
      const int lim = q0 + ln - blk * 32;
#pragma unroll
      for (int r = 0; r < 16; ++r) s[r] = 8 * (r >> 2) + 4 * h + (r & 3) > lim ? -INFINITY : s[r];
    }
    float bm = s[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) bm = fmaxf(bm, s[r]);
    // the running maximum moves only when a block passes it by 2^8 (fp32 probabilities carry any such scale); it
    // stays -inf over blocks whose scores have all overflowed to -inf
    const float mc = pair_max(bm) * a.scale_log2e, mn = mc > m + 8.f ? mc : m, ref = mn > -INFINITY ? mn : 0.f;
    const float corr = __builtin_amdgcn_exp2f(m - ref);
    m = mn;
    float ps = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      s[r] = __builtin_amdgcn_exp2f(fmaf(s[r], a.scale_log2e, -ref));
      ps += s[r];
    }
    l = fmaf(l, corr, ps);
    if (__builtin_amdgcn_ballot_w64(corr != 1.f) != 0) {
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[t][r] *= corr;
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {
#pragma unroll
      for (int t = 0; t < NT; ++t) acc[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(cf[r][t], s[r], acc[t], 0, 0, 0);
      cload(blk + 4, r);
    }
  }
  // sums of the wave that holds the diagonal not finite: its blocks again, every query on the keys it sees (registers are
  // scarce here, not time: 24 tokens of NaN behind 1000 in four sequences of the paper's layer 60 -> 400 us)
  bool finite = true;
  if (wave == (nblk - 1) % 4) {
    float z[4] = {};
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) z[r % 4] = fmaf(acc[t][r], 0.f, z[r % 4]);
    finite = __builtin_amdgcn_ballot_w64((z[0] + z[1]) + (z[2] + z[3]) != 0.f) == 0;
  }
  if (__builtin_expect(!finite, 0)) {
#pragma unroll
    for (int t = 0; t < NT; ++t) zero16(acc[t]);
    m = -INFINITY;
    l = 0.f;
    const float *qr = a.q + (start + min(q0 + ln, Tb - 1)) * a.wq_w + g * DH + h * 4;
#pragma unroll 1
    for (int j = wave * 32; j < min(q0 + ln + 1, nkeys); j += (j & 31) == 31 ? 97 : 1) {
      const float *kr = K + (int64_t)j * a.wk_w, *cr = C + (4 * h - ln) * NT + (int64_t)j * a.wc_w;
      float d = 0.f;
#pragma unroll 1
      for (int c = 0; c < DH; c += 8) {
        const f32x4 k = *reinterpret_cast<const f32x4 *>(kr + c), q = *reinterpret_cast<const f32x4 *>(qr + c);
#pragma unroll
        for (int i = 0; i < 4; ++i) d = fmaf(k[i], q[i], d);
      }
      const float sc = pair_sum(d) * a.scale_log2e, mn = fmaxf(m, sc), ref = mn > -INFINITY ? mn : 0.f;
      const float corr = __builtin_amdgcn_exp2f(m - ref), p = __builtin_amdgcn_exp2f(sc - ref);
      m = mn;
      l = fmaf(l, corr, h == 0 ? p : 0.f);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const cvec c = *reinterpret_cast<const cvec *>(cr + (8 * (r >> 2) + (r & 3)) * NT);
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[t][r] = fmaf(p, c[t], acc[t][r] * corr);
      }
    }
  }
  // merge the waves: tile t, register r of a lane is column (8 (r/4) + 4 h + r % 4) * NT + t of its query
  l = pair_sum(l);
  if (h == 0) { sm[wave][ln] = m; sl[wave][ln] = l; }
  __syncthreads();
  float mx = sm[0][ln];
#pragma unroll
  for (int w = 1; w < 4; ++w) mx = fmaxf(mx, sm[w][ln]);
  const float ws = m > -INFINITY ? __builtin_amdgcn_exp2f(m - mx) : 0.f;   // a wave without blocks
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    cvec v;
#pragma unroll
    for (int t = 0; t < NT; ++t) v[t] = acc[t][r] * ws;
    *reinterpret_cast<cvec *>(&lacc[wave][ln][(8 * (r >> 2) + 4 * h + (r & 3)) * NT]) = v;
  }
  __syncthreads();
  for (int i = tid; i < 32 * (DLW / 4); i += 256) {
    const int row = i / (DLW / 4), col = (i % (DLW / 4)) * 4;
    if (q0 + row >= Tb) continue;
    float rm = sm[0][row];
#pragma unroll
    for (int w = 1; w < 4; ++w) rm = fmaxf(rm, sm[w][row]);
    float ls = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) ls += sm[w][row] > -INFINITY ? sl[w][row] * __builtin_amdgcn_exp2f(sm[w][row] - rm) : 0.f;
    f32x4 v = *reinterpret_cast<const f32x4 *>(&lacc[0][row][col]);
#pragma unroll
    for (int w = 1; w < 4; ++w) v += *reinterpret_cast<const f32x4 *>(&lacc[w][row][col]);
    const float inv = 1.0f / ls;
    *reinterpret_cast<f32x4 *>(a.L + (start + q0 + row) * (int64_t)(a.nq * a.dl) + g * a.dl + sl_i * DLW + col) = v * inv;
  }
}

// ------------------------------------------------------------------------------ decode attention
// Split-K stream over the caches for shapes with ONE key and ONE latent shared by all (at most 16) maps: a
// workgroup of four waves takes a slice of a sequence's rows, a wave 16 rows per step with
// v_mfma_f32_16x16x4_f32 (columns = the maps, padded to 16; the padding costs matrix time that the stream does
// not need).  A key row is read by four lanes of 16 bytes per 64-byte piece, a latent row by 16 lanes of 16
// bytes per 256-byte piece, straight into operand layout; two steps are in flight per wave.  The score
// registers of a step (row 4 (lane / 16) + r, map lane % 16) are the operand of the second product as they are.
struct DecF32 {
  const float *q; const int32_t *oldlen;         // [batch, n_q*d_h] rotated; newest row that takes part, or -1
  const float *kc, *cc; const int32_t *slots; int max_seq; PageMap pm; int ps_shift;
  int nq, splits; float scale_log2e;
  float *pacc, *pml;
};

template <int DH, int DL>
__global__ __launch_bounds__(256, 2) void decode_attn_f32_kernel(DecF32 a) {
  constexpr int KC = DH / 16, NU = DL / 64, OP = DL + 4;
  __shared__ __attribute__((aligned(16))) float lacc[4][16][OP];
  __shared__ float sm[4][16], sl[4][16];
  const int tid = threadIdx.x, lane = tid & 63, kq = lane >> 4, ln = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int s = blockIdx.x, b = blockIdx.y;
  float *pa = a.pacc + (int64_t)(b * a.splits + s) * a.nq * DL, *pml = a.pml + (int64_t)(b * a.splits + s) * a.nq * 2;
  const int old = a.oldlen[b];
  if (old < 0) {   // no rows (or slot full): weight 0 for the merge
    if (tid < a.nq) { pml[2 * tid] = -INFINITY; pml[2 * tid + 1] = 0.f; }
    return;
  }
  const int n = old + 1, units = (n + 15) / 16;
  const int u0 = (int)((int64_t)units * s / a.splits), u1 = (int)((int64_t)units * (s + 1) / a.splits);
  const int slot = a.slots ? a.slots[b] : b;
  auto row0 = [&](int j) -> int64_t {            // pool row of logical row j, a multiple of 16
    if (!a.pm.table) return (int64_t)slot * a.max_seq + j;
    int pg = a.pm.table[(int64_t)slot * a.pm.pages_per_slot + __builtin_amdgcn_readfirstlane(j >> a.ps_shift)];
    pg = (unsigned)pg >= (unsigned)a.pm.num_pages ? 0 : pg;
    return ((int64_t)pg << a.ps_shift) + (j & (a.pm.page_size - 1));
  };
  struct Step { f32x4 k[KC], c[4][NU]; };
  auto load = [&](Step &st, int u) {             // rows past the sequence re-read its last one; weight 0
    const int j = u * 16, last = n - 1 - j;
    const int64_t r0 = row0(j);
    const f32x4 *kp = reinterpret_cast<const f32x4 *>(a.kc + (r0 + min(ln, last)) * DH) + kq;
#pragma unroll
    for (int c = 0; c < KC; ++c) st.k[c] = __builtin_nontemporal_load(kp + c * 4);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const f32x4 *cp = reinterpret_cast<const f32x4 *>(a.cc + (r0 + min(4 * kq + r, last)) * DL) + ln;
#pragma unroll
      for (int v = 0; v < NU; ++v) st.c[r][v] = __builtin_nontemporal_load(cp + v * 16);
    }
  };
  // rows of the maps that do not exist re-read the last map; their results are not stored
  f32x4 qf[KC];
  {
    const f32x4 *qp = reinterpret_cast<const f32x4 *>(a.q + ((int64_t)b * a.nq + min(ln, a.nq - 1)) * DH) + kq;
#pragma unroll
    for (int c = 0; c < KC; ++c) qf[c] = qp[c * 4];
  }
  f32x4 acc[NU][4];
#pragma unroll
  for (int v = 0; v < NU; ++v)
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[v][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, l = 0.f;
  auto compute = [&](Step &st, int u) {
    f32x4 sc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < KC; ++c)
#pragma unroll
      for (int j = 0; j < 4; ++j) sc = __builtin_amdgcn_mfma_f32_16x16x4f32(st.k[c][j], qf[c][j], sc, 0, 0, 0);
    const int left = n - u * 16 - 4 * kq;        // valid rows of this lane's four
#pragma unroll
    for (int r = 0; r < 4; ++r) sc[r] = r < left ? sc[r] : -INFINITY;
    if (n - u * 16 < 16) {                       // 0 times the last row's infinity would be NaN
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int v = 0; v < NU; ++v) st.c[r][v] = r < left ? st.c[r][v] : f32x4{0.f, 0.f, 0.f, 0.f};
    }
    float bm = fmaxf(fmaxf(sc[0], sc[1]), fmaxf(sc[2], sc[3]));
    bm = fmaxf(bm, __shfl_xor(bm, 16, 64));
    bm = fmaxf(bm, __shfl_xor(bm, 32, 64));
    // -inf as long as all scores have overflowed to -inf
    const float mn = fmaxf(m, bm * a.scale_log2e), ref = mn > -INFINITY ? mn : 0.f;
    const float corr = __builtin_amdgcn_exp2f(m - ref);
    m = mn;
    float ps = 0.f;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      sc[r] = __builtin_amdgcn_exp2f(fmaf(sc[r], a.scale_log2e, -ref));
      ps += sc[r];
    }
    l = fmaf(l, corr, ps);                       // this lane's rows only; summed over the lane groups at the end
    if (__builtin_amdgcn_ballot_w64(corr != 1.f) != 0) {
#pragma unroll
      for (int v = 0; v < NU; ++v)
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[v][t] *= corr;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int v = 0; v < NU; ++v)
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[v][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(st.c[r][v][t], sc[r], acc[v][t], 0, 0, 0);
  };
  Step s0, s1;
  int u = u0 + wave;
  if (u < u1) load(s0, u);
  if (u + 4 < u1) load(s1, u + 4);
  while (u < u1) {
    compute(s0, u);
    if (u + 8 < u1) load(s0, u + 8);
    if ((u += 4) >= u1) break;
    compute(s1, u);
    if (u + 8 < u1) load(s1, u + 8);
    u += 4;
  }
  // merge the four waves; register r of tile (v, t) is column 64 v + 4 (4 (lane / 16) + r) + t of map lane % 16
  l += __shfl_xor(l, 16, 64);
  l += __shfl_xor(l, 32, 64);
  if (kq == 0) { sm[wave][ln] = m; sl[wave][ln] = l; }
  __syncthreads();
  float mx = sm[0][ln];
#pragma unroll
  for (int w = 1; w < 4; ++w) mx = fmaxf(mx, sm[w][ln]);
  const float ws = m > -INFINITY ? __builtin_amdgcn_exp2f(m - mx) : 0.f;
#pragma unroll
  for (int v = 0; v < NU; ++v)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      *reinterpret_cast<f32x4 *>(&lacc[wave][ln][64 * v + 4 * (4 * kq + r)]) =
          f32x4{acc[v][0][r] * ws, acc[v][1][r] * ws, acc[v][2][r] * ws, acc[v][3][r] * ws};
  __syncthreads();
  for (int i = tid; i < a.nq * (DL / 4); i += 256) {
    const int g = i / (DL / 4), col = (i % (DL / 4)) * 4;
    f32x4 v = *reinterpret_cast<const f32x4 *>(&lacc[0][g][col]);
#pragma unroll
    for (int w = 1; w < 4; ++w) v += *reinterpret_cast<const f32x4 *>(&lacc[w][g][col]);
    *reinterpret_cast<f32x4 *>(pa + g * DL + col) = v;
  }
  if (tid < a.nq) {
    float rm = sm[0][tid];
#pragma unroll
    for (int w = 1; w < 4; ++w) rm = fmaxf(rm, sm[w][tid]);
    float ls = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w)   // no maximum: a wave without rows (sum 0) or with nothing but NaN (sum NaN)
      ls = fmaf(sl[w][tid], sm[w][tid] > -INFINITY ? __builtin_amdgcn_exp2f(sm[w][tid] - rm) : 1.f, ls);
    pml[2 * tid] = rm;
    pml[2 * tid + 1] = ls;
  }
}

// ------------------------------------------------------------------------------ launches
// Columns in units of 32.
template <int BM, int BN, class Epi>
void launch_gemm_rows_f32(GemmOperands g, int cols, const Epi &epi, hipStream_t st) {
  g.tiles = (cols / BN) * ((g.M + BM - 1) / BM);
  auto launch = [&](auto kernel, int w) {
    const int smem = w * BM * (BN + 4) * (int)sizeof(float);
    if (smem > 64 * 1024) allow_dynamic_lds((const void *)kernel, smem);
    kernel<<<g.tiles + (epi.side_waves() + w - 1) / w, 64 * w, smem, st>>>(g, epi);
  };
  // two rounds of loads per wave at most: K = 1280 over 16 waves (64 rows of the paper's projection 16 us, 20 us with
  // eight waves of 64 columns), K = 256 over eight (5 us; 16 mostly idle waves 9 us), K = 64 over four
  auto launch_waves = [&](auto waves) {
    constexpr int W = decltype(waves)::value;
    if (g.K / (BN == 32 ? 8 : 16) > kRowsInFlight * W) launch(gemm_rows_f32_kernel<W, BM, BN, true, Epi>, W);
    else launch(gemm_rows_f32_kernel<W, BM, BN, false, Epi>, W);
  };
  if (g.K >= 640) launch_waves(std::integral_constant<int, 16>{});
  else if (g.K >= 192) launch_waves(std::integral_constant<int, 8>{});
  else launch_waves(std::integral_constant<int, 4>{});
}
// The smallest tile of which every CU gets at most one: a tile's time is its own loads and its matrix instructions, 4.4 us of
// them for 32 x 32 at K = 1280, and a CU without a tile is idle.  Whole calls with 32 x 32 / 32 x 16 / 16 x 16 tiles, paper's
// layer (56 column tiles of 32 in the projection, 40 in W_O): decode of 1 sequence behind 1000 rows 37.1 / 28.2 / 24.7 us, 16
// 41.3 / 33.3 / 30.2, 32 43.9 / 36.4 / 30.9 (224 tiles of 16 x 16), 48 49.8 / 42.3 / 42.4 (336; 168 of 32 x 16), 64 behind
// 2048 57.0 / 50.0 / 52.8 (448; 224); prompts of 100 tokens 44.2 / 53.1 / 49.6 (224 of 32 x 32, 448 of 32 x 16).
template <class Epi>
void launch_gemm_rows_f32(const GemmOperands &g, int cols, const Epi &epi, hipStream_t st) {
  const int64_t tiles16 = (int64_t)(cols / 16) * ((g.M + 15) / 16), tiles32 = (int64_t)(cols / 16) * ((g.M + 31) / 32);
  if (tiles16 <= 256) launch_gemm_rows_f32<16, 16>(g, cols, epi, st);
  else if (tiles32 <= 256) launch_gemm_rows_f32<32, 16>(g, cols, epi, st);
  else launch_gemm_rows_f32<32, 32>(g, cols, epi, st);
}
// Up to 256 rows the kernel that splits K inside the workgroup is the faster one (the paper's layer, whole prefill
// of one sequence: 128 tokens 50 us against 82 with 64 x 64 tiles, 256 tokens 82 against 86, 512 tokens 131 against
// 88; a decode step of 128 sequences 57 against 91).
constexpr int kRowsMax = 256;
template <class Epi>
void launch_gemm_f32(const GemmOperands &g, int cols, const Epi &epi, hipStream_t st) {
  if (g.M <= kRowsMax) launch_gemm_rows_f32(g, cols, epi, st);
  else gemm_tiles_f32_kernel<Epi><<<(cols / 64) * ((g.M + 63) / 64), 256, 0, st>>>(g, cols / 64, epi);
}

}  // namespace

// Shapes of the fp32 MFMA GEMMs: every output width in units of 64 columns (a tile lies in one of Q, K, C, gate
// and holds whole heads), contraction lengths in units of 16.
bool f32_gemms_ok(const Dims &d, int64_t M) {
  // a launch holds at most 2^32 threads, up to 1024 per 32 x 32 tile (of the output projection only for few rows)
  const int64_t nrt = M / 32 + 1, most = 1 << 22;
  if (d.dtype != GTA_F32 || nrt * (d.wtot / 32) >= most || (M <= kRowsMax && nrt * (d.H / 32) >= most)) return false;
  if (d.dh % 8 || 64 % d.dh) return false;
  return !(d.wq_w % 64 || d.wk_w % 64 || d.wc_w % 64 || d.wg_w % 64 || d.H % 64 || d.dl % 16);
}

// Latent columns of a workgroup of the attention kernel and how many such slices there are.
static int attn_slice(const Dims &d) { return d.dl % 128 == 0 ? 128 : 64; }

bool f32_attn_ok(const Dims &d, int batch, int max_len) {
  if (((int64_t)max_len / 32 + 1) * batch * d.nq * (d.dl / 64 + 1) >= (1 << 24)) return false;
  if (d.dtype != GTA_F32 || (d.dh != 32 && d.dh != 64 && d.dh != 128) || d.dl % 64) return false;
  // Many sequences of a few tokens: a workgroup costs what 32 queries cost, 5 to 7 us a round of the chip, and every latent
  // slice forms the scores again, where the shape-generic kernel has a wave per row.  MFMA / shape-generic, 400 sequences:
  // heads of 64, 5 maps, latent of 128 4 tokens 26 / 19 us, 5 26 / 33; heads of 128 (one workgroup per CU), 4 maps, latent of
  // 128 6 tokens 52 / 42, 8 53 / 64; latent of 512 (4 slices) 8 tokens 187 / 104, 13 197 / 251; 8 maps, latent of 1024 (8
  // slices) 12 tokens 774 / 493, 16 786 / 911.  Launches that the chip holds at once keep the MFMA kernel (8 x 8 tokens of
  // the last shape, 512 workgroups: 17 / 25).
  const int nslice = d.dl / attn_slice(d);
  const bool one_per_cu = d.dh + attn_slice(d) >= 256;
  const int few = std::min(12, std::max(one_per_cu ? 6 : 4, 2 * nslice));
  return !(max_len <= few && (int64_t)batch * d.nq * nslice > (one_per_cu && max_len <= 4 ? 256 : 512));
}

// one key and one latent for all maps, pages that hold whole steps of 16 rows
bool f32_decode_ok(const Dims &d, const gta_cache &cache, int batch) {
  return f32_gemms_ok(d, batch) && d.nk == 1 && d.nc == 1 && d.nq <= 16 && d.dh == 64 && d.dl == 128 &&
         tuned_decode_layout_ok(cache) && rope_angles_small(d.rope, d.rope_base);
}

template <bool FOLD>
static ProjEpi<float, float, false, FOLD> proj_epi(const Dims &d, float *q, float *k, float *c, float *g, const gta_cache *cache, const int32_t *slots) {
  ProjEpi<float, float, false, FOLD> e{};
  e.dst[0] = q; e.dst[1] = k; e.dst[2] = c; e.dst[3] = g;
  e.width[0] = d.wq_w; e.width[1] = d.wk_w; e.width[2] = d.wc_w; e.width[3] = d.wg_w;
  e.dh = d.dh; e.rope = d.rope;
  if (cache) {
    e.kcache = (float *)cache->k; e.ccache = (float *)cache->c; e.slots = slots;
    e.max_batch = cache->max_batch; e.max_seq = cache->max_seq; e.pm = page_map_of(*cache);
  }
  return e;
}

static GemmOperands proj_operands(const Dims &d, const gta_weights &w, const void *x, int M) {
  GemmOperands g{};
  g.A = (const float *)x; g.lda = d.H; g.M = M; g.K = d.H;
  const void *wm[4] = {w.wq, w.wk, w.wc, w.wg};
  const int wd[4] = {d.wq_w, d.wk_w, d.wc_w, d.wg_w};
  for (int i = 0; i < 4; ++i) { g.B[i] = (const float *)wm[i]; g.ldb[i] = wd[i]; g.seg_cols[i] = wd[i]; }
  return g;
}

// 64 x 64 tiles keep the setup launch: they find the tokens of 16 groups of columns a thread and would work out as many sines
// (toy layer, 7 x 20..82 tokens 23.4 us with it, 23.7 without).
bool f32_proj_folds(const Dims &d, int batch, int64_t M) {
  return batch <= kFoldBatch && M <= kRowsMax && rope_angles_small(d.rope, d.rope_base);
}

void launch_proj_f32(const Dims &d, const gta_weights &w, const void *x, int M, const PrefillWs &ws, const gta_cache *cache,
                     const int32_t *slots, int max_len, bool rope_by_token, const Fold &fold, hipStream_t st) {
  float *q = (float *)ws.q, *k = (float *)ws.k, *c = (float *)ws.c, *g = (float *)ws.g;
  if (fold.batch) {   // few rows (f32_proj_folds)
    auto e = proj_epi<true>(d, q, k, c, g, cache, slots);
    e.max_len = max_len;
    e.fold = fold;
    e.commit_to = view_of(cache, slots);
    for (int j = 0; d.rope && j < d.dh / 2; ++j) e.freq[j] = pow(d.rope_base, -2.0 * (double)j / (double)d.dh);
    launch_gemm_rows_f32(proj_operands(d, w, x, M), d.wtot, e, st);
    return;
  }
  auto e = proj_epi<false>(d, q, k, c, g, cache, slots);
  e.seq_id = ws.seq_id; e.pos = ws.pos; e.table = ws.rope; e.max_len = max_len; e.rope_by_token = rope_by_token;
  launch_gemm_f32(proj_operands(d, w, x, M), d.wtot, e, st);
}

void launch_decoder_f32(const Dims &d, const float *L, const void *wp, const float *gate, float *out, int M, hipStream_t st) {
  GemmOperands g{};
  g.A = L; g.lda = d.nq * d.dl; g.M = M; g.K = d.dl;
  g.B[0] = (const float *)wp; g.seg_cols[0] = d.dh;
  g.heads_per_group = d.hpq; g.a_group_stride = d.dl;
  const GateEpi<float> e{out, gate, d.wg_w, d.gate};
  if (d.dh == 64) { launch_gemm_f32(g, d.wg_w, e, st); return; }
  launch_gemm_rows_f32(g, d.wg_w, e, st);   // heads of 32: 32-column tiles
}

bool f32_decoder_ok(const Dims &d, int64_t M) { return f32_gemms_ok(d, M) && (d.dh == 64 || d.dh == 32); }

void launch_out_proj_f32(const Dims &d, const float *O, const void *wo, float *out, int M, hipStream_t st) {
  GemmOperands g{};
  g.A = O; g.lda = d.wg_w; g.M = M; g.K = d.wg_w;
  g.B[0] = (const float *)wo; g.ldb[0] = d.H; g.seg_cols[0] = d.H;
  launch_gemm_f32(g, d.H, StoreEpi<float>{out, d.H}, st);
}

void launch_attn_prefill_f32(const Dims &d, const float *q, const float *k, const float *c, const int32_t *cu, int batch,
                             int64_t total, int max_len, float *L, hipStream_t st) {
  AttnF32 a{};
  a.q = q; a.k = k; a.c = c; a.L = L; a.cu = cu; a.per_seq = (int)(total / batch); a.max_len = max_len;
  a.nq = d.nq; a.qpk = d.qpk; a.qpc = d.qpc; a.wq_w = d.wq_w; a.wk_w = d.wk_w; a.wc_w = d.wc_w; a.dl = d.dl;
  a.n_qtiles = (max_len + 31) / 32; a.batch = batch; a.scale_log2e = d.scale * 1.4426950408889634f;
  const bool wide = attn_slice(d) == 128;
  a.nslice = d.dl / attn_slice(d);
  const unsigned grid = (unsigned)a.n_qtiles * batch * d.nq * a.nslice;
  const bool pair = grid > 288 && grid <= 512;
  a.back = 255 + (int)grid;
  auto launch = [&](auto kernel, int dlw) {
    const int smem = 4 * 32 * (dlw + 4) * (int)sizeof(float);
    if (smem > 64 * 1024) allow_dynamic_lds((const void *)kernel, smem);
    kernel<<<grid, 256, smem, st>>>(a);
  };
#define GTA_ATTN_OF(DH, DLW) if (pair && DH + DLW < 256) launch(attn_prefill_f32_kernel<DH, DLW, DH + DLW < 256>, DLW); else launch(attn_prefill_f32_kernel<DH, DLW, false>, DLW)
#define GTA_ATTN(DH) if (wide) { GTA_ATTN_OF(DH, 128); } else { GTA_ATTN_OF(DH, 64); }
  if (d.dh == 32) { GTA_ATTN(32); }
  else if (d.dh == 64) { GTA_ATTN(64); }
  else { GTA_ATTN(128); }
#undef GTA_ATTN
#undef GTA_ATTN_OF
}

void launch_decode_attn_f32(const Dims &d, const float *q, const int32_t *oldlen, const gta_cache &cache, const int32_t *slots,
                            int batch, int splits, float *part, hipStream_t st) {
  DecF32 a{};
  a.q = q; a.oldlen = oldlen; a.kc = (const float *)cache.k; a.cc = (const float *)cache.c; a.slots = slots;
  a.max_seq = cache.max_seq; a.pm = page_map_of(cache);
  while (a.pm.table && (1 << a.ps_shift) < a.pm.page_size) ++a.ps_shift;
  a.nq = d.nq; a.splits = splits; a.scale_log2e = d.scale * 1.4426950408889634f;
  a.pacc = part; a.pml = part + (int64_t)batch * splits * d.nq * d.dl;
  decode_attn_f32_kernel<64, 128><<<dim3(splits, batch), 256, 0, st>>>(a);
}

// Decode step in four launches: projection (with RoPE and the append in its epilogue), split-K attention over the
// caches, tail (merge, value decoder, gate, bookkeeping), output projection.
int f32_decode(const Dims &d, const gta_weights &w, const void *x_new, int batch, const gta_cache &cache, const int32_t *slots,
               void *out, const DecodeWs &ws, hipStream_t st) {
  auto e = proj_epi<false>(d, ws.q, nullptr, nullptr, ws.g, &cache, slots);
  e.seq_lens = cache.seq_lens; e.oldlen = ws.oldlen;
  for (int j = 0; j < d.dh / 2; ++j) e.freq[j] = pow(d.rope_base, -2.0 * (double)j / (double)d.dh);
  launch_gemm_f32(proj_operands(d, w, x_new, batch), d.wtot, e, st);
  launch_decode_attn_f32(d, ws.q, ws.oldlen, cache, slots, batch, ws.splits, ws.part, st);
  float *heads = w.wo ? ws.o : (float *)out;
  if (!launch_decode_tail_f32(d, ws, batch, (const float *)w.wp, heads, cache, slots, st)) {
    tuned_decode_combine(d, ws.part, ws.oldlen, ws.splits, batch, ws.l, st);
    launch_decoder_f32(d, ws.l, w.wp, ws.g, heads, batch, st);
    launch_decode_commit(cache, slots, ws.oldlen, batch, st);
  }
  if (w.wo) launch_out_proj_f32(d, ws.o, w.wo, (float *)out, batch, st);
  return check_launch();
}

}  // namespace gta
