// bf16 GEMMs for few rows (a decode step's new tokens, short prompts) for gfx950: K split over the waves of a
// workgroup.  Up to about one 32 x 32 tile per CU gemm_rows_bf16_kernel, beyond that gemm_mid_bf16_kernel below.
//
// gemm_rows: tile of 32 rows x 32 columns; each of the W waves takes every W-th chunk of 16 k: the row operand is read
// straight into MFMA layout (16 bytes per lane), the weight chunk (16 k x 32 columns, 16 bytes per lane) passes
// through a slot of LDS that only its wave touches and comes back through the transpose read, so there is no
// barrier before the sums; the loads of U chunks are in flight at once.  The W partial tiles are summed through LDS
// in a fixed order and go to the epilogue finished: RoPE, rounding, cache rows and gate are applied here and no
// fp32 partials go through memory.  Bound: the latency of one or two rounds of loads, a launch, and how many
// workgroups pull on the weights.
#include <math.h>

#include "gta_epilogues.h"
#include "gta_lds_load.h"
#include "gta_tuned.h"

namespace gta {
namespace {

typedef __bf16 bf16;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(8))) short s16x8;
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

// weights side by side: W_Q | W_K | W_C | W_G, or one matrix
struct RowsOperands { const bf16 *A; int64_t lda; int M, K; const bf16 *B[4]; int cols[4]; int tiles; };   // tiles: of the launch (32-row tiles)

template <int W, class Epi>
__global__ __launch_bounds__(64 * W) void gemm_rows_bf16_kernel(RowsOperands g, Epi epi) {
  constexpr int U = 8, PITCH = 32 + 4, SLOT = 16 * 64;   // SLOT: bytes of a weight chunk
  extern __shared__ __attribute__((aligned(16))) char smem[];   // W x 2 chunk slots, then [W][32][PITCH] floats
  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, ln = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // consecutive workgroup ids go to different XCDs; each XCD takes a contiguous eighth of the tiles, row tiles
  // fastest: neighbouring tiles share the 128-byte lines of the weights, which should reach one L2 only
  const int id = blockIdx.x, per = g.tiles / 8, at = id < per * 8 ? (id % 8) * per + id / 8 : id;
  if (id >= g.tiles) { epi.commit((id - g.tiles) * W + wave); return; }
  const int ntm = (g.M + 31) / 32, nt = at / ntm, m0 = at % ntm * 32;
  const bool rot = epi.rotates(nt * 32);
  const RowTile ct = row_tile(nt, rot, epi.head_dim());
  int seg = 0, col = ct.col0;
  while (seg < 3 && col >= g.cols[seg]) { col -= g.cols[seg]; ++seg; }
  const int ldb = g.cols[seg];
  const bf16 *ap = g.A + (int64_t)min(m0 + ln, g.M - 1) * g.lda + h * 8;
  const bf16 *bp = g.B[seg] + (int64_t)(lane >> 2) * ldb + col + ((lane >> 1) & 1) * ct.step + (lane & 1) * 8;
  const int nch = g.K / 16;
  u32x4 a[U], b[U];
  auto load = [&](int u, int c) {
    if (c < nch) {   // wave-uniform
      a[u] = *reinterpret_cast<const u32x4 *>(ap + c * 16);
      b[u] = *reinterpret_cast<const u32x4 *>(bp + (int64_t)c * 16 * ldb);
    }
  };
  const int row = tid >> 3, c = (tid & 7) * 4, fcol = ct.col0 + (c & 15) + (c >> 4) * ct.step;   // what this thread finishes
  const bool finisher = tid < 256 && m0 + row < g.M;
  typename Epi::Early early{};
  if (finisher) early = epi.early(m0 + row, fcol, rot);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int u = 0; u < U; ++u) load(u, wave + u * W);
  __builtin_amdgcn_sched_barrier(0);
  typename Epi::Ctx ctx{};
  if (finisher) ctx = epi.prepare(early, m0 + row, fcol, rot);
  char *slot = smem + wave * 2 * SLOT;
  const int wr = (lane >> 2) * 64 + (lane & 3) * 16;
  const int rd = (h * 8 + ((lane & 15) >> 2)) * 64 + (((lane >> 4) & 1) * 16 + (lane & 3) * 4) * 2;
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  for (int c0 = wave; c0 < nch; c0 += U * W) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (c0 + u * W < nch) {
        char *s = slot + (u & 1) * SLOT;
        *reinterpret_cast<u32x4 *>(s + wr) = b[u];
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(s + rd));
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(s + rd + 4 * 64));
        const s16x8 w8 = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[u]), __builtin_bit_cast(bf16x8, w8), acc, 0, 0, 0);
        load(u, c0 + (u + U) * W);
      }
    }
  }
  __syncthreads();   // every wave is done with its slots
  float *red = reinterpret_cast<float *>(smem), *mine = red + wave * 32 * PITCH;
#pragma unroll
  for (int r = 0; r < 16; ++r) mine[(8 * (r >> 2) + 4 * h + (r & 3)) * PITCH + ln] = acc[r];
  __syncthreads();
  auto sum4 = [&](int row, int col) {
    const float *p = red + row * PITCH + col;
    f32x4 v = *reinterpret_cast<const f32x4 *>(p);
#pragma unroll
    for (int w = 1; w < W; ++w) v += *reinterpret_cast<const f32x4 *>(p + w * 32 * PITCH);
    return v;
  };
  if (!finisher) return;
  epi.store(ctx, m0 + row, sum4(row, c), [&](int off) { return sum4(row, c + (ct.pair ? (off > 0 ? 16 : -16) : off)); });
}

template <class Epi>
void launch_rows(RowsOperands g, int cols, const Epi &epi, hipStream_t st) {
  constexpr int W = 16, SMEM = W * 32 * (32 + 4) * 4;
  allow_dynamic_lds((const void *)gemm_rows_bf16_kernel<W, Epi>, SMEM);
  g.tiles = (cols / 32) * ((g.M + 31) / 32);
  gemm_rows_bf16_kernel<W, Epi><<<g.tiles + (epi.side_waves() + W - 1) / W, 64 * W, SMEM, st>>>(g, epi);
}

// ---- tiles of 64 rows -----------------------------------------------------------------------------
// Tile of 64 rows x 128 (64) columns, contraction in stages of 64; wave = 64 x 64 outputs x a quarter of every stage.
// Both operands go from memory straight into LDS (buffer_load_dwordx4 .. lds) through three stages, two steps ahead of
// their use, one barrier per step; 72 (48) KiB, so two (three) workgroups share a CU and one's barrier is filled by the
// other.  The four partial tiles are summed through LDS in a fixed order and go to the epilogue finished, four columns
// per thread: no fp32 partials in memory and no second kernel.
// LDS layout (a load fills 1 KiB in lane order, so lanes fetch the 16-byte chunk that belongs in their slot): X rows are
// 8 chunks, chunk c of row r in slot c ^ (r % 8) ^ (r / 8 % 2), so 8 (16) rows in a row read one logical chunk from
// different 16-byte columns of 128 (256) bytes; weight rows of 16 (8) chunks, chunk c of k-row k in slot c ^ 4 (k % 4)
// (c ^ 4 (k / 2 % 2)), so the four k-rows of a transpose read lie in different 64-byte columns.
// Bound: the loads (768 KiB per tile at K = 2048, of which a CU takes 64 bytes per clock) and, with one tile per CU, the
// read-MFMA chain of a step.  Measured against a split-K projection with fp32 partials in memory plus a finishing kernel
// and two-stage 64-row tiles for decoder and W_O, whole calls: 1B shape 500 tokens 60.7 -> 47.9 us, 1000 82 -> 66, 1500
// 105 -> 88; paper's layer 500 tokens 55 -> 43, 2000 84 -> 67; 8 x 128 + 1024 shape 1000 tokens 169 -> 130 us.  Four
// stages (one workgroup per CU) lose 10 to 18 % beyond one tile per CU; up to there SUB = 2 stages make a step.
struct MidOperands { RowsOperands g; int hpq; };   // hpq > 0: value decoder, one matrix [K, BN] per head and hpq heads per row operand

template <int BN_, int SUB_ = 1>
struct MidTile {
  static constexpr int SUB = SUB_, BN = BN_, BM = 64, BK = 64, KG = 4, NH = BN / 64, NW = KG * NH, NT = 64 * NW, NSTAGE = 3;
  static constexpr int X_BYTES = BM * BK * 2, STAGE = X_BYTES + BK * BN * 2;
  static constexpr int XL = X_BYTES / 1024 / NW, WL = BK * BN * 2 / 1024 / NW;   // load instructions per wave and stage
  static constexpr int PITCH = BN + 4, RED = BM * PITCH * 4;                     // a partial tile in LDS (fp32)
  static constexpr int RING = NSTAGE * SUB * STAGE, SMEM = RING > 2 * RED ? RING : 2 * RED;
};

template <int BN, int SUB, class Epi>
__global__ __launch_bounds__(MidTile<BN>::NT, SUB == 1 ? 4 : 2) void gemm_mid_bf16_kernel(MidOperands o, Epi epi) {
  typedef MidTile<BN, SUB> T;
  const RowsOperands &g = o.g;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, ln = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), nh = wave % T::NH, kg = wave / T::NH;
  const int id = blockIdx.x, per = gridDim.x / 8, at = id < per * 8 ? (id % 8) * per + id / 8 : id;
  const int ntm = (g.M + T::BM - 1) / T::BM, nt = at / ntm, m0 = at % ntm * T::BM;
  int seg = 0, col = nt * BN;
  const bf16 *A = g.A + (int64_t)m0 * g.lda, *B;
  if (o.hpq) { A += (int64_t)(nt / o.hpq) * g.K; B = g.B[0] + (int64_t)nt * g.K * BN; }
  else {
    while (seg < 3 && col >= g.cols[seg]) { col -= g.cols[seg]; ++seg; }
    B = g.B[seg] + col;
  }
  const int ldb = o.hpq ? BN : g.cols[seg];
  const int rv = min(g.M - m0, T::BM);
  // what this thread finishes: four columns of rows frow + 16 i
  const int frow = tid / (BN / 4), fc = tid % (BN / 4) * 4, fcol = nt * BN + fc;
  const bool rot = epi.rotates(nt * BN);
  typename Epi::Early early[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) early[i] = epi.early(m0 + min(frow + 16 * i, rv - 1), fcol, rot);

  unsigned xv[T::XL], wv[T::WL];
#pragma unroll
  for (int j = 0; j < T::XL; ++j) {
    const int r = (wave + T::NW * j) * 8 + (lane >> 3);
    xv[j] = (unsigned)(min(r, rv - 1) * g.lda * 2) + ((lane & 7) ^ (r & 7) ^ ((r >> 3) & 1)) * 16;
  }
#pragma unroll
  for (int j = 0; j < T::WL; ++j) {
    constexpr int CPR = BN / 8;
    const int k = (wave + T::NW * j) * (64 / CPR) + lane / CPR, sw = BN == 128 ? (k & 3) << 2 : (k & 2) << 1;
    wv[j] = (unsigned)(k * ldb * 2) + ((lane % CPR) ^ sw) * 16;
  }
  const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char *)smem;
  const u32x4 xr = buffer_of(A, (unsigned)((rv - 1) * g.lda * 2) + (unsigned)g.K * 2u);
  const char *wbase = reinterpret_cast<const char *>(B);   // of the stage that is requested next
  const unsigned wbytes = (unsigned)((T::BK - 1) * ldb * 2 + BN * 2);
  const int nk = g.K / T::BK / SUB;   // steps
  unsigned fill = 0, xs = 0;   // LDS offset and k offset of the stage that is requested next
  auto request_stage = [&] {
#pragma unroll
    for (int j = 0; j < T::XL; ++j) load_to_lds(xr, xv[j], xs, lds0 + fill + (wave + T::NW * j) * 1024);
    const u32x4 wr = buffer_of(wbase, wbytes);
#pragma unroll
    for (int j = 0; j < T::WL; ++j) load_to_lds(wr, wv[j], 0u, lds0 + fill + T::X_BYTES + (wave + T::NW * j) * 1024);
    xs += T::BK * 2;
    wbase += (int64_t)T::BK * ldb * 2;
    fill = fill == T::RING - T::STAGE ? 0u : fill + T::STAGE;
  };
  auto request = [&] {
#pragma unroll
    for (int u = 0; u < SUB; ++u) request_stage();
  };
  const int xo = ln * 128 + ((kg * 2 + h) ^ (ln & 7) ^ ((ln >> 3) & 1)) * 16;
  const int wq = (lane & 15) >> 2, sw = BN == 128 ? wq << 2 : (wq & 2) << 1;
  int wo[2];
#pragma unroll
  for (int tn = 0; tn < 2; ++tn)
    wo[tn] = T::X_BYTES + (kg * 16 + h * 8 + wq) * BN * 2 +
             ((nh * 8 + tn * 4 + ((lane >> 4) & 1) * 2 + ((lane & 3) >> 1)) ^ sw) * 16 + (lane & 1) * 8;
  f32x16 acc[2][2];
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[0][0][r] = acc[0][1][r] = acc[1][0][r] = acc[1][1][r] = 0.f;
  __builtin_amdgcn_sched_barrier(0);
  for (int t = 0; t < T::NSTAGE - 1 && t < nk; ++t) request();
  int cur = 0;
#pragma unroll 1
  for (int t = 0; t < nk; ++t) {
    if (t + T::NSTAGE - 1 <= nk) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((T::NSTAGE - 2) * SUB * (T::XL + T::WL)) : "memory");
    else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    s16x4 lo[SUB][2], hi[SUB][2];
    bf16x8 x[SUB][2];
#pragma unroll
    for (int u = 0; u < SUB; ++u) {
      const char *st = smem + cur + u * T::STAGE;
#pragma unroll
      for (int tn = 0; tn < 2; ++tn) {
        lo[u][tn] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(st + wo[tn]));
        hi[u][tn] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(st + wo[tn] + 4 * BN * 2));
        x[u][tn] = *reinterpret_cast<const bf16x8 *>(st + xo + tn * 32 * 128);
      }
    }
    cur = cur == T::RING - SUB * T::STAGE ? 0 : cur + SUB * T::STAGE;
    __builtin_amdgcn_sched_barrier(0);
    if (t + T::NSTAGE - 1 < nk) request();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < SUB; ++u)
#pragma unroll
      for (int tn = 0; tn < 2; ++tn)
#pragma unroll
        for (int tm = 0; tm < 2; ++tm) {
          const s16x8 w8 = __builtin_shufflevector(lo[u][tn], hi[u][tn], 0, 1, 2, 3, 4, 5, 6, 7);
          acc[tn][tm] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, w8), x[u][tm], acc[tn][tm], 0, 0, 0);
        }
  }
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");   // every wave is done with the stages
  float *mine = reinterpret_cast<float *>(smem + (kg >> 1) * T::RED) + ln * T::PITCH + nh * 64 + 4 * h;
  auto exchange = [&](bool add) {
#pragma unroll
    for (int tn = 0; tn < 2; ++tn)
#pragma unroll
      for (int tm = 0; tm < 2; ++tm)
#pragma unroll
        for (int rq = 0; rq < 4; ++rq) {
          f32x4 *q = reinterpret_cast<f32x4 *>(mine + tm * 32 * T::PITCH + tn * 32 + rq * 8);
          f32x4 v{acc[tn][tm][rq * 4], acc[tn][tm][rq * 4 + 1], acc[tn][tm][rq * 4 + 2], acc[tn][tm][rq * 4 + 3]};
          if (add) v += *q;
          *q = v;
        }
  };
  if (kg & 1) exchange(false);
  __syncthreads();
  if (!(kg & 1)) exchange(true);
  __builtin_amdgcn_sched_barrier(0);
  typename Epi::Ctx ctx[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) ctx[i] = epi.prepare(early[i], m0 + min(frow + 16 * i, rv - 1), fcol, rot);
  __syncthreads();
  const float *red = reinterpret_cast<const float *>(smem);
  auto sum4 = [&](int row, int c) {
    const float *q = red + row * T::PITCH + c;
    return *reinterpret_cast<const f32x4 *>(q) + *reinterpret_cast<const f32x4 *>(q + T::RED / 4);
  };
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = frow + 16 * i;
    if (row < rv) epi.store(ctx[i], m0 + row, sum4(row, fc), [&](int off) { return sum4(row, fc + off); });
  }
}

template <int BN, int SUB, class Epi>
void launch_mid_tiles(const MidOperands &o, int tiles, const Epi &epi, hipStream_t st) {
  typedef MidTile<BN, SUB> T;
  allow_dynamic_lds((const void *)gemm_mid_bf16_kernel<BN, SUB, Epi>, T::SMEM);
  gemm_mid_bf16_kernel<BN, SUB, Epi><<<tiles, T::NT, T::SMEM, st>>>(o, epi);
}
// Where no CU gets a second tile a step takes two stages, so that it has half the barriers and more loads in flight (1B shape,
// whole call of 500 tokens 43.7 -> 42.9 us, 256 39.2 -> 38.2; paper's layer 500 tokens 44.0 -> 42.8).
template <int BN, class Epi>
void launch_mid(const MidOperands &o, int cols, const Epi &epi, hipStream_t st) {
  const int tiles = (cols / BN) * ((o.g.M + 63) / 64);
  if (tiles <= 256 && o.g.K % 128 == 0) launch_mid_tiles<BN, 2>(o, tiles, epi, st);
  else launch_mid_tiles<BN, 1>(o, tiles, epi, st);
}

}  // namespace

// Widths in units of 32 (a tile lies in one of Q, K, C, gate), heads of 64 or 128.
bool rows_gemm_ok(const Dims &d) {
  return d.dtype == GTA_BF16 && (d.dh == 64 || d.dh == 128) && d.H % 32 == 0 && d.wc_w % 32 == 0;
}

// Decode step: q (rotated) and gate in fp32 to ws.q / ws.g, the new key and latent rows to the caches, oldlen.
void launch_rows_proj_decode(const Dims &d, const gta_weights &w, const void *x, int batch, const gta_cache &cache,
                             const int32_t *slots, const DecodeWs &ws, hipStream_t st) {
  RowsOperands g{(const bf16 *)x, d.H, batch, d.H, {(const bf16 *)w.wq, (const bf16 *)w.wk, (const bf16 *)w.wc, (const bf16 *)w.wg},
                 {d.wq_w, d.wk_w, d.wc_w, d.wg_w}};
  ProjEpi<float, bf16> e{};
  e.dst[0] = ws.q; e.dst[3] = ws.g;
  e.width[0] = d.wq_w; e.width[1] = d.wk_w; e.width[2] = d.wc_w; e.width[3] = d.wg_w;
  e.dh = d.dh; e.rope = d.rope;
  e.seq_lens = cache.seq_lens; e.oldlen = ws.oldlen;
  for (int j = 0; j < d.dh / 2; ++j) e.freq[j] = pow(d.rope_base, -2.0 * (double)j / (double)d.dh);
  e.kcache = (bf16 *)cache.k; e.ccache = (bf16 *)cache.c; e.slots = slots;
  e.max_batch = cache.max_batch; e.max_seq = cache.max_seq; e.pm = page_map_of(cache);
  launch_rows(g, d.wtot, e, st);
}

template <bool FOLD>
static ProjEpi<bf16, bf16, true, FOLD> prefill_epi(const Dims &d, const PrefillWs &ws, const gta_cache *cache, const int32_t *slots,
                                             int max_len, bool rope_by_token, const Fold &fold) {
  ProjEpi<bf16, bf16, true, FOLD> e{};
  void *dst[4] = {ws.q, ws.k, ws.c, ws.g};
  const int width[4] = {d.wq_w, d.wk_w, d.wc_w, d.wg_w};
  for (int i = 0; i < 4; ++i) { e.dst[i] = (bf16 *)dst[i]; e.width[i] = width[i]; }
  e.dh = d.dh; e.rope = d.rope;
  e.seq_id = ws.seq_id; e.pos = ws.pos; e.table = ws.rope; e.max_len = max_len; e.rope_by_token = rope_by_token;
  if (cache) {
    e.kcache = (bf16 *)cache->k; e.ccache = (bf16 *)cache->c; e.slots = slots;
    e.max_batch = cache->max_batch; e.max_seq = cache->max_seq; e.pm = page_map_of(*cache);
  }
  if (fold.batch) {
    e.fold = fold;
    e.commit_to = view_of(cache, slots);
    for (int j = 0; d.rope && j < d.dh / 2; ++j) e.freq[j] = pow(d.rope_base, -2.0 * (double)j / (double)d.dh);
  }
  return e;
}

// 128 columns per tile once such tiles give every CU one (paper's layer, W_O alone: 3000 tokens 83 -> 77 us at 470 tiles,
// equal at 320; with 160 and 80 tiles 64 and 128 columns are the same)
static bool wide_tiles_fill(int M, int N) { return N / 128 * ((M + 63) / 64) >= 256; }

// Measured whole calls, 32-row against 64-row tiles: 1B shape 33 tokens 28.6 / 33.4 us (224 tiles of 32 x 32), 65 38.4
// / 36.5 (336); paper's layer 128 tokens 37.2 / 40.4 (224), 256 47.2 / 44.8 (448); 8 x 128 + 1024 48 tokens 54 / 45 (448)
static bool short_rows(const Dims &d, int64_t M) { return (int64_t)(d.wtot / 32) * ((M + 31) / 32) <= 256; }

// A thread of the 64-row tiles finishes 16 rotated values and would work out as many sines behind its main loop (1B shape,
// 1000 tokens 64.4 -> 66.8 us, 1700 94 -> 104), or 8 under its first loads (500 tokens 42.9 -> 44.2, one tile per CU); they
// keep the table.  32-row tiles: paper's layer, 100 tokens 36.7 -> 33.3.
bool short_proj_folds(const Dims &d, int64_t M) { return short_rows(d, M) && rope_angles_small(d.rope, d.rope_base); }

// Prefill of few rows: q (rotated), k (rotated), latents and gate rows in bf16, key and latent rows to the caches.  Widths
// in units of 64 (heads of 128: of 128), H a multiple of 64.
void launch_short_proj(const Dims &d, const gta_weights &w, const void *x, int M, const PrefillWs &ws, const gta_cache *cache,
                       const int32_t *slots, int max_len, bool rope_by_token, const Fold &fold, hipStream_t st) {
  const RowsOperands g{(const bf16 *)x, d.H, M, d.H, {(const bf16 *)w.wq, (const bf16 *)w.wk, (const bf16 *)w.wc, (const bf16 *)w.wg},
                       {d.wq_w, d.wk_w, d.wc_w, d.wg_w}};
  const bool wide = !(d.wq_w % 128 || d.wk_w % 128 || d.wc_w % 128 || d.wg_w % 128);
  if (short_rows(d, M)) {
    launch_rows(g, d.wtot, prefill_epi<true>(d, ws, cache, slots, max_len, rope_by_token, fold), st);
    return;
  }
  const auto e = prefill_epi<false>(d, ws, cache, slots, max_len, rope_by_token, Fold{});
  if (wide && (d.dh == 128 || wide_tiles_fill(M, d.wtot))) launch_mid<128>(MidOperands{g, 0}, d.wtot, e, st);
  else launch_mid<64>(MidOperands{g, 0}, d.wtot, e, st);
}

void launch_short_decoder(const Dims &d, const void *L, const void *wp, const void *g, void *out, int M, hipStream_t st) {
  const MidOperands o{{(const bf16 *)L, (int64_t)d.nq * d.dl, M, d.dl, {(const bf16 *)wp}, {}}, d.hpq};
  const GateEpi<bf16, bf16> e{(bf16 *)out, (const bf16 *)g, d.nh * d.dh, d.gate};
  if (d.dh == 128) launch_mid<128>(o, d.nh * 128, e, st);
  else launch_mid<64>(o, d.nh * 64, e, st);
}

void launch_short_plain(const void *A, int64_t lda, int M, int N, int K, const void *B, void *C, hipStream_t st) {
  const MidOperands o{{(const bf16 *)A, lda, M, K, {(const bf16 *)B}, {N}}, 0};
  const StoreEpi<bf16> e{(bf16 *)C, N};
  if (N % 128 == 0 && wide_tiles_fill(M, N)) launch_mid<128>(o, N, e, st);
  else launch_mid<64>(o, N, e, st);
}

void launch_rows_plain(const void *A, int64_t lda, int M, int N, int K, const void *B, void *C, hipStream_t st) {
  launch_rows(RowsOperands{(const bf16 *)A, lda, M, K, {(const bf16 *)B}, {N}}, N, StoreEpi<bf16>{(bf16 *)C, N}, st);
}

}  // namespace gta
