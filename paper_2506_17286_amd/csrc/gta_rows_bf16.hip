// bf16 GEMMs for few rows (a decode step's new tokens, short prompts) for gfx950: K split over the waves of a
// workgroup.
//
// Tile of 32 rows x 32 columns; each of the W waves takes every W-th chunk of 16 k: the row operand is read
// straight into MFMA layout (16 bytes per lane), the weight chunk (16 k x 32 columns, 16 bytes per lane) passes
// through a slot of LDS that only its wave touches and comes back through the transpose read, so there is no
// barrier before the sums; the loads of U chunks are in flight at once.  The W partial tiles are summed through LDS
// in a fixed order and go to the epilogue finished: RoPE, rounding, cache rows and gate are applied here and no
// fp32 partials go through memory.  Bound: the latency of one or two rounds of loads, a launch, and how many
// workgroups pull on the weights.
#include <math.h>

#include "gta_epilogues.h"
#include "gta_tuned.h"

namespace gta {
namespace {

typedef __bf16 bf16;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(8))) short s16x8;
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

// weights side by side: W_Q | W_K | W_C | W_G, or one matrix
struct RowsOperands { const bf16 *A; int64_t lda; int M, K; const bf16 *B[4]; int cols[4]; };

template <int W, class Epi>
__global__ __launch_bounds__(64 * W) void gemm_rows_bf16_kernel(RowsOperands g, Epi epi) {
  constexpr int U = 8, PITCH = 32 + 4, SLOT = 16 * 64;   // SLOT: bytes of a weight chunk
  extern __shared__ __attribute__((aligned(16))) char smem[];   // W x 2 chunk slots, then [W][32][PITCH] floats
  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, ln = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // consecutive workgroup ids go to different XCDs; each XCD takes a contiguous eighth of the tiles, row tiles
  // fastest: neighbouring tiles share the 128-byte lines of the weights, which should reach one L2 only
  const int id = blockIdx.x, per = gridDim.x / 8, at = id < per * 8 ? (id % 8) * per + id / 8 : id;
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
void launch_rows(const RowsOperands &g, int cols, const Epi &epi, hipStream_t st) {
  constexpr int W = 16, SMEM = W * 32 * (32 + 4) * 4;
  allow_dynamic_lds((const void *)gemm_rows_bf16_kernel<W, Epi>, SMEM);
  gemm_rows_bf16_kernel<W, Epi><<<(cols / 32) * ((g.M + 31) / 32), 64 * W, SMEM, st>>>(g, epi);
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

void launch_rows_plain(const void *A, int64_t lda, int M, int N, int K, const void *B, void *C, hipStream_t st) {
  launch_rows(RowsOperands{(const bf16 *)A, lda, M, K, {(const bf16 *)B}, {N}}, N, StoreEpi<bf16>{(bf16 *)C, N}, st);
}

}  // namespace gta
