// bf16 MFMA GEMMs of the GTA pass for gfx950 (fp32 accumulation):
//   * fused input projection  [Q | K | C | gate] = X . [W_Q | W_K | W_C | W_G]   (paper Sec. 3.2)
//     with RoPE on q and k (App. B.1.1) and the cache write (App. B.1.3) in the epilogue,
//   * value decoder  O_i = (L_{q(i)} W_{P,i}) * Sigmoid(gate)                     (Sec. 3.2),
//   * plain output projection  U = O . W_O                                         (Sec. 3.3).
//
// All weights are row-major [in, out], i.e. the contraction index is the SLOW index of the weight
// operand.  The kernel therefore computes the transposed tile D'[n][m] = sum_k W[k][n] X[m][k]:
// the MFMA row operand comes from the weight tile through the LDS transpose read of gfx950
// (ds_read_b64_tr_b16: each lane receives 4 consecutive k of one n), the MFMA column operand is
// a plain 16-byte LDS read of an X row.  Each lane then owns 4 consecutive output columns of one
// output row, which makes the RoPE pairing (j, j + d_h/2) lane-local.
//
// Workgroup tile BM x BN x BK with WGM x WGN waves of 32x32x16 MFMA tiles.  The 256 x 256 x 64 tiles
// run the hand-pipelined main loop below (operands straight into LDS, four stages); their result
// is rounded to bf16, parked in LDS in output layout and written with 16-byte row-contiguous stores.
// The small tiles (split-K projection of the decode step) take the plain two-stage loop and store straight from the
// accumulator layout.  Short prefills take the kernels for few rows (short_gemm_ok).
#include <math.h>

#include <type_traits>

#include "gta_lds_load.h"
#include "gta_tuned.h"

namespace gta {
namespace {
typedef __bf16 bf16;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(8))) short s16x8;
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

template <int BM_, int BN_, int BK_, int WGM_, int WGN_>
struct GemmTile {
  static constexpr int BM = BM_, BN = BN_, BK = BK_, WGM = WGM_, WGN = WGN_;
  static constexpr int WM = BM / WGM, WN = BN / WGN, TM = WM / 32, TN = WN / 32;
  static constexpr int NT = 64 * WGM * WGN;
  static constexpr int A_PITCH = BK * 2 + 16;    // bytes per X row: 16 * odd -> conflict-free b128 reads
  static constexpr int B_PITCH = BN * 2 + 64;    // bytes per weight k-row: == 64 mod 256 for the tr reads
  static constexpr int A_BYTES = BM * A_PITCH, B_BYTES = BK * B_PITCH, STAGE = A_BYTES + B_BYTES;
  static constexpr int SMEM = 2 * STAGE;
  static_assert(WM % 32 == 0 && WN % 32 == 0 && BK % 16 == 0, "tile");
};

// acc[tn][tm][r]:  n = n_wave + tn*32 + 8*(r/4) + 4*(lane/32) + r%4,  m = m_wave + tm*32 + lane%32
template <class T>
__device__ __forceinline__ void gemm_mainloop(const bf16 *__restrict__ A, int64_t lda, int M, int m0,
                                              const bf16 *__restrict__ B, int64_t ldb, int n0, int K, char *smem,
                                              f32x16 (&acc)[T::TN][T::TM]) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wn = wave % T::WGN, wm = wave / T::WGN;
  constexpr int A_CPR = T::BK / 8, A_RPP = T::NT / A_CPR, A_PASSES = T::BM / A_RPP;
  constexpr int B_CPR = T::BN / 8, B_RPP = T::NT / B_CPR, B_PASSES = T::BK / B_RPP;
  static_assert(T::BM % A_RPP == 0 && T::BK % B_RPP == 0 && A_PASSES >= 1 && B_PASSES >= 1, "staging");
  const int a_c = tid % A_CPR, a_r = tid / A_CPR;
  const int b_c = tid % B_CPR, b_r = tid / B_CPR;
  u32x4 ra[A_PASSES], rb[B_PASSES];

  auto gload = [&](int kt) {
#pragma unroll
    for (int i = 0; i < A_PASSES; ++i) {
      const int row = min(m0 + a_r + i * A_RPP, M - 1);
      ra[i] = *reinterpret_cast<const u32x4 *>(A + (int64_t)row * lda + kt * T::BK + a_c * 8);
    }
#pragma unroll
    for (int i = 0; i < B_PASSES; ++i) {
      const int krow = kt * T::BK + b_r + i * B_RPP;
      rb[i] = *reinterpret_cast<const u32x4 *>(B + (int64_t)krow * ldb + n0 + b_c * 8);
    }
  };
  auto sstore = [&](char *st) {
#pragma unroll
    for (int i = 0; i < A_PASSES; ++i)
      *reinterpret_cast<u32x4 *>(st + (a_r + i * A_RPP) * T::A_PITCH + a_c * 16) = ra[i];
#pragma unroll
    for (int i = 0; i < B_PASSES; ++i)
      *reinterpret_cast<u32x4 *>(st + T::A_BYTES + (b_r + i * B_RPP) * T::B_PITCH + b_c * 16) = rb[i];
  };
  // per-lane constant parts of the operand addresses
  const int xoff = (wm * T::WM + (lane & 31)) * T::A_PITCH + (lane >> 5) * 16;
  const int woff = T::A_BYTES + ((lane >> 5) * 8 + ((lane & 15) >> 2)) * T::B_PITCH +
                   (wn * T::WN + ((lane >> 4) & 1) * 16 + (lane & 3) * 4) * 2;
  auto compute = [&](const char *st) {
#pragma unroll
    for (int kk = 0; kk < T::BK / 16; ++kk) {
      bf16x8 xf[T::TM];
#pragma unroll
      for (int tm = 0; tm < T::TM; ++tm)
        xf[tm] = *reinterpret_cast<const bf16x8 *>(st + xoff + tm * 32 * T::A_PITCH + kk * 32);
#pragma unroll
      for (int tn = 0; tn < T::TN; ++tn) {
        const char *wp = st + woff + kk * 16 * T::B_PITCH + tn * 64;
        s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(wp));
        s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(wp + 4 * T::B_PITCH));
        s16x8 w8 = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        bf16x8 wf = __builtin_bit_cast(bf16x8, w8);
#pragma unroll
        for (int tm = 0; tm < T::TM; ++tm)
          acc[tn][tm] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf, xf[tm], acc[tn][tm], 0, 0, 0);
      }
    }
  };

  const int nk = K / T::BK;
  gload(0);
  sstore(smem);
  __syncthreads();
  for (int kt = 0; kt < nk; ++kt) {
    char *cur = smem + (kt & 1) * T::STAGE;
    char *nxt = smem + ((kt & 1) ^ 1) * T::STAGE;
    if (kt + 1 < nk) gload(kt + 1);
    compute(cur);
    if (kt + 1 < nk) sstore(nxt);
    __syncthreads();
  }
}

// ---- software-pipelined main loop for the big tiles --------------------------------------------
// 256 x 256 tile, eight waves (two per SIMD) of 64 x 128, k-tiles of 32.  Both operand tiles go from memory straight
// into LDS (buffer_load_dwordx4 .. lds: no staging registers, no LDS writes by the waves) through four stages, so a
// k-tile is requested three tiles ahead of its use.  The loop is laid out in steps of one MFMA:
//   * the fragment reads of k-step kk+1 go out under the MFMAs of step kk (two fragment sets);
//   * the barrier of tile t sits in its first k-step, behind that step's fragment reads: every wave has then read all
//     of stage t, and (each wave having waited for its own loads) tile t+1 is complete;
//   * behind it, under the MFMAs of the second k-step, go the reads of tile t+1's first step and the wave's loads of
//     tile t+4 into the stage just left.
// LDS layout: a load instruction fills 1 KiB in lane order, so there is no padding; instead each lane fetches the
// 16-byte chunk that belongs in its slot.  X rows are 4 chunks, chunk c of row r in slot c ^ x_swz(r): any 8 (16)
// consecutive rows read one logical chunk from 8 (16) different 16-byte columns of 128 (256) bytes.  Weight rows are
// 32 chunks, chunk c of k-row k in slot c ^ 4 (k % 4): the four k-rows of a transpose read lie in different 64-byte
// columns.
// Bound: what the chip sustains on such data (1240 TFLOP/s for a large library GEMM; the projection of 112 K rows x
// 4096 x 7168 reaches 1180).  Measured against four waves of 128 x 128 that staged through registers (one wave per
// SIMD, 512 registers and spills): projection 16384 x 2048 x 3584 273 -> 252 us, 65536 x 1280 x 1792 394 -> 325,
// W_O 65536 x 1280 x 1280 251 -> 225, decoder of 16384 rows 76 -> 69.  The same loop with four waves was no faster
// than the staged one; wave priorities, the barrier's place and free scheduling changed nothing.
__device__ __forceinline__ int x_swz(int r) { return ((r >> 2) & 3) ^ (r & 2); }

struct BigLoop {
  static constexpr int BM = 256, BN = 256, BK = 32, NSTAGE = 4, X_BYTES = BM * BK * 2, STAGE = X_BYTES + BK * BN * 2;
  static constexpr int SMEM = NSTAGE * STAGE;
};

// What the last four tiles fetch instead of operands: load j (0..7) of stage `s` of this wave.
struct NoTail {
  static constexpr bool active = false;
  __device__ void load(int, int, unsigned) const {}
};

// Weight operand of a big tile: `base` points at its first k-row, rows are ld elements apart; column chunk c (8
// columns) sits chunk_bytes(c) behind the start of a row; `bytes` covers 32 rows.
struct WeightTile {
  const bf16 *base; int64_t ld; unsigned bytes;
  unsigned head_bytes;   // > 0: columns 128 .. 255 are another matrix (the next head) this far behind the first
  __device__ __forceinline__ unsigned chunk_bytes(int c) const { return head_bytes ? (c >> 4) * head_bytes + (c & 15) * 16 : c * 16; }
};
__device__ __forceinline__ WeightTile weight_tile(const bf16 *base, int64_t ld, unsigned head_bytes = 0) {
  return WeightTile{base, ld, (unsigned)(31 * ld * 2) + (head_bytes ? head_bytes + 256u : 512u), head_bytes};
}

// acc[tn][tm][r]:  n = wn*128 + tn*32 + 8*(r/4) + 4*(lane/32) + r%4,  m = wm*64 + tm*32 + lane%32, wn = wave % 2, wm = wave / 2.
// `Abase` points at row m0 of the row operand.  K a multiple of 32, at least 128.  All loads have landed on return and
// every wave has passed a barrier behind its last LDS read.
template <class G, class Tail>
__device__ __forceinline__ void gemm_mainloop_big(const bf16 *__restrict__ Abase, int64_t lda, int rows_valid, WeightTile B, int K,
                                                  char *smem, f32x16 (&acc)[G::TN][G::TM], const Tail &tail) {
  typedef BigLoop T;
  constexpr int TM = G::TM, TN = G::TN, NW = G::NT / 64, LPW = 16 / NW;   // LPW: load instructions per wave and operand
  const int lane = threadIdx.x & 63, h = lane >> 5, ln = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wn = wave % G::WGN, wm = wave / G::WGN;
  const int nk = K / T::BK;
  const int rv = min(rows_valid, T::BM);
  const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char *)smem;
  // this wave's loads of a tile: rows 32 wave + 16 j + lane/4 of X (rows past the last valid one re-read it), k-rows
  // 4 wave + 2 j + lane/32 of the weights
  unsigned xv[LPW], wv[LPW];
#pragma unroll
  for (int j = 0; j < LPW; ++j) {
    const int r = (wave * LPW + j) * 16 + (lane >> 2), k = (wave * LPW + j) * 2 + h;
    xv[j] = (unsigned)(min(r, rv - 1) * lda * 2) + ((lane & 3) ^ x_swz(lane >> 2)) * 16;
    wv[j] = (unsigned)(k * B.ld * 2) + B.chunk_bytes(ln ^ ((k & 3) << 2));
  }
  const u32x4 xr = buffer_of(Abase, (unsigned)((rv - 1) * lda * 2) + (unsigned)K * 2u);
  const int64_t wstep = (int64_t)T::BK * B.ld * 2;
  const char *wbase = reinterpret_cast<const char *>(B.base);   // of the tile that is requested next
  auto load_x = [&](int t, int j) { load_to_lds(xr, xv[j], (unsigned)(t * T::BK * 2), lds0 + (t & 3) * T::STAGE + (wave * LPW + j) * 1024); };
  auto load_w = [&](int t, int j) {
    load_to_lds(buffer_of(wbase, B.bytes), wv[j], 0u, lds0 + (t & 3) * T::STAGE + T::X_BYTES + (wave * LPW + j) * 1024);
  };
  // fragment addresses: X chunk 2 kk + h of row ln (+ 32 tm), weight rows 8 h + (lane%16)/4 (+ 16 kk, + 4)
  int xo[2], wo[TN];
  const int wr = (lane & 15) >> 2;
#pragma unroll
  for (int kk = 0; kk < 2; ++kk) xo[kk] = (wm * G::WM + ln) * 64 + (((kk * 2 + h) ^ x_swz(ln & 15)) * 16);
#pragma unroll
  for (int tn = 0; tn < TN; ++tn)
    wo[tn] = T::X_BYTES + (h * 8 + wr) * 512 + (wn * (G::WN / 8) + ((tn ^ wr) << 2) + ((lane >> 4) & 1) * 2 + ((lane & 3) >> 1)) * 16 + (lane & 1) * 8;
  struct Frags { bf16x8 x[TM]; s16x4 lo[TN], hi[TN]; };
  constexpr int NR = TM + 2 * TN, NM = TM * TN;   // fragment reads and MFMAs of a k-step
  // fragment read i, in the order the MFMAs of the step need them
  auto read_frag = [&](Frags &f, const char *st, int kk, int i) {
    if (i >= 2 && i < 2 + TM) { f.x[i - 2] = *reinterpret_cast<const bf16x8 *>(st + xo[kk] + (i - 2) * 2048); return; }
    const int w = i < 2 ? i : i - TM, tn = w / 2;
    const s16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(st + wo[tn] + kk * 8192 + (w & 1) * 2048));
    if (w & 1) f.hi[tn] = v; else f.lo[tn] = v;
  };
  // the reads of step i of NM: all of them within the first NM - 2 steps
  auto read_frags = [&](Frags &f, const char *st, int kk, int i) {
    constexpr int S = NM - 3;
#pragma unroll
    for (int r = 0; r < NR; ++r)
      if (r * S / NR == i) read_frag(f, st, kk, r);
  };
  auto mma = [&](const Frags &f, int i) {
    const int tn = i / TM, tm = i % TM;
    const s16x8 w8 = __builtin_shufflevector(f.lo[tn], f.hi[tn], 0, 1, 2, 3, 4, 5, 6, 7);
    acc[tn][tm] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, w8), f.x[tm], acc[tn][tm], 0, 0, 0);
  };
  constexpr int PER_TILE = 2 * LPW;   // loads of a wave per tile
#pragma unroll
  for (int t = 0; t < 4; ++t) {
#pragma unroll
    for (int j = 0; j < LPW; ++j) { load_x(t, j); load_w(t, j); }
    wbase += wstep;
  }
  asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(3 * PER_TILE) : "memory");
  Frags f0, f1;
#pragma unroll
  for (int i = 0; i < NR; ++i) read_frag(f0, smem, 0, i);
#pragma unroll 1
  for (int t = 0; t < nk; ++t) {
    const char *cur = smem + (t & 3) * T::STAGE, *nxt = smem + ((t + 1) & 3) * T::STAGE;
    const bool more = t + 4 < nk;
#pragma unroll
    for (int i = 0; i < NM; ++i) {
      read_frags(f1, cur, 1, i);
      mma(f0, i);
      if (i == NM - 3) {   // three tiles in flight (t+1 .. t+3); at the end there may be fewer
        if (Tail::active || t < nk - 3) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(2 * PER_TILE) : "memory");
        else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
      }
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int i = 0; i < NM; ++i) {
      read_frags(f0, nxt, 0, i);
      if (i % 2 == 1) {
        const int l = i / 2;   // NM / 2 = PER_TILE
        if (more) { if (l % 2 == 0) load_x(t + 4, l / 2); else load_w(t + 4, l / 2); }
        else if (Tail::active) tail.load(t & 3, l, lds0 + (t & 3) * T::STAGE);
      }
      mma(f1, i);
      __builtin_amdgcn_sched_barrier(0);
    }
    wbase += wstep;
  }
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

template <class T>
__device__ __forceinline__ void zero_acc(f32x16 (&acc)[T::TN][T::TM]) {
#pragma unroll
  for (int tn = 0; tn < T::TN; ++tn)
#pragma unroll
    for (int tm = 0; tm < T::TM; ++tm)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[tn][tm][r] = 0.f;
}

__device__ __forceinline__ bf16x4 pack4(float a, float b, float c, float d) {
  bf16x4 v;
  v[0] = (bf16)a; v[1] = (bf16)b; v[2] = (bf16)c; v[3] = (bf16)d;
  return v;
}

// Workgroup -> tile mapping.  Consecutive workgroup ids land on different XCDs (8 of them, each with
// its own L2), and an XCD works through its ids in order, about 32 workgroups at a time.  The tiles are
// put in one global order -- blocks of 8 row strips x 4 column tiles, row strip fastest inside a block,
// blocks column-panel by column-panel inside a band of 8 row strips, band after band -- and XCD x takes
// the x-th eighth of that order: the 32 workgroups that run together on an XCD then form one block,
// share 8 X strips and 4 weight strips (every operand slice fetched into the L2 is used 4 or 8 times),
// whatever the numbers of row strips and column tiles are.  Edge blocks are simply smaller.
__device__ __forceinline__ void tile_of_block(int ntn, int ntm, int &mt, int &nt) {
  constexpr int RB = 8, PW = 4;
  const int nblk = ntn * ntm, id = blockIdx.x, per = nblk / 8;
  const int pos = id < per * 8 ? (id % 8) * per + id / 8 : id;   // the last nblk % 8 tiles keep their place
  const int band = pos / (RB * ntn);
  int rem = pos - band * RB * ntn;
  const int h = min(RB, ntm - band * RB);      // row strips of this band
  const int panel = rem / (h * PW);
  rem -= panel * h * PW;
  mt = band * RB + rem % h;
  nt = panel * PW + rem / h;
}

// ---- epilogue of the 256 x 256 tile through LDS -------------------------------------------------
// In the accumulator layout a lane owns 4 consecutive columns of one row, so direct stores would be
// 8 bytes wide and scattered over 32 rows per instruction.  The tile is therefore rounded to bf16,
// parked in LDS in output layout and written out with 16-byte stores in which 32 consecutive lanes cover one
// 512-byte row segment.  Chunk c (8 columns) of row r sits in slot c ^ (r % 16) of its row, which spreads the rows
// of an access in accumulator layout over the banks.
__device__ __forceinline__ int out_chunk(int row, int c) { return row * 512 + ((c ^ (row & 15)) << 4); }
constexpr int kOutBytes = 256 * 512;

template <class T>
__device__ __forceinline__ int out_lds_offset(int tm, int tn, int rq) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wn = wave % T::WGN, wm = wave / T::WGN;
  return out_chunk(wm * T::WM + tm * 32 + (lane & 31), (wn * T::WN + tn * 32) / 8 + rq) + (lane >> 5) * 8;
}

template <class T>
__device__ __forceinline__ void tile_to_lds(const f32x16 (&acc)[T::TN][T::TM], char *smem) {
  static_assert(T::BM == 256 && T::BN == 256, "epilogue staging");
#pragma unroll
  for (int tm = 0; tm < T::TM; ++tm)
#pragma unroll
    for (int tn = 0; tn < T::TN; ++tn)
#pragma unroll
      for (int rq = 0; rq < 4; ++rq)
        *reinterpret_cast<bf16x4 *>(smem + out_lds_offset<T>(tm, tn, rq)) =
            pack4(acc[tn][tm][rq * 4], acc[tn][tm][rq * 4 + 1], acc[tn][tm][rq * 4 + 2], acc[tn][tm][rq * 4 + 3]);
}

// calls f(row, chunk, value) for every 16-byte chunk (8 columns) of the staged tile: 32 lanes per row
template <int NT = 256, class F>
__device__ __forceinline__ void for_each_out_chunk(const char *smem, F f) {
  constexpr int RPP = NT / 32;   // rows per pass
  const int r0 = threadIdx.x >> 5, ch = threadIdx.x & 31;
#pragma unroll 4
  for (int it = 0; it < 256 / RPP; ++it) {
    const int r = it * RPP + r0;
    f(r, ch, *reinterpret_cast<const u32x4 *>(smem + out_chunk(r, ch)));
  }
}

// ------------------------------------------------------------------------------ projection
constexpr int kHeadDim = 128;   // the RoPE epilogue is compiled for d_h = 128

struct ProjArgs {
  const bf16 *x; int64_t lda; int M, K;
  const bf16 *w[4]; int width[4];     // W_Q, W_K, W_C, W_G and their output widths
  bf16 *dst[4];                       // Q, K, C, gate pre-activation  [M, width]
  const int32_t *seq_id, *pos;        // per packed token
  const float2 *rope; int max_len;    // (cos, sin)[pos][j], NULL = no RoPE
  int rope_by_token;                  // chunked prefill: the table has one row per packed token instead
  int dh;
  bf16 *kcache, *ccache; const int32_t *slots; int max_batch, max_seq;   // kcache NULL = no cache write
  PageMap pm;                                                             // contiguous or block-table rows
};

template <class T>
__global__ __launch_bounds__(T::NT) void proj_gemm_kernel(ProjArgs a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int wtot = a.width[0] + a.width[1] + a.width[2] + a.width[3];
  int mt, nt;
  tile_of_block(wtot / T::BN, (a.M + T::BM - 1) / T::BM, mt, nt);
  int n_glob = nt * T::BN, seg = 0;
  while (n_glob >= a.width[seg]) { n_glob -= a.width[seg]; ++seg; }   // widths are multiples of BN
  const int m0 = mt * T::BM;
  f32x16 acc[T::TN][T::TM];
  zero_acc<T>(acc);
  // positions of this lane's rows: asked for before the main loop (a tile of Q or K rotates by them right
  // after it: 0.8 us of load latency per tile otherwise), not at all by the big tiles that do not rotate
  const bool rotate = a.rope != nullptr && seg < 2;
  constexpr bool kBig = T::BM == 256 && T::BN == 256;
  int pos_of[T::TM];
  if (rotate || !kBig) {
#pragma unroll
    for (int tm = 0; tm < T::TM; ++tm)
      pos_of[tm] = a.pos[min(m0 + (int)(threadIdx.x >> 6) / T::WGN * T::WM + tm * 32 + (int)(threadIdx.x & 31), a.M - 1)];
  }
  if constexpr (kBig) {
    gemm_mainloop_big<T>(a.x + (int64_t)m0 * a.lda, a.lda, a.M - m0, weight_tile(a.w[seg] + n_glob, a.width[seg]), a.K, smem, acc,
                      NoTail{});
  } else {
    gemm_mainloop<T>(a.x, a.lda, a.M, m0, a.w[seg], a.width[seg], n_glob, a.K, smem, acc);
  }

  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wn = wave % T::WGN, wm = wave / T::WGN;
  const int nw = n_glob + wn * T::WN;            // first column of this wave inside its segment
  const int half = a.dh / 2;
  bf16 *cache = seg == 1 ? a.kcache : (seg == 2 ? a.ccache : nullptr);
  const int width = a.width[seg];
  if constexpr (kBig) {
    if (rotate) {
      // wave tile = one head: column j pairs with j + d_h/2.  16 groups of 4 pairs per lane (2 row blocks x
      // 2 column blocks x 4 register quads); the table values of a group are asked for two groups ahead of
      // their use (one after the other, every group would wait out a whole memory round trip: 9 us per tile with
      // four row blocks)
      constexpr int tiles_half = kHeadDim / 64;
      static_assert(T::TN == 2 * tiles_half, "a wave tile of the rotating segments is one head wide");
      constexpr int G = T::TM * tiles_half * 4, AHEAD = 2;
      bool rot[T::TM];
      const float2 *trow[T::TM];
#pragma unroll
      for (int tm = 0; tm < T::TM; ++tm) {
        const int m = m0 + wm * T::WM + tm * 32 + (lane & 31), p = pos_of[tm];
        rot[tm] = m < a.M && (a.rope_by_token || p < a.max_len);
        // rows that do not rotate read row 0 of the table and keep their values
        trow[tm] = a.rope + (int64_t)(rot[tm] ? (a.rope_by_token ? m : p) : 0) * half + (lane >> 5) * 4;
      }
      float4 tv[AHEAD + 1][2];
      auto ask = [&](int g) {
        const int tm = g / (tiles_half * 4), tn = (g / 4) % tiles_half, rq = g % 4;
        const float4 *tp = reinterpret_cast<const float4 *>(trow[tm] + tn * 32 + rq * 8);
        tv[g % (AHEAD + 1)][0] = tp[0]; tv[g % (AHEAD + 1)][1] = tp[1];
      };
#pragma unroll
      for (int g = 0; g < AHEAD; ++g) ask(g);
#pragma unroll
      for (int g = 0; g < G; ++g) {
        if (g + AHEAD < G) ask(g + AHEAD);
        const int tm = g / (tiles_half * 4), tn = (g / 4) % tiles_half, rq = g % 4, tn_hi = tn + tiles_half;
        const float4 t0 = tv[g % (AHEAD + 1)][0], t1 = tv[g % (AHEAD + 1)][1];
        const float cs[4] = {t0.x, t0.z, t1.x, t1.z}, sn[4] = {t0.y, t0.w, t1.y, t1.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float lo = acc[tn][tm][rq * 4 + i], hi = acc[tn_hi][tm][rq * 4 + i];
          acc[tn][tm][rq * 4 + i] = rot[tm] ? lo * cs[i] - hi * sn[i] : lo;
          acc[tn_hi][tm][rq * 4 + i] = rot[tm] ? hi * cs[i] + lo * sn[i] : hi;
        }
      }
    }
  }
  if constexpr (!kBig)
#pragma unroll
  for (int tm = 0; tm < T::TM; ++tm) {
    const int m = m0 + wm * T::WM + tm * 32 + (lane & 31);
    if (m >= a.M) continue;
    const int p = pos_of[tm];
    const int rrow = a.rope_by_token ? m : p;   // RoPE table row
    if (rotate && (a.rope_by_token || p < a.max_len)) {
      // wave tile spans whole heads (WN % d_h == 0); pair column j with j + d_h/2 of the same head
      constexpr int tiles_half = kHeadDim / 64, tiles_head = kHeadDim / 32;
#pragma unroll
      for (int tn = 0; tn < T::TN; ++tn) {
        if ((tn % tiles_head) >= tiles_half) continue;
        const int tn_hi = tn + tiles_half;
        if (tn_hi >= T::TN) continue;
#pragma unroll
        for (int rq = 0; rq < 4; ++rq) {
          const int j = (tn % tiles_head) * 32 + rq * 8 + (lane >> 5) * 4;
          const float4 *tp = reinterpret_cast<const float4 *>(a.rope + (int64_t)rrow * half + j);
          const float4 t0 = tp[0], t1 = tp[1];
          const float cs[4] = {t0.x, t0.z, t1.x, t1.z}, sn[4] = {t0.y, t0.w, t1.y, t1.w};
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float lo = acc[tn][tm][rq * 4 + i], hi = acc[tn_hi][tm][rq * 4 + i];
            acc[tn][tm][rq * 4 + i] = lo * cs[i] - hi * sn[i];
            acc[tn_hi][tm][rq * 4 + i] = hi * cs[i] + lo * sn[i];
          }
        }
      }
    }
    bf16 *drow = a.dst[seg] + (int64_t)m * width + nw;
    bf16 *crow = nullptr;
    if (cache) {
      const int b = a.seq_id[m];
      const int slot = a.slots ? a.slots[b] : b;
      if (slot >= 0 && slot < a.max_batch && p >= 0 && p < a.max_seq) {
        const int64_t cr = cache_row(a.pm, a.max_seq, slot, p);
        if (cr >= 0) crow = cache + cr * width + nw;
      }
    }
#pragma unroll
    for (int tn = 0; tn < T::TN; ++tn)
#pragma unroll
      for (int rq = 0; rq < 4; ++rq) {
        const int n = tn * 32 + rq * 8 + (lane >> 5) * 4;
        const bf16x4 v = pack4(acc[tn][tm][rq * 4], acc[tn][tm][rq * 4 + 1], acc[tn][tm][rq * 4 + 2], acc[tn][tm][rq * 4 + 3]);
        *reinterpret_cast<bf16x4 *>(drow + n) = v;
        if (crow) *reinterpret_cast<bf16x4 *>(crow + n) = v;
      }
  }
  if constexpr (kBig) {
    tile_to_lds<T>(acc, smem);
    // cache row of every tile row (or -1), looked up once and shared through LDS
    int64_t *crow_of = reinterpret_cast<int64_t *>(smem + kOutBytes);
    if (cache && threadIdx.x < 256) {
      const int m = m0 + (int)threadIdx.x;
      int64_t cr = -1;
      if (m < a.M) {
        const int p = a.pos[m], b = a.seq_id[m];
        const int slot = a.slots ? a.slots[b] : b;
        if (slot >= 0 && slot < a.max_batch && p >= 0 && p < a.max_seq) cr = cache_row(a.pm, a.max_seq, slot, p);
      }
      crow_of[threadIdx.x] = cr;
    }
    __syncthreads();
    bf16 *dst = a.dst[seg] + n_glob;
    for_each_out_chunk<T::NT>(smem, [&](int r, int ch, u32x4 v) {
      const int m = m0 + r;
      if (m >= a.M) return;
      *reinterpret_cast<u32x4 *>(dst + (int64_t)m * width + ch * 8) = v;
      if (cache) {
        const int64_t cr = crow_of[r];
        if (cr >= 0) *reinterpret_cast<u32x4 *>(cache + cr * width + n_glob + ch * 8) = v;
      }
    });
  }
}

// ---- projection against packed weights -----------------------------------------------------------
// The four weight matrices are first copied side by side into one [H, Wtot] matrix, so that a
// 256-column tile may straddle Q | K | C | gate: this serves output widths that are multiples of 64
// but not of 256 (heads of 64, a single shared key).  Columns are routed to their outputs per
// 64-column group for RoPE (a head never straddles a group) and per 16-byte chunk for the stores.
// The packed row is padded with zero columns to a multiple of 256 (wpad); the last tile computes
// them and stores nothing for them.
__global__ void pack_weights_kernel(ProjArgs a, int wtot, int wpad, bf16 *dst) {
  const int cpr = wpad / 8;   // 16-byte chunks per packed row
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i >= (int64_t)a.K * cpr) return;
  const int k = (int)(i / cpr);
  int col = (int)(i % cpr) * 8, seg = 0;
  u32x4 v = {0u, 0u, 0u, 0u};
  if (col < wtot) {
    while (col >= a.width[seg]) { col -= a.width[seg]; ++seg; }
    v = *reinterpret_cast<const u32x4 *>(a.w[seg] + (int64_t)k * a.width[seg] + col);
  }
  *reinterpret_cast<u32x4 *>(dst + i * 8) = v;
}

template <class T, int DH>
__global__ __launch_bounds__(T::NT) void proj_packed_kernel(ProjArgs a, const bf16 *wpack, int wpad) {
  static_assert(T::BM == 256 && T::BN == 256 && T::WN == 128 && (DH == 64 || DH == 128), "tile");
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int b1 = a.width[0], b2 = b1 + a.width[1], b3 = b2 + a.width[2], wtot = b3 + a.width[3];
  int mt, nt;
  tile_of_block(wpad / T::BN, (a.M + T::BM - 1) / T::BM, mt, nt);
  const int m0 = mt * T::BM, n0 = nt * T::BN;
  f32x16 acc[T::TN][T::TM];
  zero_acc<T>(acc);
  {
    gemm_mainloop_big<T>(a.x + (int64_t)m0 * a.lda, a.lda, a.M - m0, weight_tile(wpack + n0, wpad), a.K, smem, acc, NoTail{});
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wn = wave % T::WGN, wm = wave / T::WGN;
  if (a.rope && n0 < b2) {   // the tile holds q or k columns
    constexpr int half = DH / 2, tiles_half = DH / 64, tiles_head = DH / 32;
#pragma unroll
    for (int tm = 0; tm < T::TM; ++tm) {
      const int m = m0 + wm * T::WM + tm * 32 + (lane & 31);
      const int p = a.rope_by_token ? min(m, a.M - 1) : max(min(a.pos[min(m, a.M - 1)], a.max_len - 1), 0);   // RoPE table row
#pragma unroll
      for (int tn = 0; tn < T::TN; ++tn) {
        if ((tn % tiles_head) >= tiles_half) continue;
        const int tn_hi = tn + tiles_half;
        if (tn_hi >= T::TN) continue;
        // latent and gate columns of a straddling tile take the identity rotation (no branch: the
        // accumulators stay where they are)
        const bool rot = n0 + wn * T::WN + tn * 32 < b2;
#pragma unroll
        for (int rq = 0; rq < 4; ++rq) {
          const int j = (tn % tiles_head) * 32 + rq * 8 + (lane >> 5) * 4;
          const float4 *tp = reinterpret_cast<const float4 *>(a.rope + (int64_t)p * half + j);
          const float4 t0 = tp[0], t1 = tp[1];
          const float cs[4] = {t0.x, t0.z, t1.x, t1.z}, sn[4] = {t0.y, t0.w, t1.y, t1.w};
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float c = rot ? cs[i] : 1.f, sv = rot ? sn[i] : 0.f;
            const float lo = acc[tn][tm][rq * 4 + i], hi = acc[tn_hi][tm][rq * 4 + i];
            acc[tn][tm][rq * 4 + i] = lo * c - hi * sv;
            acc[tn_hi][tm][rq * 4 + i] = hi * c + lo * sv;
          }
        }
      }
    }
  }
  tile_to_lds<T>(acc, smem);
  int64_t *crow_of = reinterpret_cast<int64_t *>(smem + kOutBytes);
  if (a.kcache && threadIdx.x < 256) {
    const int m = m0 + (int)threadIdx.x;
    int64_t cr = -1;
    if (m < a.M) {
      const int p = a.pos[m], b = a.seq_id[m];
      const int slot = a.slots ? a.slots[b] : b;
      if (slot >= 0 && slot < a.max_batch && p >= 0 && p < a.max_seq) cr = cache_row(a.pm, a.max_seq, slot, p);
    }
    crow_of[threadIdx.x] = cr;
  }
  __syncthreads();
  // a thread stores the same 16-byte chunk column of every row: its destination is fixed
  const int gcol = n0 + (threadIdx.x & 31) * 8;
  if (gcol >= wtot) return;        // zero padding of the packed row; no barrier follows
  const int seg = (gcol >= b1) + (gcol >= b2) + (gcol >= b3);
  const int lcol = gcol - (seg == 0 ? 0 : seg == 1 ? b1 : seg == 2 ? b2 : b3);
  const int width = a.width[seg];
  bf16 *dst = a.dst[seg] + lcol;
  bf16 *cache = !a.kcache ? nullptr : seg == 1 ? a.kcache + lcol : seg == 2 ? a.ccache + lcol : nullptr;
  for_each_out_chunk<T::NT>(smem, [&](int r, int, u32x4 v) {
    const int m = m0 + r;
    if (m >= a.M) return;
    *reinterpret_cast<u32x4 *>(dst + (int64_t)m * width) = v;
    if (cache) {
      const int64_t cr = crow_of[r];
      if (cr >= 0) *reinterpret_cast<u32x4 *>(cache + cr * width) = v;
    }
  });
}

// ------------------------------------------------------------------------------ value decoder
struct DecoderArgs {
  const bf16 *L; int64_t ldl; int M;          // [M, n_q*d_l] normalised group outputs
  const bf16 *wp; int dl, dh, hpq, nh;        // [n_h, d_l, d_h]
  const bf16 *g; int gate;                    // [M, n_h*d_h] gate pre-activation
  bf16 *out;                                  // [M, n_h*d_h]
};

template <class T>
__global__ __launch_bounds__(T::NT) void decoder_gemm_kernel(DecoderArgs a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int tiles_per_head = a.dh / T::BN;     // BN divides d_h
  int mt, nt;
  tile_of_block(a.nh * tiles_per_head, (a.M + T::BM - 1) / T::BM, mt, nt);
  const int head = nt / tiles_per_head, n_in_head = (nt % tiles_per_head) * T::BN;
  const int m0 = mt * T::BM;
  f32x16 acc[T::TN][T::TM];
  zero_acc<T>(acc);
  gemm_mainloop<T>(a.L + (head / a.hpq) * a.dl, a.ldl, a.M, m0, a.wp + (int64_t)head * a.dl * a.dh, a.dh, n_in_head,
                   a.dl, smem, acc);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wn = wave % T::WGN, wm = wave / T::WGN;
  const int64_t ldo = (int64_t)a.nh * a.dh;
  const int col0 = head * a.dh + n_in_head + wn * T::WN;
#pragma unroll
  for (int tm = 0; tm < T::TM; ++tm) {
    const int m = m0 + wm * T::WM + tm * 32 + (lane & 31);
    if (m >= a.M) continue;
#pragma unroll
    for (int tn = 0; tn < T::TN; ++tn)
#pragma unroll
      for (int rq = 0; rq < 4; ++rq) {
        const int64_t o = (int64_t)m * ldo + col0 + tn * 32 + rq * 8 + (lane >> 5) * 4;
        float v[4] = {acc[tn][tm][rq * 4], acc[tn][tm][rq * 4 + 1], acc[tn][tm][rq * 4 + 2], acc[tn][tm][rq * 4 + 3]};
        if (a.gate) {
          const bf16x4 gz = *reinterpret_cast<const bf16x4 *>(a.g + o);
#pragma unroll
          for (int i = 0; i < 4; ++i)
            v[i] *= a.gate == kGateSigmoid ? 1.0f / (1.0f + __expf(-(float)gz[i])) : gate_factor(a.gate, (float)gz[i]);
        }
        *reinterpret_cast<bf16x4 *>(a.out + o) = pack4(v[0], v[1], v[2], v[3]);
      }
  }
}

// The decoder's gate tile (256 rows x 512 bytes) fills the four stages as the last four k-tiles leave them, in output
// layout: stage s takes rows 64 s .. 64 s + 63, two per load (rows past the end of the matrix re-read the last valid
// one).
template <int NW>
struct GateTail {
  static constexpr bool active = true;
  u32x4 rsrc; unsigned ld_bytes; int last;   // last valid row of the tile
  __device__ __forceinline__ void load(int s, int j, unsigned lds) const {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), r = (wave * (32 / NW) + j) * 2 + (lane >> 5);
    load_to_lds(rsrc, (unsigned)min(s * 64 + r, last) * ld_bytes + ((lane & 31) ^ (r & 15)) * 16, 0u, lds + (wave * (32 / NW) + j) * 1024);
  }
};

// Two heads of one map group per 256-wide tile (they share the row operand L_g), pipelined main
// loop.  The gate is applied to the fp32 accumulators: the gate tile is fetched into LDS in output layout, every
// lane reads the pre-activations of its own elements from there and puts the gated, rounded result back in the
// same place.
template <class T, bool GATE>
__global__ __launch_bounds__(T::NT) void decoder_pair_kernel(DecoderArgs a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  int mt, nt;
  tile_of_block(a.nh / 2, (a.M + T::BM - 1) / T::BM, mt, nt);
  const int head = nt * 2, m0 = mt * T::BM;
  f32x16 acc[T::TN][T::TM];
  zero_acc<T>(acc);
  const int64_t ldo = (int64_t)a.nh * a.dh;
  const int col0 = head * a.dh;
  const int rv = min(a.M - m0, T::BM);
  {
    const bf16 *Ab = a.L + (int64_t)m0 * a.ldl + (head / a.hpq) * a.dl;
    const WeightTile wt = weight_tile(a.wp + (int64_t)head * a.dl * a.dh, a.dh, (unsigned)(a.dl * a.dh * 2));
    if constexpr (GATE) {
      const GateTail<T::NT / 64> gate{buffer_of(a.g + (int64_t)m0 * ldo + col0, (unsigned)((rv - 1) * ldo * 2) + 512u), (unsigned)(ldo * 2), rv - 1};
      gemm_mainloop_big<T>(Ab, a.ldl, rv, wt, a.dl, smem, acc, gate);
    } else {
      gemm_mainloop_big<T>(Ab, a.ldl, rv, wt, a.dl, smem, acc, NoTail{});
    }
  }
  // one row block (tm) at a time: all 16 gate reads of the block are issued before the first is used
  // the Sigmoid of the method takes the short path; the other nonlinearities a general one
  auto gate_rows = [&](auto sig_tag) {
    constexpr bool SIG = decltype(sig_tag)::value;
  #pragma unroll
    for (int tm = 0; tm < T::TM; ++tm) {
      bf16x4 gz[T::TN][4];
      if constexpr (GATE) {
  #pragma unroll
        for (int tn = 0; tn < T::TN; ++tn)
  #pragma unroll
          for (int rq = 0; rq < 4; ++rq) gz[tn][rq] = *reinterpret_cast<const bf16x4 *>(smem + out_lds_offset<T>(tm, tn, rq));
      }
  #pragma unroll
      for (int tn = 0; tn < T::TN; ++tn)
  #pragma unroll
        for (int rq = 0; rq < 4; ++rq) {
          float v[4] = {acc[tn][tm][rq * 4], acc[tn][tm][rq * 4 + 1], acc[tn][tm][rq * 4 + 2], acc[tn][tm][rq * 4 + 3]};
          if constexpr (GATE) {
  #pragma unroll
            for (int i = 0; i < 4; ++i)
              v[i] *= SIG ? __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * (float)gz[tn][rq][i]))
                          : gate_factor(a.gate, (float)gz[tn][rq][i]);
          }
          *reinterpret_cast<bf16x4 *>(smem + out_lds_offset<T>(tm, tn, rq)) = pack4(v[0], v[1], v[2], v[3]);
        }
    }
  };
  if (!GATE || a.gate == kGateSigmoid) gate_rows(std::true_type{});
  else gate_rows(std::false_type{});
  __syncthreads();
  for_each_out_chunk<T::NT>(smem, [&](int r, int ch, u32x4 v) {
    if (m0 + r < a.M) *reinterpret_cast<u32x4 *>(a.out + (int64_t)(m0 + r) * ldo + col0 + ch * 8) = v;
  });
}

// All 256 / d_h heads of one 256-wide tile share the row operand L_g (they lie in one map group);
// short contraction (d_l of 64 .. 192, or any multiple of 64): plain main loop.  The gate tile is
// fetched with coalesced 16-byte loads before the main loop starts and applied as above.
template <class T, bool GATE>
__global__ __launch_bounds__(T::NT) void decoder_multi_kernel(DecoderArgs a) {
  static_assert(T::BM == 256 && T::BN == 256 && T::NT == 256 && T::SMEM >= kOutBytes, "tile");
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int hpt = T::BN / a.dh;   // heads per tile
  int mt, nt;
  tile_of_block(a.nh / hpt, (a.M + T::BM - 1) / T::BM, mt, nt);
  const int head = nt * hpt, m0 = mt * T::BM;
  f32x16 acc[T::TN][T::TM];
  zero_acc<T>(acc);
  const int64_t ldo = (int64_t)a.nh * a.dh;
  const int col0 = head * a.dh;
  const int r0 = threadIdx.x >> 5, ch = threadIdx.x & 31;
  u32x4 gt[32];
  if constexpr (GATE) {
    const bf16 *gp = a.g + col0 + ch * 8;
#pragma unroll
    for (int it = 0; it < 32; ++it)
      gt[it] = *reinterpret_cast<const u32x4 *>(gp + (int64_t)min(m0 + it * 8 + r0, a.M - 1) * ldo);
  }
  {
    // column chunk -> head of the tile: the loop adds (chunk column) to the pointer it is given
    const int col = (threadIdx.x % (T::BN / 8)) * 8;
    const bf16 *Bt = a.wp + (int64_t)head * a.dl * a.dh + (int64_t)(col / a.dh) * a.dl * a.dh + (col % a.dh) - col;
    gemm_mainloop<T>(a.L + (head / a.hpq) * a.dl, a.ldl, a.M, m0, Bt, a.dh, 0, a.dl, smem, acc);
  }
  if constexpr (GATE) {
#pragma unroll
    for (int it = 0; it < 32; ++it) *reinterpret_cast<u32x4 *>(smem + out_chunk(it * 8 + r0, ch)) = gt[it];
    __syncthreads();
  }
  // the Sigmoid of the method takes the short path; the other nonlinearities a general one
  auto gate_rows = [&](auto sig_tag) {
    constexpr bool SIG = decltype(sig_tag)::value;
  #pragma unroll
    for (int tm = 0; tm < T::TM; ++tm) {
      bf16x4 gz[T::TN][4];
      if constexpr (GATE) {
  #pragma unroll
        for (int tn = 0; tn < T::TN; ++tn)
  #pragma unroll
          for (int rq = 0; rq < 4; ++rq) gz[tn][rq] = *reinterpret_cast<const bf16x4 *>(smem + out_lds_offset<T>(tm, tn, rq));
      }
  #pragma unroll
      for (int tn = 0; tn < T::TN; ++tn)
  #pragma unroll
        for (int rq = 0; rq < 4; ++rq) {
          float v[4] = {acc[tn][tm][rq * 4], acc[tn][tm][rq * 4 + 1], acc[tn][tm][rq * 4 + 2], acc[tn][tm][rq * 4 + 3]};
          if constexpr (GATE) {
  #pragma unroll
            for (int i = 0; i < 4; ++i)
              v[i] *= SIG ? __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * (float)gz[tn][rq][i]))
                          : gate_factor(a.gate, (float)gz[tn][rq][i]);
          }
          *reinterpret_cast<bf16x4 *>(smem + out_lds_offset<T>(tm, tn, rq)) = pack4(v[0], v[1], v[2], v[3]);
        }
    }
  };
  if (!GATE || a.gate == kGateSigmoid) gate_rows(std::true_type{});
  else gate_rows(std::false_type{});
  __syncthreads();
  for_each_out_chunk<T::NT>(smem, [&](int r, int ch, u32x4 v) {
    if (m0 + r < a.M) *reinterpret_cast<u32x4 *>(a.out + (int64_t)(m0 + r) * ldo + col0 + ch * 8) = v;
  });
}

// ------------------------------------------------------------------------------ plain GEMM
struct PlainArgs { const bf16 *A; int64_t lda; int M, N, K; const bf16 *B; bf16 *C; };

template <class T>
__global__ __launch_bounds__(T::NT) void plain_gemm_kernel(PlainArgs a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  int mt, nt;
  tile_of_block(a.N / T::BN, (a.M + T::BM - 1) / T::BM, mt, nt);
  const int m0 = mt * T::BM, n0 = nt * T::BN;
  f32x16 acc[T::TN][T::TM];
  zero_acc<T>(acc);
  if constexpr (T::BM == 256 && T::BN == 256) {
    gemm_mainloop_big<T>(a.A + (int64_t)m0 * a.lda, a.lda, a.M - m0, weight_tile(a.B + n0, a.N), a.K, smem, acc, NoTail{});
  } else {
    gemm_mainloop<T>(a.A, a.lda, a.M, m0, a.B, a.N, n0, a.K, smem, acc);
  }
  if constexpr (T::BM == 256 && T::BN == 256) {
    tile_to_lds<T>(acc, smem);
    __syncthreads();
    for_each_out_chunk<T::NT>(smem, [&](int r, int ch, u32x4 v) {
      if (m0 + r < a.M) *reinterpret_cast<u32x4 *>(a.C + (int64_t)(m0 + r) * a.N + n0 + ch * 8) = v;
    });
    return;
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wn = wave % T::WGN, wm = wave / T::WGN;
#pragma unroll
  for (int tm = 0; tm < T::TM; ++tm) {
    const int m = m0 + wm * T::WM + tm * 32 + (lane & 31);
    if (m >= a.M) continue;
#pragma unroll
    for (int tn = 0; tn < T::TN; ++tn)
#pragma unroll
      for (int rq = 0; rq < 4; ++rq) {
        const int n = n0 + wn * T::WN + tn * 32 + rq * 8 + (lane >> 5) * 4;
        *reinterpret_cast<bf16x4 *>(a.C + (int64_t)m * a.N + n) =
            pack4(acc[tn][tm][rq * 4], acc[tn][tm][rq * 4 + 1], acc[tn][tm][rq * 4 + 2], acc[tn][tm][rq * 4 + 3]);
      }
  }
}

// ------------------------------------------------------------------------------ decode projection
// Few rows (one new token per sequence) against all four weight matrices: weight-streaming bound.
// Split-K over H so that several hundred workgroups pull on HBM at once; every (k-split, n-tile)
// writes an fp32 partial that the finalize kernel sums before RoPE / cache append.
struct SkinnyArgs {
  const bf16 *x; int64_t lda; int M, K;
  const bf16 *w[4]; int width[4];
  float *part;            // [ksplit, M, wtot]
  int ksplit, wtot;
};

template <class T>
__global__ __launch_bounds__(T::NT) void skinny_proj_kernel(SkinnyArgs a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int ntn = a.wtot / T::BN, ntm = (a.M + T::BM - 1) / T::BM;
  const int ks = blockIdx.x / (ntn * ntm), rem = blockIdx.x % (ntn * ntm);
  const int mt = rem / ntn, nt = rem % ntn;
  int n_seg = nt * T::BN, seg = 0;
  while (n_seg >= a.width[seg]) { n_seg -= a.width[seg]; ++seg; }
  const int m0 = mt * T::BM, klen = a.K / a.ksplit, k0 = ks * klen;
  f32x16 acc[T::TN][T::TM];
  zero_acc<T>(acc);
  gemm_mainloop<T>(a.x + k0, a.lda, a.M, m0, a.w[seg] + (int64_t)k0 * a.width[seg], a.width[seg], n_seg, klen, smem, acc);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wn = wave % T::WGN, wm = wave / T::WGN;
  float *prow = a.part + (int64_t)ks * a.M * a.wtot;
#pragma unroll
  for (int tm = 0; tm < T::TM; ++tm) {
    const int m = m0 + wm * T::WM + tm * 32 + (lane & 31);
    if (m >= a.M) continue;
#pragma unroll
    for (int tn = 0; tn < T::TN; ++tn)
#pragma unroll
      for (int rq = 0; rq < 4; ++rq) {
        const int n = nt * T::BN + wn * T::WN + tn * 32 + rq * 8 + (lane >> 5) * 4;
        *reinterpret_cast<float4 *>(prow + (int64_t)m * a.wtot + n) =
            make_float4(acc[tn][tm][rq * 4], acc[tn][tm][rq * 4 + 1], acc[tn][tm][rq * 4 + 2], acc[tn][tm][rq * 4 + 3]);
      }
  }
}

typedef GemmTile<32, 128, 64, 1, 4> TileSkinny32;
typedef GemmTile<64, 128, 64, 1, 4> TileSkinny64;
typedef GemmTile<32, 64, 64, 1, 2> TileSkinny32N64;   // 64-wide tiles for widths that are not multiples of 128
typedef GemmTile<64, 64, 64, 2, 2> TileSkinny64N64;

typedef GemmTile<256, 256, 64, 4, 2> TileBig;    // eight waves, wave tile 64(m) x 128(n)
typedef GemmTile<256, 256, 64, 2, 2> TileBig4;   // four waves of 128 x 128 (plain main loop)
typedef GemmTile<256, 128, 64, 4, 1> TileHead;   // one 128-wide head per workgroup, wave tile 64(m) x 128(n)
typedef GemmTile<256, 64, 64, 4, 1> TileHead64;  // one 64-wide head per workgroup, wave tile 64(m) x 64(n)

template <class T, class K, class Args>
void launch(K kernel, const Args &a, int ntiles, hipStream_t st) {
  allow_dynamic_lds((const void *)kernel, T::SMEM);
  kernel<<<ntiles, T::NT, T::SMEM, st>>>(a);
}

}  // namespace

// The pipelined 256 x 256 tile against packed weights: widths in units of a 64-column group that
// holds whole heads, at least four k-tiles of 32 (H in units of 128 like everything on this path).
static bool proj_packed_ok(const Dims &d) {
  if (d.dh != 64 && d.dh != 128) return false;
  if (d.wq_w % d.dh || d.wk_w % d.dh || d.wc_w % 64 || d.wg_w % 64 || d.wq_w % 64 || d.wk_w % 64) return false;
  if (d.dh == 128 && (d.wq_w % 128 || d.wk_w % 128 || d.wc_w % 128)) return false;   // head inside one wave tile
  return d.H % 128 == 0 && d.H >= 256;
}
static int proj_packed_width(const Dims &d) { return (d.wtot + 255) / 256 * 256; }
static bool proj_direct_ok(const Dims &d) {
  // RoPE pairing is lane-local only if a wave tile (128 columns) holds whole heads
  if (d.dh != 128) return false;
  return !(d.H % 64 || d.dl % 64 || d.wq_w % 128 || d.wk_w % 128 || d.wc_w % 128 || d.wg_w % 128);
}
static bool proj_direct_big(const Dims &d) {
  // the pipelined loop takes at least four k-tiles of 32
  return proj_direct_ok(d) && !(d.wq_w % 256 || d.wk_w % 256 || d.wc_w % 256 || d.wg_w % 256) && d.H % 128 == 0 && d.H >= 256;
}

bool gemm_shapes_supported(const Dims &d) {
  if (d.dtype != GTA_BF16) return false;
  if (d.H % 128) return false;   // H is also the output width of the W_O GEMM, tiled in 128 columns
  if (!proj_direct_ok(d) && !proj_packed_ok(d)) return false;
  if (d.dl % 64) return false;
  // row offsets inside a 256-row tile are kept in 32 bits
  if (d.H > (1 << 20) || (int64_t)d.nq * d.dl > (1 << 20) || d.wg_w > (1 << 20)) return false;
  return true;
}

size_t proj_packed_bytes(const Dims &d) {
  return d.dtype == GTA_BF16 && !proj_direct_big(d) && proj_packed_ok(d) ? (size_t)d.H * proj_packed_width(d) * 2 : 0;
}


// Up to one and a half rounds of 64 x 128 tiles (512 are on the chip at once) the tiles that split K over their waves
// are ahead of the 256 x 256 ones, which would be too few; measured whole calls, 64-row against 256-row tiles:
// projection of the 1B shape 1700 tokens 94 against 104 us (756 tiles), 1900 109 / 110 (840), 2300 126 / 124 (1008); the
// 8 x 128 + 1024 shape 800 tokens 104 / 125 (728), 1000 127 / 130 (896); the paper's layer 3200 tokens 78 / 81 (700),
// 4000 97 / 90 (882).  Value decoder of the 1B shape 3000 tokens 137.7 / 138.8 (752), 4000 169.8 / 167.4 (1008).  W_O of
// the paper's layer 4000 tokens 97 / 101 (630), 5600 100.6 / 97.7 (880).
static bool short_gemm_ok(int M, int N) { return (int64_t)((M + 63) / 64) * ((N + 127) / 128) <= 768; }

bool proj_folds(const Dims &d, int batch, int64_t M) {
  return batch <= kFoldBatch && short_gemm_ok((int)M, d.wtot) && short_proj_folds(d, M);
}

void launch_proj_gemm(const Dims &d, const gta_weights &w, const void *x, int M, const PrefillWs &ws,
                      const gta_cache *cache, const int32_t *slots, int max_len, bool rope_by_token, const Fold &fold,
                      hipStream_t st) {
  ProjArgs a{};
  a.rope_by_token = rope_by_token ? 1 : 0;
  a.x = (const bf16 *)x; a.lda = d.H; a.M = M; a.K = d.H;
  const void *wm[4] = {w.wq, w.wk, w.wc, w.wg};
  const int wd[4] = {d.wq_w, d.wk_w, d.wc_w, d.wg_w};
  void *dst[4] = {ws.q, ws.k, ws.c, ws.g};
  for (int i = 0; i < 4; ++i) { a.w[i] = (const bf16 *)wm[i]; a.width[i] = wd[i]; a.dst[i] = (bf16 *)dst[i]; }
  a.seq_id = ws.seq_id; a.pos = ws.pos;
  a.rope = d.rope ? ws.rope : nullptr; a.max_len = max_len; a.dh = d.dh;
  if (cache) {
    a.kcache = (bf16 *)cache->k; a.ccache = (bf16 *)cache->c; a.slots = slots;
    a.max_batch = cache->max_batch; a.max_seq = cache->max_seq;
    a.pm = page_map_of(*cache);
  }
  if (short_gemm_ok(M, d.wtot)) { launch_short_proj(d, w, x, M, ws, cache, slots, max_len, rope_by_token, fold, st); return; }
  if (proj_direct_big(d)) {
    const int nt = (d.wtot / 256) * ((M + 255) / 256);
    launch<TileBig>(proj_gemm_kernel<TileBig>, a, nt, st);
  } else if (proj_packed_ok(d)) {
    bf16 *wpack = (bf16 *)ws.wpack;
    const int wpad = proj_packed_width(d);
    const int64_t chunks = (int64_t)d.H * (wpad / 8);
    pack_weights_kernel<<<(unsigned)((chunks + 255) / 256), 256, 0, st>>>(a, d.wtot, wpad, wpack);
    const int nt = (wpad / 256) * ((M + 255) / 256);
    const int which = d.dh == 64 ? 0 : 1;
    allow_dynamic_lds(which == 0 ? (const void *)proj_packed_kernel<TileBig, 64> : (const void *)proj_packed_kernel<TileBig, 128>,
                      TileBig::SMEM);
    if (which == 0) proj_packed_kernel<TileBig, 64><<<nt, TileBig::NT, TileBig::SMEM, st>>>(a, wpack, wpad);
    else proj_packed_kernel<TileBig, 128><<<nt, TileBig::NT, TileBig::SMEM, st>>>(a, wpack, wpad);
  } else {
    const int nt = (d.wtot / 128) * ((M + 255) / 256);
    launch<TileHead>(proj_gemm_kernel<TileHead>, a, nt, st);
  }
}

static bool skinny_wide_tiles(const Dims &d) { return !(d.wq_w % 128 || d.wk_w % 128 || d.wc_w % 128 || d.wg_w % 128); }

int skinny_ksplit(const Dims &d, int M) {
  const int ktiles = d.H / 64;
  const int bn = skinny_wide_tiles(d) ? 128 : 64;
  const int tiles = (d.wtot / bn) * ((M + 63) / 64);
  int want = (768 + tiles - 1) / tiles;
  if (want > 8) want = 8;
  int ks = 1;
  for (int c = 1; c <= want; ++c)
    if (ktiles % c == 0) ks = c;
  return ks;
}

// [M, wtot] = X . [W_Q | W_K | W_C | W_G] as `ksplit` fp32 partials (M small)
void launch_skinny_proj(const Dims &d, const gta_weights &w, const void *x, int M, float *part, int ksplit,
                        hipStream_t st) {
  SkinnyArgs a{};
  a.x = (const bf16 *)x; a.lda = d.H; a.M = M; a.K = d.H;
  const void *wm[4] = {w.wq, w.wk, w.wc, w.wg};
  const int wd[4] = {d.wq_w, d.wk_w, d.wc_w, d.wg_w};
  for (int i = 0; i < 4; ++i) { a.w[i] = (const bf16 *)wm[i]; a.width[i] = wd[i]; }
  a.part = part; a.ksplit = ksplit; a.wtot = d.wtot;
  if (skinny_wide_tiles(d)) {
    if (M <= 32) launch<TileSkinny32>(skinny_proj_kernel<TileSkinny32>, a, ksplit * (d.wtot / 128) * ((M + 31) / 32), st);
    else launch<TileSkinny64>(skinny_proj_kernel<TileSkinny64>, a, ksplit * (d.wtot / 128) * ((M + 63) / 64), st);
  } else {   // every width is a multiple of 64
    if (M <= 32) launch<TileSkinny32N64>(skinny_proj_kernel<TileSkinny32N64>, a, ksplit * (d.wtot / 64) * ((M + 31) / 32), st);
    else launch<TileSkinny64N64>(skinny_proj_kernel<TileSkinny64N64>, a, ksplit * (d.wtot / 64) * ((M + 63) / 64), st);
  }
}

void launch_decoder_gemm(const Dims &d, const void *L, const void *wp, const void *g, void *out, int M,
                         hipStream_t st) {
  DecoderArgs a{};
  a.L = (const bf16 *)L; a.ldl = (int64_t)d.nq * d.dl; a.M = M;
  a.wp = (const bf16 *)wp; a.dl = d.dl; a.dh = d.dh; a.hpq = d.hpq; a.nh = d.nh;
  a.g = (const bf16 *)g; a.gate = d.gate; a.out = (bf16 *)out;
  if (short_gemm_ok(M, d.nh * d.dh)) { launch_short_decoder(d, L, wp, g, out, M, st); return; }
  if (d.dh == 128 && d.hpq % 2 == 0 && d.dl % 128 == 0 && d.dl >= 256) {
    if (d.gate) launch<TileBig>(decoder_pair_kernel<TileBig, true>, a, (d.nh / 2) * ((M + 255) / 256), st);
    else launch<TileBig>(decoder_pair_kernel<TileBig, false>, a, (d.nh / 2) * ((M + 255) / 256), st);
    return;
  }
  if ((d.dh == 64 || d.dh == 128) && d.hpq % (256 / d.dh) == 0) {
    const int nt = (d.nh * d.dh / 256) * ((M + 255) / 256);
    if (d.gate) launch<TileBig4>(decoder_multi_kernel<TileBig4, true>, a, nt, st);
    else launch<TileBig4>(decoder_multi_kernel<TileBig4, false>, a, nt, st);
  } else if (d.dh % 128 == 0) {
    launch<TileHead>(decoder_gemm_kernel<TileHead>, a, d.nh * (d.dh / 128) * ((M + 255) / 256), st);
  } else {   // heads of 64: one head per 64-wide tile
    launch<TileHead64>(decoder_gemm_kernel<TileHead64>, a, d.nh * (d.dh / 64) * ((M + 255) / 256), st);
  }
}

void launch_plain_gemm(const void *A, int64_t lda, int M, int N, int K, const void *B, void *C, hipStream_t st) {
  PlainArgs a{(const bf16 *)A, lda, M, N, K, (const bf16 *)B, (bf16 *)C};
  if (M <= 128 && N % 32 == 0 && K % 16 == 0) {
    // a decode step's few rows: K split inside the workgroups (paper layer: 11 -> 6 us, whole step at batch 64
    // 49 -> 45 us, at batch 128 55 -> 46 us; before that 32 x 32 tiles of one wave each up to 64 rows)
    launch_rows_plain(A, lda, M, N, K, B, C, st);
    return;
  }
  if (short_gemm_ok(M, N)) { launch_short_plain(A, lda, M, N, K, B, C, st); return; }
  if (N % 256 == 0 && K % 128 == 0 && K >= 256) launch<TileBig>(plain_gemm_kernel<TileBig>, a, (N / 256) * ((M + 255) / 256), st);
  else launch<TileHead>(plain_gemm_kernel<TileHead>, a, (N / 128) * ((M + 255) / 256), st);
}

}  // namespace gta
