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
// Workgroup tile BM x BN x BK with WGM x WGN waves of 32x32x16 MFMA tiles.  Many rows run as a stream of 256 x 256 tiles
// through one workgroup per CU (gemm_stream): operands straight into LDS, results rounded to bf16, passed through LDS and
// written with 16-byte row-contiguous stores.
// The small tiles (split-K projection of the decode step) take the plain two-stage loop and store straight from the
// accumulator layout.  Short prefills take the kernels for few rows (short_gemm_ok).
#include <math.h>

#include <algorithm>
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

// Weight operand of a 256 x 256 tile: `base` points at its first k-row, rows are ld elements apart; column chunk c (8
// columns) sits chunk_bytes(c) behind the start of a row; `bytes` covers 32 rows.
struct WeightTile {
  const bf16 *base; int64_t ld; unsigned bytes;
  unsigned head_bytes;   // > 0: columns 128 .. 255 are another matrix (the next head) this far behind the first
  __device__ __forceinline__ unsigned chunk_bytes(int c) const { return head_bytes ? (c >> 4) * head_bytes + (c & 15) * 16 : c * 16; }
};
__device__ __forceinline__ WeightTile weight_tile(const bf16 *base, int64_t ld, unsigned head_bytes = 0) {
  return WeightTile{base, ld, (unsigned)(31 * ld * 2) + (head_bytes ? head_bytes + 256u : 512u), head_bytes};
}

// Order of a stream's tiles, of which XCD x (workgroup ids x mod 8) takes the x-th eighth: bands of 8 row strips, a band in
// panels of 4 columns (5, if there are no more), a panel row strip by row strip.  The 32 workgroups of an XCD then work on
// one block of 8 strips of X x 4 of the weights.  Panels of 7 where 7 divides the columns were slower (projections
// 16384 x 2048 x 3584 224 -> 228 us, 121600 x 4096 x 7168 5.96 -> 6.23 ms), 3 + 2 columns of 5 too (65536 x 1280 x 1280 196
// -> 199).  The divisors are known to the host.
// Up to 128 tiles behind the last whole round of 256 are shared by two workgroups of the XCD, 128 rows each: half a tile takes
// about 0.7 of the time of a whole one, and the CUs that would have had none take part (projections 16384 x 2048 x 3584, three and
// a half rounds, 211 -> 203 us; 6500 x 2048 x 3584, 1.4, 99 -> 91; W_O 16384 x 1280 x 1280, 1.25, 59 -> 54).
constexpr int kStreamGroups = 256;   // workgroups of a launch: one per CU
struct Divisor { unsigned magic; int d; };
inline Divisor divisor(int d) { return Divisor{0xffffffffu / (unsigned)d, d}; }
__device__ __forceinline__ int quotient(int x, Divisor v) {   // x >= 0; the product is at most one too few
  const int q = (int)__umulhi((unsigned)x, v.magic);
  return x - q * v.d >= v.d ? q + 1 : q;
}
struct StreamOrder {
  static constexpr int kBand = 8, kPanel = 4;
  int ntn, ntm;
  int rounds, halves;   // whole rounds of 256 tiles; tiles behind them that two workgroups share (else: workgroups with one more)
  Divisor band, panel, panel_end, width, width_end;   // tiles of a band, of a panel (and in the last band), columns of a panel (and of the last)
  int tiles() const { return ntn * ntm; }
  // half tiles: id (r & 7) + 16 (r >> 3) + 8 half takes half of tile r
  int workgroups() const { return rounds ? std::min(std::max(tiles(), 1), kStreamGroups) : (halves + 7) / 8 * 16; }
};
inline StreamOrder stream_order(int ntn, int ntm) {
  StreamOrder o;
  o.ntn = ntn; o.ntm = ntm;
  const int np = ntn <= StreamOrder::kPanel + 1 ? 1 : (ntn + StreamOrder::kPanel - 1) / StreamOrder::kPanel;
  const int w = (ntn + np - 1) / np;
  const int end = ntm % StreamOrder::kBand ? ntm % StreamOrder::kBand : StreamOrder::kBand, last = ntn - (ntn - 1) / w * w;
  o.band = divisor(StreamOrder::kBand * ntn);
  o.panel = divisor(StreamOrder::kBand * w);
  o.panel_end = divisor(end * w);
  o.width = divisor(w);
  o.width_end = divisor(last);
  const int rem = o.tiles() % kStreamGroups;
  o.halves = rem <= kStreamGroups / 2 ? rem : 0;
  o.rounds = o.tiles() / kStreamGroups + (rem > o.halves ? 1 : 0);
  return o;
}
struct TileAt { int m0, nt; };   // first row, column tile
__device__ __forceinline__ TileAt tile_at(const StreamOrder &order, int id) {
  const StreamOrder o = order;   // one round of scalar loads, no branches
  const int nblk = o.ntn * o.ntm, per = nblk >> 3;
  const int pos = id < per * 8 ? (id & 7) * per + (id >> 3) : id;   // the last nblk % 8 tiles keep their place
  const int band = quotient(pos, o.band), row0 = band * StreamOrder::kBand;
  const bool end = o.ntm - row0 < StreamOrder::kBand;
  const Divisor pd{end ? o.panel_end.magic : o.panel.magic, end ? o.panel_end.d : o.panel.d};
  int rem = pos - band * o.band.d;
  const int panel = quotient(rem, pd), col0 = panel * o.width.d;
  const bool narrow = o.ntn - col0 < o.width.d;
  const Divisor wd{narrow ? o.width_end.magic : o.width.magic, narrow ? o.width_end.d : o.width.d};
  rem -= panel * pd.d;
  const int row = quotient(rem, wd);
  return TileAt{(row0 + row) * 256, col0 + rem - row * wd.d};
}

// The kernel's only argument, read again where this is called: what a tile needs once would, held over the main loop, take
// more scalar registers than there are.
template <class A>
__device__ __forceinline__ const A &kernel_args() {
  typedef const __attribute__((address_space(4))) A Const;
  Const *args = (Const *)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(args));
  return *(const A *)args;
}

// ---- main loop over a stream of tiles ----------------------------------------------------------
// A workgroup works through the tiles blockIdx.x, + gridDim.x, .. of a launch of one workgroup per CU; the loads of a tile
// start under the last k-steps of the tile before it, and what is behind its epilogue's stores does not wait for them.
// 256 x 256 tile, eight waves (two per SIMD) of 64 x 128.  X comes in rows of 64 k (128 bytes: with 64 bytes of a row per
// load, the L2 moved every line twice and the loads alone took longer than the matrix instructions, 0.52 against 0.43 us
// per 32 k at K = 1280; now 0.38), three stages of 32 KiB; weights in four stages of 32 k, 16 KiB each.  The unit of the loop is a
// half step of 32 k (two k-steps of eight MFMAs per wave); half step u
//   * reads the fragments of its second k-step under the MFMAs of the first;
//   * waits at a barrier: every wave has then read all of weight stage u (u odd: and of X stage u / 2), and the loads of
//     half step u - 3 have landed, which brought weights u + 1 and, if u is odd, the rest of X stage (u + 1) / 2;
//   * reads the fragments of half step u + 1 under the MFMAs of the second k-step, and requests weights u + 4 and half of an
//     X stage: the first half of stage s + 3 with u = 2 s + 1, the second with u = 2 s + 2.
// The epilogue gets the X stage the tile has left as scratch: 4 KiB that belong to the wave until it has the same rows of
// that stage loaded.  It issues kStores stores at least, always (rows past the end are left to the buffer's bounds), so
// that the first half steps of the next tile can wait for loads that are older.
// LDS layout: a load instruction fills 1 KiB in lane order, so there is no padding; each lane fetches the 16-byte chunk that
// belongs in its slot.  X rows are 8 chunks, chunk c of row r in slot c ^ xs_swz(r): any 8 (16) consecutive rows read one
// logical chunk from 8 (16) different 16-byte columns of 128 (256) bytes.  Weight rows are 32 chunks, chunk c of k-row k in
// slot c ^ 4 (k % 4): the four k-rows of a transpose read lie in different 64-byte columns.
// Bound: power.  Without loads a half step takes 0.73 us on such data and 0.54 on zeros, the loads alone 0.38; together 0.8 and
// 0.6, of which the matrix instructions are 0.43 at 2.4 GHz.  Against a workgroup per tile, four stages of 32 k for both operands
// (0.87 and 0.77; kernels inside the calls): projection 65536 x 1280 x 1792 334 -> 293 us, W_O 65536 x 1280 x 1280 234 -> 195,
// projection 16384 x 2048 x 3584 243 -> 221, 6500 x 2048 x 3584 114 -> 110, 121600 x 4096 x 7168 6.10 -> 5.96 ms (5.51 on a
// day when that took 5.67, with a tile's place worked out in one round of scalar loads and no branches).
struct StreamTile { const bf16 *A; int rows; WeightTile B; };   // row m0 of the row operand, rows from there, weight columns

struct StreamLoop {
  static constexpr int BM = 256, BN = 256, X_BYTES = BM * 64 * 2, W_BYTES = 32 * BN * 2, W_OFF = 3 * X_BYTES, SMEM = W_OFF + 4 * W_BYTES;
  static constexpr int WGM = 4, WGN = 2, NT = 512, WM = BM / WGM, WN = BN / WGN, TM = WM / 32, TN = WN / 32;
};
__device__ __forceinline__ int xs_swz(int r) { return (r & 7) ^ ((r >> 3) & 1); }

// acc[tn][tm][r]:  n = wn*128 + tn*32 + 8*(r/4) + 4*(lane/32) + r%4,  m = wm*64 + tm*32 + lane%32, wn = wave % 2, wm = wave / 2.
// K a multiple of 128, at least 256.
// Args: the kernel's argument, with the order; src(args, tile), epi(args, blocks of 32 rows of a wave, tile, acc, scratch).
template <class Args, class Src, class Epi>
__device__ __forceinline__ void gemm_stream(int64_t lda, int K, char *smem, const Src &src, const Epi &epi) {
  typedef StreamLoop T;
  constexpr int TN = T::TN, kSet = 4;   // load instructions of a wave per half step
  const int lane = threadIdx.x & 63, h = lane >> 5, ln = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wn = wave % T::WGN, wm = wave / T::WGN;
  const int nk = K / 64;
  const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char *)smem;
  // what is requested next.  Rows past the last valid one read as 0, and so does everything behind the last tile.
  // This wave's loads: rows 32 wave + 8 j + lane/8 of an X stage, k-rows 4 wave + 2 j + lane/32 of a weight stage.
  unsigned xv[4], wv[2], xbytes = 0, wbytes = 0;
  int64_t wstep = 0;
  const char *xbase = nullptr, *wbase = nullptr;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int r = wave * 32 + j * 8 + (lane >> 3);
    xv[j] = (unsigned)(r * lda * 2) + ((lane & 7) ^ xs_swz(r)) * 16;
  }
  TileAt now{}, next{};   // the tile that is worked on and the one that is requested
  bool any = false;       // is there one?
  // tile `round` of this workgroup, or half a tile behind the rounds
  auto request_x = [&](int round) {
    const Args &args = kernel_args<Args>();
    const StreamOrder &order = args.order;
    xbytes = 0;
    int id = blockIdx.x + round * kStreamGroups, half = 0;
    if (round < order.rounds) any = id < order.ntn * order.ntm;
    else {
      const int r = (blockIdx.x & 7) + (blockIdx.x >> 4) * 8;
      half = (blockIdx.x >> 3) & 1;
      id = order.rounds * kStreamGroups + r;
      any = round == order.rounds && r < order.halves;
    }
    if (!any) return;
    next = tile_at(order, id);
    next.m0 += half * (T::BM / 2);
    const StreamTile s = src(args, next);
    any = s.rows > 0;
    if (!any) return;
    xbase = reinterpret_cast<const char *>(s.A);
    xbytes = (unsigned)((min(s.rows, round < order.rounds ? T::BM : T::BM / 2) - 1) * lda * 2) + 128u;
  };
  auto request_w = [&]() {
    wbytes = 0;
    if (!any) return;
    const StreamTile s = src(kernel_args<Args>(), next);
    wbase = reinterpret_cast<const char *>(s.B.base);
    wbytes = s.B.bytes;
    wstep = (int64_t)32 * s.B.ld * 2;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int k = (wave * 2 + j) * 2 + h;
      wv[j] = (unsigned)(k * s.B.ld * 2) + s.B.chunk_bytes(ln ^ ((k & 3) << 2));
    }
  };
  // LDS offsets of X stages s, s + 1, s + 2 and weight stages u .. u + 3
  int xs[3] = {0, T::X_BYTES, 2 * T::X_BYTES}, ws[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) ws[i] = T::W_OFF + i * T::W_BYTES;
  auto load_x = [&](int at, int j) { load_to_lds(buffer_of(xbase, xbytes), xv[j], lds0 + at + (wave * 4 + j) * 1024); };
  auto load_w = [&](int at, int j) { load_to_lds(buffer_of(wbase, wbytes), wv[j], lds0 + at + (wave * 2 + j) * 1024); };
  // fragment addresses: X chunk 2 kk + h of row ln (+ 32 tm), weight rows 8 h + (lane%16)/4 (+ 16 kk, + 4)
  const int wr = (lane & 15) >> 2;
  const int wo = (h * 8 + wr) * 512 + (wn * 16 + (wr << 2) + ((lane >> 4) & 1) * 2 + ((lane & 3) >> 1)) * 16 + (lane & 1) * 8;
  struct Frags { bf16x8 x[T::TM]; s16x4 lo[TN], hi[TN]; };
  Frags f0, f1;
  f32x16 acc[TN][T::TM];
  // a tile of TM x 128 rows, whose first fragments are in f0; `loose`: half steps that wait for loads older than the stores of
  // the tile before
  auto fragments = [&](auto tm_tag) {   // reads of a k-step: (f, X stage at, its k-step, weights at, their k-step, i)
    constexpr int TM = decltype(tm_tag)::value;
    const int xo = (wm * TM * 32 + ln) * 128 + ((h ^ xs_swz(ln)) << 4);
    return [=](Frags &f, int xat, int xkk, int wat, int wkk, int i) {   // read i, in the order the MFMAs of the step need them
      if (i >= 2 && i < 2 + TM) {
        f.x[i - 2] = *reinterpret_cast<const bf16x8 *>(smem + ((xat + xo) ^ (xkk << 5)) + (i - 2) * 4096);
        return;
      }
      const int w = i < 2 ? i : i - TM, tn = w / 2;
      const s16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(smem + ((wat + wo) ^ (tn << 6)) + wkk * 8192 + (w & 1) * 2048));
      if (w & 1) f.hi[tn] = v; else f.lo[tn] = v;
    };
  };
  auto first_fragments = [&](auto tm_tag) {
    const auto read_frag = fragments(tm_tag);
#pragma unroll
    for (int i = 0; i < decltype(tm_tag)::value + 2 * TN; ++i) read_frag(f0, xs[0], 0, ws[0], 0, i);
  };
  auto work_tile = [&](auto tm_tag, int round, int loose) {
    constexpr int TM = decltype(tm_tag)::value;
    constexpr int NR = TM + 2 * TN, NM = TM * TN;         // fragment reads and MFMAs of a k-step
    constexpr int READS = NM - 3, MEET = TM == 1 ? 2 : NM - 3;   // the reads go out under the first READS MFMAs; the barrier's place
    const auto read_frag = fragments(tm_tag);
    auto read_frags = [&](Frags &f, int xat, int xkk, int wat, int wkk, int i) {
#pragma unroll
      for (int r = 0; r < NR; ++r)
        if (r * READS / NR == i) read_frag(f, xat, xkk, wat, wkk, r);
    };
    auto mma = [&](const Frags &f, int i) {
      const int tn = i / TM, tm = i % TM;
      const s16x8 w8 = __builtin_shufflevector(f.lo[tn], f.hi[tn], 0, 1, 2, 3, 4, 5, 6, 7);
      acc[tn][tm] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, w8), f.x[tm], acc[tn][tm], 0, 0, 0);
    };
    now = next;
#pragma unroll
    for (int tn = 0; tn < TN; ++tn)
#pragma unroll
      for (int tm = 0; tm < TM; ++tm)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[tn][tm][r] = 0.f;
#pragma unroll 1
    for (int s = 0; s < nk; ++s) {
#pragma unroll
      for (int p = 0; p < 2; ++p) {   // half step 2 s + p
#pragma unroll
        for (int i = 0; i < NM; ++i) {
          read_frags(f1, xs[0], 2 * p + 1, ws[0], 1, i);
          mma(f0, i);
          if (i == MEET) {
            if (2 * s + p < loose) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(2 * kSet + Epi::kStores) : "memory");
            else asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(2 * kSet) : "memory");
          }
          __builtin_amdgcn_sched_barrier(0);
        }
        if (p == 0) { if (s == nk - 2) request_w(); }
        else if (s == nk - 3) request_x(round + 1);
        else xbase += 128;
#pragma unroll
        for (int i = 0; i < NM; ++i) {
          read_frags(f0, p ? xs[1] : xs[0], p ? 0 : 2, ws[1], 0, i);
#pragma unroll
          for (int l = 0; l < 4; ++l)
            if ((NM == 8 ? 2 * l + 1 : l) == i) {
              if (l >= 2) load_w(ws[0], l - 2);
              else if (p == 0) load_x(xs[2], 2 + l);
              else if (s + 1 < nk) load_x(xs[0], l);   // the last one: behind the epilogue
            }
          mma(f1, i);
          __builtin_amdgcn_sched_barrier(0);
        }
        wbase += wstep;
        const int w0 = ws[0];
        ws[0] = ws[1]; ws[1] = ws[2]; ws[2] = ws[3]; ws[3] = w0;
      }
      const int x0 = xs[0];
      xs[0] = xs[1]; xs[1] = xs[2]; xs[2] = x0;
    }
    asm volatile("" ::: "memory");
    epi(kernel_args<Args>(), tm_tag, now, acc, smem + xs[2] + wave * 4096);
  };
  typedef std::integral_constant<int, T::TM> Whole;
  typedef std::integral_constant<int, T::TM / 2> Half;

  request_x(0);
  request_w();
  if (!any) return;
  load_x(xs[0], 0); load_x(xs[0], 1);
#pragma unroll
  for (int i = 0; i < 4; ++i) {   // X 0b W 0 | X 1a W 1 | X 1b W 2 | X 2a W 3
    if (i & 1) xbase += 128;
    load_x(xs[(i + 1) / 2], i & 1 ? 0 : 2); load_x(xs[(i + 1) / 2], i & 1 ? 1 : 3);
    load_w(ws[i], 0); load_w(ws[i], 1);
    wbase += wstep;
  }
  asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(3 * kSet) : "memory");
  const int rounds = kernel_args<Args>().order.rounds;
  if (rounds) first_fragments(Whole{});
  else first_fragments(Half{});
  for (int round = 0;;) {
    const int loose = round ? 3 : 0;
    if (round == rounds) { work_tile(Half{}, round, loose); break; }
    work_tile(Whole{}, round, loose);
    if (!any) break;
    ++round;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    load_x(xs[2], 0); load_x(xs[2], 1);
    // the fragments that the last half step has read were those of a whole tile, or gave their registers to the epilogue
    if (round == rounds) first_fragments(Half{});
    else if constexpr (Epi::kReread) first_fragments(Whole{});
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // what was requested behind the last tile still writes LDS
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
  const int id = blockIdx.x, nblk = ntn * ntm, per = nblk / 8;
  const int pos = id < per * 8 ? (id % 8) * per + id / 8 : id;   // the last nblk % 8 tiles keep their place
  const int band = pos / (RB * ntn);
  int rem = pos - band * RB * ntn;
  const int h = min(RB, ntm - band * RB);      // row strips of this band
  const int panel = rem / (h * PW);
  rem -= panel * h * PW;
  mt = band * RB + rem % h;
  nt = panel * PW + rem / h;
}

// ---- epilogue of a stream's tile ----------------------------------------------------------------
// A wave rounds its 64 x 128 part to bf16 and writes it through its 4 KiB of scratch, 32 rows x 64 columns at a time (in the
// accumulator layout a lane owns 4 consecutive columns of one row: stores would be 8 bytes wide): 16-byte stores, eight
// lanes per 128 bytes of a row.  Chunk c of row r sits in slot c ^ (r % 8).  Rows past the end are beyond `bytes`.
constexpr int kStreamStores = 16;
// The lane, in a form that keeps what the compiler derives from it inside the epilogue: hoisted out of the loop over tiles,
// addresses of a few instructions each took the registers of the main loop (30 spills).
__device__ __forceinline__ int epilogue_lane() {
  int lane = threadIdx.x & 63;
  asm volatile("" : "+v"(lane));
  return lane;
}
// columns 64 tp .. of the wave to `base` (row 0 of the tile, first of the 64 columns); also(r, v) gets row r of the tile's wave
template <int TM, class Also>
__device__ __forceinline__ void store_columns(const f32x16 (&acc)[StreamLoop::TN][StreamLoop::TM], int tp, char *st, bf16 *base, unsigned bytes,
                                              int ld, const Also &also) {
  typedef StreamLoop T;
  const int lane = epilogue_lane(), ln = lane & 31, h = lane >> 5;
  const int wm = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) / T::WGN;
  const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(base, 0, bytes, 0x00020000);
  const unsigned voff = (unsigned)((wm * TM * 32 + (lane >> 3)) * ld + (lane & 7) * 8) * 2;
#pragma unroll
  for (int tm = 0; tm < TM; ++tm) {
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int rq = 0; rq < 4; ++rq) {
        const f32x16 &v = acc[tp * 2 + q][tm];
        *reinterpret_cast<bf16x4 *>(st + ln * 128 + (((q * 4 + rq) ^ (ln & 7)) << 4) + h * 8) = pack4(v[rq * 4], v[rq * 4 + 1], v[rq * 4 + 2], v[rq * 4 + 3]);
      }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = i * 8 + (lane >> 3);
      const u32x4 v = *reinterpret_cast<const u32x4 *>(st + r * 128 + (((lane & 7) ^ (r & 7)) << 4));
      __builtin_amdgcn_raw_buffer_store_b128(v, rs, voff + (tm * 32 + i * 8) * ld * 2, 0, 0);
      also(tm * 32 + r, v);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
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
  // positions of this lane's rows: asked for before the main loop (0.8 us of load latency per tile otherwise)
  const bool rotate = a.rope != nullptr && seg < 2;
  int pos_of[T::TM];
#pragma unroll
  for (int tm = 0; tm < T::TM; ++tm)
    pos_of[tm] = a.pos[min(m0 + (int)(threadIdx.x >> 6) / T::WGN * T::WM + tm * 32 + (int)(threadIdx.x & 31), a.M - 1)];
  gemm_mainloop<T>(a.x, a.lda, a.M, m0, a.w[seg], a.width[seg], n_glob, a.K, smem, acc);

  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wn = wave % T::WGN, wm = wave / T::WGN;
  const int nw = n_glob + wn * T::WN;            // first column of this wave inside its segment
  const int half = a.dh / 2;
  bf16 *cache = seg == 1 ? a.kcache : (seg == 2 ? a.ccache : nullptr);
  const int width = a.width[seg];
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
}

// ---- projection against packed weights -----------------------------------------------------------
// The setup launch copies the four weight matrices side by side into one [H, Wtot] matrix (pack_of), so that a
// 256-column tile may straddle Q | K | C | gate: this serves output widths that are multiples of 64
// but not of 256 (heads of 64, a single shared key).  Columns are routed to their outputs per
// 64-column group (a head never straddles one).
// The packed row is padded with zero columns to a multiple of 256 (wpad); the last tile computes
// them and stores nothing for them.
//
// ---- both projections as streams of tiles --------------------------------------------------------
// PACKED: weights from wpack (rows of wpad columns), else from the four matrices (widths multiples of 256).  A group of 64
// columns lies in one of Q | K | C | gate, whole heads in a wave's 128 columns.
struct ProjStream { StreamOrder order; ProjArgs a; const bf16 *wpack; int wpad; };

template <int DH, bool PACKED>
struct ProjStreamEpi {
  static constexpr int kStores = kStreamStores;
  static constexpr bool kReread = true;
  template <class Rows>
  __device__ __forceinline__ void operator()(const ProjStream &args, Rows, TileAt t, f32x16 (&acc)[StreamLoop::TN][StreamLoop::TM], char *st) const {
    typedef StreamLoop T;
    const ProjArgs &a = args.a;
    const int lane = epilogue_lane(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wn = wave % T::WGN, wm = wave / T::WGN;
    constexpr int TM = Rows::value;
    const int m0 = t.m0, mw = m0 + wm * TM * 32, n0 = t.nt * T::BN + wn * T::WN;   // first row of the tile and of the wave, first column of the wave
    const int b1 = a.width[0], b2 = b1 + a.width[1], b3 = b2 + a.width[2], wtot = b3 + a.width[3];
    if (a.rope && n0 < b2) {   // q or k columns: column j of a head pairs with j + DH/2
      constexpr int half = DH / 2, tiles_half = DH / 64, tiles_head = DH / 32, heads = T::WN / DH;
      constexpr int G = TM * tiles_half * 4, AHEAD = 2;   // groups of 4 columns; table values asked for AHEAD groups early
      bool rot[TM];
      const float2 *trow[TM];
#pragma unroll
      for (int tm = 0; tm < TM; ++tm) {
        const int mc = min(mw + tm * 32 + (lane & 31), a.M - 1);
        const int p = a.rope_by_token ? mc : a.pos[mc];
        // a row that does not rotate takes row 0 of the table and keeps its values
        rot[tm] = PACKED || a.rope_by_token || p < a.max_len;
        trow[tm] = a.rope + (int64_t)(a.rope_by_token ? p : PACKED ? max(min(p, a.max_len - 1), 0) : rot[tm] ? p : 0) * half + (lane >> 5) * 4;
      }
      float4 tv[AHEAD + 1][2];
      auto ask = [&](int g) {
        const float4 *tp = reinterpret_cast<const float4 *>(trow[g / (tiles_half * 4)] + (g / 4) % tiles_half * 32 + g % 4 * 8);
        tv[g % (AHEAD + 1)][0] = tp[0]; tv[g % (AHEAD + 1)][1] = tp[1];
      };
#pragma unroll
      for (int g = 0; g < AHEAD; ++g) ask(g);
#pragma unroll
      for (int g = 0; g < G; ++g) {
        if (g + AHEAD < G) ask(g + AHEAD);
        const int tm = g / (tiles_half * 4), rq = g % 4;
        const float4 t0 = tv[g % (AHEAD + 1)][0], t1 = tv[g % (AHEAD + 1)][1];
        const float cs[4] = {t0.x, t0.z, t1.x, t1.z}, sn[4] = {t0.y, t0.w, t1.y, t1.w};
#pragma unroll
        for (int hd = 0; hd < heads; ++hd) {
          const int tn = hd * tiles_head + (g / 4) % tiles_half, tn_hi = tn + tiles_half;
          const bool turn = n0 + hd * DH < b2 && rot[tm];   // columns behind q and k stay as they are, infinities and all
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float lo = acc[tn][tm][rq * 4 + i], hi = acc[tn_hi][tm][rq * 4 + i];
            // spelled out, as the product that is rounded by itself decides the last bit: against packed weights hi cos, else lo sin
            const float tl = fmaf(lo, cs[i], -(hi * sn[i])), th = PACKED ? fmaf(lo, sn[i], hi * cs[i]) : fmaf(hi, cs[i], lo * sn[i]);
            acc[tn][tm][rq * 4 + i] = turn ? tl : lo;
            acc[tn_hi][tm][rq * 4 + i] = turn ? th : hi;
          }
        }
        __builtin_amdgcn_sched_barrier(0);   // else the values of all groups are asked for at once: spills
      }
    }
    // cache rows of the wave's rows, one per lane
    const bool caches = a.kcache && n0 < b3 && n0 + T::WN > b1;
    int64_t crow = -1;
    if (caches) {
      const int m = mw + lane;
      if (m < a.M && lane < TM * 32) {
        const int p = a.pos[m], b = a.seq_id[m];
        const int slot = a.slots ? a.slots[b] : b;
        if (slot >= 0 && slot < a.max_batch && p >= 0 && p < a.max_seq) crow = cache_row(PageMap{a.pm.table, a.pm.page_size, a.pm.pages_per_slot, a.pm.num_pages}, a.max_seq, slot, p);
      }
    }
#pragma unroll
    for (int tp = 0; tp < 2; ++tp) {
      const int col = n0 + tp * 64;
      const bool s1 = col >= b1, s2 = col >= b2, s3 = col >= b3;
      const int lcol = col - (s3 ? b3 : s2 ? b2 : s1 ? b1 : 0), width = s3 ? a.width[3] : s2 ? a.width[2] : s1 ? a.width[1] : a.width[0];
      bf16 *dst = (s3 ? a.dst[3] : s2 ? a.dst[2] : s1 ? a.dst[1] : a.dst[0]) + (int64_t)m0 * width + lcol;
      const unsigned bytes = PACKED && col >= wtot ? 0u : (unsigned)((min(a.M - m0, TM * 128) - 1) * width * 2) + 128u;   // padding: none
      if (caches && s1 && !s3) {
        bf16 *cache = (s2 ? a.ccache : a.kcache) + lcol + (lane & 7) * 8;
        store_columns<TM>(acc, tp, st, dst, bytes, width, [&](int r, u32x4 v) {
          const int64_t cr = ((int64_t)__shfl((int)(crow >> 32), r) << 32) | (unsigned)__shfl((int)crow, r);
          if (cr >= 0) *reinterpret_cast<u32x4 *>(cache + cr * width) = v;
        });
      } else {
        store_columns<TM>(acc, tp, st, dst, bytes, width, [](int, u32x4) {});
      }
    }
  }
};

template <int DH, bool PACKED>
__global__ __launch_bounds__(StreamLoop::NT) void proj_stream_kernel(ProjStream args) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  typedef StreamLoop T;
  gemm_stream<ProjStream>(args.a.lda, args.a.K, smem, [](const ProjStream &g, TileAt t) {
    const ProjArgs &a = g.a;
    const int n0 = t.nt * T::BN;
    const bf16 *x = a.x + (int64_t)t.m0 * a.lda;
    if constexpr (PACKED) return StreamTile{x, a.M - t.m0, weight_tile(g.wpack + n0, g.wpad)};
    const int b1 = a.width[0], b2 = b1 + a.width[1], b3 = b2 + a.width[2];
    const bool s1 = n0 >= b1, s2 = n0 >= b2, s3 = n0 >= b3;
    const int lcol = n0 - (s3 ? b3 : s2 ? b2 : s1 ? b1 : 0), width = s3 ? a.width[3] : s2 ? a.width[2] : s1 ? a.width[1] : a.width[0];
    return StreamTile{x, a.M - t.m0, weight_tile((s3 ? a.w[3] : s2 ? a.w[2] : s1 ? a.w[1] : a.w[0]) + lcol, width)};
  }, ProjStreamEpi<DH, PACKED>{});
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

// Two heads of one map group per 256-wide tile (they share the row operand L_g), as a stream of tiles.  The gate is applied to
// the fp32 accumulators: the wave asks for its 64 x 128 pre-activations at the start of the epilogue (64 registers, the
// fragments' and more), and they pass through its scratch into accumulator layout, 32 rows x 64 columns at a time.
// Bound: 201 MB for 16384 rows of the 1B shape (40 us of a large copy).  Measured against a workgroup per tile whose gate tile
// took the place of the last four k-tiles' operands, with X in rows of 64 bytes: 16384 rows of the 1B shape 72 -> 64 us, 4000 rows (125 tiles,
// shared) 23 -> 18, 16384 rows of the 8 x 128 + 1024 shape 182 -> 163.
struct DecoderStream { StreamOrder order; DecoderArgs a; };

// KIND: kGateOff, kGateSigmoid (the method's, the short path) or -1, any other.  A kernel each: with both nonlinearities behind a branch
// in one the compiler sees a way around both, on which the gate values are still in flight, and waits for them in the main loop.
template <int KIND>
struct DecoderStreamEpi {
  static constexpr bool GATE = KIND != kGateOff;
  static constexpr int kStores = kStreamStores;
  static constexpr bool kReread = true;
  template <class Rows>
  __device__ __forceinline__ void operator()(const DecoderStream &args, Rows, TileAt t, f32x16 (&acc)[StreamLoop::TN][StreamLoop::TM], char *st) const {
    typedef StreamLoop T;
    constexpr int TM = Rows::value;
    const DecoderArgs &a = args.a;
    const int lane = epilogue_lane(), ln = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wn = wave % T::WGN, wm = wave / T::WGN;
    const int ldo = a.nh * a.dh;
    const int64_t at = (int64_t)t.m0 * ldo + t.nt * T::BN + wn * T::WN;
    const unsigned bytes = (unsigned)((min(a.M - t.m0, TM * 128) - 1) * ldo * 2) + 256u;
    const unsigned voff = (unsigned)((wm * TM * 32 + (lane >> 3)) * ldo + (lane & 7) * 8) * 2;
    const __amdgpu_buffer_rsrc_t ro = __builtin_amdgcn_make_buffer_rsrc(a.out + at, 0, bytes, 0x00020000);
    u32x4 gt[TM][2][4];
    auto ask = [&](int tm) {
      const __amdgpu_buffer_rsrc_t rg = __builtin_amdgcn_make_buffer_rsrc((void *)(a.g + at), 0, bytes, 0x00020000);
#pragma unroll
      for (int tp = 0; tp < 2; ++tp)
#pragma unroll
        for (int i = 0; i < 4; ++i) gt[tm][tp][i] = __builtin_amdgcn_raw_buffer_load_b128(rg, voff + (tm * 32 + i * 8) * ldo * 2 + tp * 128, 0, 0);
    };
    if constexpr (GATE) {
#pragma unroll
      for (int tm = 0; tm < (KIND < 0 ? 1 : TM); ++tm) ask(tm);   // the other nonlinearities need the registers
      asm volatile("" ::: "memory");
    }
#pragma unroll
    for (int tm = 0; tm < TM; ++tm)
#pragma unroll
      for (int tp = 0; tp < 2; ++tp) {
        if (KIND < 0 && tm > 0 && tp == 0) ask(tm);
        if constexpr (GATE) {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int r = i * 8 + (lane >> 3);
            *reinterpret_cast<u32x4 *>(st + r * 128 + (((lane & 7) ^ (r & 7)) << 4)) = gt[tm][tp][i];
          }
        }
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
          for (int rq = 0; rq < 4; ++rq) {
            bf16x4 *slot = reinterpret_cast<bf16x4 *>(st + ln * 128 + (((q * 4 + rq) ^ (ln & 7)) << 4) + h * 8);
            const f32x16 &v = acc[tp * 2 + q][tm];
            float f[4] = {1.f, 1.f, 1.f, 1.f};
            if constexpr (GATE) {
              const bf16x4 gz = *slot;
#pragma unroll
              for (int e = 0; e < 4; ++e) f[e] = gate_factor(KIND < 0 ? a.gate : KIND, (float)gz[e]);
            }
            *slot = pack4(v[rq * 4] * f[0], v[rq * 4 + 1] * f[1], v[rq * 4 + 2] * f[2], v[rq * 4 + 3] * f[3]);
          }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int r = i * 8 + (lane >> 3);
          const u32x4 v = *reinterpret_cast<const u32x4 *>(st + r * 128 + (((lane & 7) ^ (r & 7)) << 4));
          __builtin_amdgcn_raw_buffer_store_b128(v, ro, voff + (tm * 32 + i * 8) * ldo * 2 + tp * 128, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
  }
};

template <int KIND>
__global__ __launch_bounds__(StreamLoop::NT) void decoder_stream_kernel(DecoderStream args) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  gemm_stream<DecoderStream>(args.a.ldl, args.a.dl, smem, [](const DecoderStream &g, TileAt t) {
    const DecoderArgs &a = g.a;
    const int head = t.nt * 2;
    return StreamTile{a.L + (int64_t)t.m0 * a.ldl + (head / a.hpq) * a.dl, a.M - t.m0,
                      weight_tile(a.wp + (int64_t)head * a.dl * a.dh, a.dh, (unsigned)(a.dl * a.dh * 2))};
  }, DecoderStreamEpi<KIND>{});
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
  gemm_mainloop<T>(a.A, a.lda, a.M, m0, a.B, a.N, n0, a.K, smem, acc);
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

struct PlainStream { StreamOrder order; PlainArgs a; };

struct PlainStreamEpi {
  static constexpr int kStores = kStreamStores;
  static constexpr bool kReread = false;
  template <class Rows>
  __device__ __forceinline__ void operator()(const PlainStream &args, Rows, TileAt t, f32x16 (&acc)[StreamLoop::TN][StreamLoop::TM], char *st) const {
    typedef StreamLoop T;
    constexpr int TM = Rows::value;
    const PlainArgs &a = args.a;
    const int wn = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) % T::WGN;
    bf16 *base = a.C + (int64_t)t.m0 * a.N + t.nt * T::BN + wn * T::WN;
    const unsigned bytes = (unsigned)((min(a.M - t.m0, TM * 128) - 1) * a.N * 2) + 128u;
    store_columns<TM>(acc, 0, st, base, bytes, a.N, [](int, u32x4) {});
    store_columns<TM>(acc, 1, st, base + 64, bytes, a.N, [](int, u32x4) {});
  }
};

__global__ __launch_bounds__(StreamLoop::NT) void plain_stream_kernel(PlainStream args) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  gemm_stream<PlainStream>(args.a.lda, args.a.K, smem, [](const PlainStream &g, TileAt t) {
    return StreamTile{g.a.A + (int64_t)t.m0 * g.a.lda, g.a.M - t.m0, weight_tile(g.a.B + t.nt * StreamLoop::BN, g.a.N)};
  }, PlainStreamEpi{});
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

typedef GemmTile<256, 256, 64, 2, 2> TileBig4;   // four waves of 128 x 128 (plain main loop)
typedef GemmTile<256, 128, 64, 4, 1> TileHead;   // one 128-wide head per workgroup, wave tile 64(m) x 128(n)
typedef GemmTile<256, 64, 64, 4, 1> TileHead64;  // one 64-wide head per workgroup, wave tile 64(m) x 64(n)

template <class Args>
void launch_stream(void (*kernel)(Args), Args args, int M, int N, hipStream_t st) {
  args.order = stream_order(N / StreamLoop::BN, (M + StreamLoop::BM - 1) / StreamLoop::BM);
  allow_dynamic_lds((const void *)kernel, StreamLoop::SMEM);
  kernel<<<args.order.workgroups(), StreamLoop::NT, StreamLoop::SMEM, st>>>(args);
}

template <class T, class K, class Args>
void launch(K kernel, const Args &a, int ntiles, hipStream_t st) {
  allow_dynamic_lds((const void *)kernel, T::SMEM);
  kernel<<<ntiles, T::NT, T::SMEM, st>>>(a);
}

}  // namespace

// The stream of 256 x 256 tiles against packed weights: widths in units of a 64-column group that
// holds whole heads, H a multiple of 128, at least 256 (gemm_stream).
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
  // the stream takes whole tiles of columns from one matrix and multiples of 128 in K, at least 256
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

// 512 tiles of 64 x 128 are on the chip at once; up to there the tiles that split K over their waves are ahead of the stream of 256 x
// 256 tiles, of which there would be too few.  Whole calls, 64-row tiles / stream: 1B shape 1200 tokens (532 tiles in the
// projection) 76.3 / 75.7 us, 1700 (756) 90.3 / 88.1, 2200 (560 in the decoder) 106.1 / 100.9, 3000 (752) 131.8 / 126.8; paper's layer 2400
// tokens (532) 90.3 / 86.9, 3200 (700) 108.3 / 98.4, 4 x 1000 (630 in W_O) 80.5 / 77.4; 768 wide layer 4 x 1000 62.6 / 59.3.  Alone the
// projections are level at 1200 (38.4 / 38.5) and 2000 tokens (paper, 448 tiles: 31.3 / 32.1).  Contractions beyond 2048 and shapes
// that no stream takes keep one and a half rounds: 8 x 128 + 1024 shape 600 tokens (560) 97.9 / 98.7, 700 (616) 102.5 / 103.1.
static int short_tiles(int K, bool stream) { return stream && K <= 2048 ? 512 : 768; }
static bool short_gemm_ok(int M, int N, int tiles) { return (int64_t)((M + 63) / 64) * ((N + 127) / 128) <= tiles; }
// Packed weights have to be laid out first: with heads of 128 (those of 64 have 64-row tiles of only 64 columns) and long contractions
// the 64-row tiles stay ahead for longer.  Whole calls, 64-row tiles / stream: 2048 -> 3456 513 tiles 72.4 / 76.3 us, 567 75.8 / 78.6, 675
// 82.4 / 83.6, 729 85.3 / 84.3; 2048 -> 3200 525 74.4 / 77.0, 600 78.6 / 80.2, 675 83.0 / 83.9; 1792 -> 3072 528 75.0 / 76.6, 648 81.1 / 81.8;
// but 1536 -> 2688 525 73.6 / 73.9, 609 78.8 / 78.2, 672 87.4 / 81.2; 1024 -> 3456 675 70.0 / 68.7; 1280 -> 2304 630 81.0 / 79.8.  Heads of
// 64: 2048 -> 2752 528 67.6 / 67.9, 550 69.5 / 68.9, 638 75.0 / 72.3.
static int proj_short_tiles(const Dims &d) {
  if (!proj_direct_big(d) && proj_packed_ok(d) && d.dh == 128 && d.H > 1536) return std::max(704, short_tiles(d.H, true));
  return short_tiles(d.H, proj_direct_big(d) || proj_packed_ok(d));
}
static bool decoder_streams(const Dims &d) { return d.dh == 128 && d.hpq % 2 == 0 && d.dl % 128 == 0 && d.dl >= 256; }

bool proj_folds(const Dims &d, int batch, int64_t M) {
  return batch <= kFoldBatch && short_gemm_ok((int)M, d.wtot, proj_short_tiles(d)) && short_proj_folds(d, M);
}

PackWeights pack_of(const Dims &d, const gta_weights &w, int64_t M, const PrefillWs &ws) {
  PackWeights p{};
  if (proj_direct_big(d) || !proj_packed_ok(d) || short_gemm_ok((int)M, d.wtot, proj_short_tiles(d))) return p;
  p.w[0] = w.wq; p.w[1] = w.wk; p.w[2] = w.wc; p.w[3] = w.wg;
  p.width[0] = d.wq_w; p.width[1] = d.wk_w; p.width[2] = d.wc_w; p.width[3] = d.wg_w;
  p.K = d.H; p.wtot = d.wtot; p.wpad = proj_packed_width(d); p.dst = ws.wpack;
  p.blocks = (int)(((int64_t)p.K * (p.wpad / 8) + 255) / 256);
  return p;
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
  if (short_gemm_ok(M, d.wtot, proj_short_tiles(d))) { launch_short_proj(d, w, x, M, ws, cache, slots, max_len, rope_by_token, fold, st); return; }
  if (proj_direct_big(d)) {
    launch_stream(proj_stream_kernel<128, false>, ProjStream{{}, a, nullptr, 0}, M, d.wtot, st);
  } else if (proj_packed_ok(d)) {
    const bf16 *wpack = (const bf16 *)ws.wpack;   // filled by the setup launch (pack_of)
    const int wpad = proj_packed_width(d);
    if (d.dh == 64) launch_stream(proj_stream_kernel<64, true>, ProjStream{{}, a, wpack, wpad}, M, wpad, st);
    else launch_stream(proj_stream_kernel<128, true>, ProjStream{{}, a, wpack, wpad}, M, wpad, st);
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
  if (short_gemm_ok(M, d.nh * d.dh, short_tiles(d.dl, decoder_streams(d)))) { launch_short_decoder(d, L, wp, g, out, M, st); return; }
  if (decoder_streams(d)) {
    launch_stream(d.gate == kGateOff ? decoder_stream_kernel<kGateOff> : d.gate == kGateSigmoid ? decoder_stream_kernel<kGateSigmoid>
                  : decoder_stream_kernel<-1>, DecoderStream{{}, a}, M, d.nh * 128, st);
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
  const bool stream = N % 256 == 0 && K % 128 == 0 && K >= 256;
  if (short_gemm_ok(M, N, short_tiles(K, stream))) { launch_short_plain(A, lda, M, N, K, B, C, st); return; }
  if (stream) launch_stream(plain_stream_kernel, PlainStream{{}, a}, M, N, st);
  else launch<TileHead>(plain_gemm_kernel<TileHead>, a, (N / 128) * ((M + 255) / 256), st);
}

}  // namespace gta
