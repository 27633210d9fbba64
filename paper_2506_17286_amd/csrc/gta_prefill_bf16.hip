// bf16 MFMA causal prefill attention of GTA for gfx950 (paper Sec. 3.3, reformulated form):
// for every map group g, L_g = Softmax(Q_g K_{k(g)}^T / sqrt(d_h)) C_{c(g)}, one shared map per
// group, output width d_l (normalised, bf16).  The value decoder runs afterwards as a GEMM.
//
// One workgroup = 128 queries of one (sequence, group) x up to 256 latent columns; each of its 4 waves owns 32 queries
// and the whole column slice (128 accumulator registers): the softmax statistics of a query live
// in one lane pair and nothing is exchanged between waves.  Two workgroups share a CU (two waves per SIMD, so one
// wave's softmax runs in the shadow of the other's MFMAs) and are out of step, so that the prologue and the epilogue of
// one, and the steps in which it waits at its barrier, are filled by the other; measured against one workgroup of
// eight waves and 256 queries: fused kernel of 4 x 4096 tokens with heads of 64 300 -> 270 us, ragged batch of 112 K
// tokens 18.9 -> 17.95 ms, 4 x 4096 tokens of the 1B shape 231 -> 225 us (whole calls 780 -> 760, 25.1 -> 24.0 ms, 509
// -> 503).  Heads of 64 and latent tiles of 128 take 168 registers, and three workgroups share a CU: with the fused decoder
// below, 32 x 2048 tokens of 5 maps 316 -> 238 us (two, decoder operands through registers and L through LDS: its epilogue alone took
// 105), 8 x 800 34 -> 26, 768 wide layer 16 x 1000 42 -> 33.  Wider latents are covered by several workgroups that each
// recompute the scores.
// Both products are computed transposed:
//   S^T[key][query] = K . Q^T      (row operand: K tile from LDS, column operand: the wave's queries,
//                                   held in 32 registers for the whole kernel)
//   L^T[col][query] += C^T . P^T   (row operand: latent tile through the LDS transpose read,
//                                   column operand: P straight from the S^T accumulator registers)
// so P never leaves registers and the per-query scale is a per-lane scalar.
//
// Online softmax runs in the log2 domain.  Around the diagonal the running maximum of a query moves
// when a block exceeds it by more than 2^8, and the factor exp2(m_old - m_new) reaches the 128
// accumulator registers in a rarely taken branch.  In the main loop (blocks entirely below the
// diagonal) the block maximum is not formed at all: probabilities are taken relative to the maximum
// the query already has, whatever their size, and only a row sum beyond 2^32 sends the wave through
// the full step (bf16 probabilities and fp32 sums carry any scale; the final division cancels it).  The lane
// pair of a query is reduced with v_permlane32_swap, P is packed with v_cvt_pk_bf16_f32 and summed with
// v_dot2_f32_bf16 (so the row sum is the sum of the rounded values the MFMA sees).
//
// Key/latent tiles of 32 rows go from memory straight into LDS (buffer_load_dwordx4 .. lds) through three stages, two of
// them ahead of their use, one barrier per step;
// measured against staging through registers and LDS writes: 7 % of the kernel at latents of 1024 and 3 % at 512 (ragged
// batch of 112 K tokens 19.6 -> 18.6 ms, 4 x 4096 tokens 238 -> 230 us).  Bound: MFMA issue, the LDS reads of the fragments (1 KiB per MFMA) and the softmax arithmetic share the cycles
// (matrix pipes busy about half of them); latents wider than a tile recompute the scores.  The finished tile is rounded
// to bf16, parked in LDS in output layout and written with 16-byte stores, 32 lanes per 512-byte row segment.
//
// Launches that would leave CUs idle split the keys of a workgroup over two times four waves, and, if that is not
// enough, over workgroups with a merge kernel (rule and figures at launch_attn).
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
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(8))) short s16x8;
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

// KS: key halves of a workgroup of 128 queries.  KS = 1: four waves walk all key tiles.  KS = 2: waves 0-3 take the even
// key tiles and waves 4-7 the odd ones, each with statistics and accumulators of its own, merged at the end: half the
// chain of key tiles per workgroup, for launches that leave CUs idle.
template <int DH_, int DLW_, int KS_ = 1>
struct AttnTile {
  static constexpr int DH = DH_, DLW = DLW_, KS = KS_, BK = 32, NDLB = DLW / 32;
  static constexpr int QW = 4, BQ = 32 * QW, NW = QW * KS, NT = 64 * NW;   // waves per key half, queries, waves, threads
  // A key / latent tile goes straight into LDS, 1 KiB per load instruction in lane order, so rows that one instruction
  // fetches cannot be padded apart; each instruction therefore fetches rows that are not read together:
  //   keys     (16 bytes per lane, 32 rows in a row): instruction a fetches rows a + K_INSTR i and lands 16 bytes
  //            further per a; every second i has its chunk halves swapped (k_sel).  8 (16) rows in a row then lie in
  //            different 16-byte columns of 128 (256) bytes.
  //   latents  (transpose read: four rows r of 64 bytes per half wave): instruction 4 b + r fetches rows 4 a + r and
  //            lands 64 bytes further per r, which puts the four rows into different 64-byte columns of 256 bytes.
  // Every fragment of a tile is then at one (keys: two) per-lane addresses plus a constant.
  static constexpr int K_ROW = DH * 2, C_ROW = DLW * 2, K_CPR = K_ROW / 16, C_CPR = C_ROW / 16;
  static constexpr int K_INSTR = BK * K_ROW / 1024, C_INSTR = BK * C_ROW / 1024, C_RPI = 1024 / C_ROW;
  static constexpr int K_PITCH = 1024 + 16, C_PITCH = 1024 + 64, C_GROUP = 4 * C_PITCH;
  static constexpr int K_BYTES = K_INSTR * K_PITCH, C_BYTES = C_INSTR / 4 * C_GROUP, TILE = K_BYTES + C_BYTES, STAGE = KS * TILE;
  // as many stages as leave room for the workgroups the registers allow on a CU: two, with latent tiles of 128 and heads of 64
  // three (32 x 2048 tokens, 5 maps, decoder fused: 246 us with four stages, 238 with three), with latent tiles of 64 four (32 x
  // 2048 tokens, 20 maps: 509 us with five stages, 482 with three)
  static constexpr int NSTAGE = 3;
  static constexpr int OUT_PITCH = DLW * 2 + 16;
  static constexpr int cmax(int a, int b) { return a > b ? a : b; }
  static constexpr int MERGE = KS == 1 ? 0 : QW * (NDLB * 16 + 2) * 256;   // the odd half's accumulators and statistics
  static constexpr int SMEM = cmax(cmax(BQ * OUT_PITCH, NSTAGE * STAGE), MERGE);
  // the hand-scheduled main loop deals 16 softmax slices over 2 * NDLB steps; others take the plain loop
  static constexpr bool PIPELINED = NDLB == 8 || NDLB == 4;
  static constexpr bool PAIRED = KS == 1 && DLW == 256;   // which workgroups share a CU is chosen (launch_tile)
  static_assert((DH == 64 || DH == 128) && (DLW == 64 || DLW == 128 || DLW == 256) && (KS == 1 || KS == 2), "tile");
  static_assert((K_INSTR >= NW && C_INSTR >= NW) || (KS == 2 && NW == 8), "load instructions of a step divide over the waves");
  static_assert(SMEM <= 160 * 1024, "LDS budget");
  __device__ static constexpr int k_sel(int i) { return K_CPR == 16 ? i & 1 : (i ^ (i >> 1)) & 1; }
  // LDS offset, inside the latent tile, of row 4 a for column 0
  __device__ static constexpr int c_row(int a) { return a / C_RPI * C_GROUP + a % C_RPI * C_ROW; }
};

enum { kRanked, kEvery, kSearched };   // AttnArgs.numbering

struct AttnArgs {
  const bf16 *q, *k, *c;     // packed [total, n_q*d_h], [total, n_k*d_h], [total, n_c*d_l]
  bf16 *L;                   // [total, n_q*d_l]
  const int32_t *cu; int per_seq;
  int nq, qpk, qpc, wq_w, wk_w, wc_w, dl, ndlc, batch;
  // query tiles of the longest sequence; bound of the levels (tile_of_rank); how workgroups get theirs (launch_tile)
  int n_qtiles, levels, numbering, spread, eighth;
  int ahead, back;           // workgroups i < ahead work as number i, the others as number back - i
  float scale_log2e;
  // fused value decoder (kernel template flag): O_i = (L_g W_{P,i}) * Sigmoid(gate) for the heads of g
  const bf16 *wp, *gate;     // [n_h, d_l, d_h]; gate pre-activations [total, n_h*d_h] or NULL (gate off)
  bf16 *out; int hpq, dh, nh;   // [total, n_h*d_h]
  int gate_kind;                // nonlinearity of the gate (kGateSigmoid, ..)
  // chunk mode (prefix != NULL): k, c are the caches [slot, max_seq, width]; the chunk's own rows are
  // already in them behind the prefix[b] rows cached before (prefix[b] < 0: sequence skipped, zero output)
  const int32_t *prefix, *slots; int max_seq;
  int32_t *seq_lens, *status; int max_batch, workgroups;   // the lengths, set by workgroups behind the others
  PageMap pm; int ps_shift;   // cache mode on a block-table layout: page_size = 1 << ps_shift, a multiple of BK
  // key range split over up to `splits` workgroups (not fused), a sequence's over as many as keep up to 2^split_shift key
  // tiles each: they write un-normalised fp32 sums pacc [split, token, n_q*d_l] and (maximum in log2 units, sum) pml [split,
  // token, n_q, column slice], merged by attn_merge_kernel.  A sequence that is not split writes its rows itself.
  // Where fewer than `splits` are used, their number is in the last one's entry, negated, in place of the sum.
  int splits, split_shift; float *pacc; float2 *pml; int64_t total;
};
// rounded up: a split of 9 tiles is ahead of a chain of 17 (1B shape, 40 tokens behind 700 rows of a slot of 4096 51.8 -> 48.3
// us, 4 x 40 60.2 -> 57.2, 40 behind 1100 of 8192 52.2 -> 50.1, 200 behind 900 of 2048 64.1 -> 62.1)
__device__ __forceinline__ int splits_of(const AttnArgs &a, int keys) { return max(min((keys + (32 << a.split_shift) - 1) >> (5 + a.split_shift), a.splits), 1); }

// The fused value decoder: the group's four heads of 64 columns one after the other (two key halves: two each).  The normalised
// tile stays in registers: its accumulators, rounded, are the column operand once the lane halves have swapped two words of
// each fragment.  A head's matrix [128, 64] goes straight into LDS, one ahead of its use (two key halves: all four at once), and a wave's
// 32 x 64 gate values through 4 KiB of its own, which then take the gated heads on their way to 16-byte stores.
template <class T>
struct FusedDecoder {
  static_assert(T::DH == 64 && T::DLW == 128, "four heads of 64 on a latent of 128 (attn_decoder_fusable)");
  static constexpr int HEADS = 4, HPW = HEADS / T::KS;          // heads of a group, of a wave
  static constexpr int W_BYTES = 128 * 128, WBUF = T::KS == 1 ? 2 : HEADS;
  static constexpr int IO_OFF = WBUF * W_BYTES, L_OFF = IO_OFF + T::NW * 4096;   // two key halves: L of the waves that merged it
  static constexpr int USED = L_OFF + (T::KS == 1 ? 0 : T::QW * 8192);
  static constexpr int SMEM = USED > T::SMEM ? USED : T::SMEM;
  static_assert(SMEM <= 160 * 1024, "LDS budget");
};

constexpr float kLazyThreshold = 8.0f;   // log2 units
constexpr float kRowSumLimit = 4294967296.0f;   // 2^32: a lane's sum of 16 probabilities that sends the wave to the full step

// maximum / sum over the lane pair (l, l + 32) that shares a query
__device__ __forceinline__ float pair_max(float v) {
  const u32x2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float pair_sum(float v) {
  const u32x2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// A scalar load, waited for in place: a vector load would make the compiler wait for every load in flight.
__device__ __forceinline__ int load_uniform(const int32_t *p) {
  int v;
  asm volatile("s_load_dword %0, %1, 0x0\n\ts_waitcnt lgkmcnt(0)" : "=s"(v) : "s"(p));
  return v;
}

__device__ __forceinline__ int wave_sum(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true);    // row_shr:1, 2, 4, 8
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, true);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, true);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, true);    // row_bcast:15, 31
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, true);
  return __builtin_amdgcn_readlane(v, 63);
}

struct QueryTile { int b, qt, start, len, prefix; };   // sequence, tile, first token, tokens, keys cached before
__device__ __forceinline__ void set_sequence(const AttnArgs &a, int b, QueryTile &t) {
  t.b = __builtin_amdgcn_readfirstlane(b);
  t.start = t.b * a.per_seq;
  t.len = a.per_seq;
  t.prefix = 0;
  if (a.cu) {   // both loads on their way at once
    u32x2 ends;
    if (a.prefix)
      asm volatile("s_load_dwordx2 %0, %2, 0x0\n\ts_load_dword %1, %3, 0x0\n\ts_waitcnt lgkmcnt(0)"
                   : "=&s"(ends), "=&s"(t.prefix) : "s"(a.cu + t.b), "s"(a.prefix + t.b));
    else asm volatile("s_load_dwordx2 %0, %1, 0x0\n\ts_waitcnt lgkmcnt(0)" : "=&s"(ends) : "s"(a.cu + t.b));
    t.start = (int)ends[0];
    t.len = (int)ends[1] - t.start;
  } else if (a.prefix) t.prefix = load_uniform(a.prefix + t.b);
}

// Query tile `u` of all sequences' tiles in the order they are started, most keys first (list scheduling needs that to
// balance the CUs), sequences in turn inside a level.  Level of tile qt: qt + tiles cached before the chunk, of which a
// sequence with n tiles behind p has p .. p + n - 1.  False: there are no more.  All lanes of the wave call this with the
// same arguments; lane i counts sequences i, i + 64, .. : G of them.
// The host knows no lengths.  With an id for every (level, sequence) up to the longest, the ids of the shorter ones'
// missing tiles fell to the same places again and again, and as ids are dealt to the XCDs and their shader engines in a
// fixed turn, some had no work: ragged batch of 112 K tokens, 16 sequences, CUs busy 0.57 of the time, 18.2 ms; with the
// tiles that exist numbered here 0.96, 13.0 ms (whole call 24.6 -> 19.6 ms; ragged chunks of 4 sequences 329 -> 306 us,
// 16 x 100..1000 tokens of the 1B shape 265 -> 257 us; sequences of one length as before).
// A lane holds its sequences in registers, so there is an end to the batch.  Beyond it tile_of_search costs a workgroup two or
// three loads; the order is worth more to chunks than the search saves (1B shape, ranked / searched: 250 x 16..150 behind
// 1..4000 770 / 848 us, 128 x 16..300 behind 1..1000 501 / 524; fresh 70 x 50..4000 3.95 / 3.99 ms, 250 x 50..1500 4.10 / 4.05).
constexpr int kRankedBatch = 256;
template <int G>
__device__ __forceinline__ bool tile_of_rank(const AttnArgs &a, int bq, int u, QueryTile &t) {
  const int lane = threadIdx.x & 63;
  int start[G], len[G], prefix[G], p[G], n[G];
#pragma unroll
  for (int j = 0; j < G; ++j) {
    const int i = 64 * j + lane;
    start[j] = len[j] = prefix[j] = p[j] = n[j] = 0;
    if (i < a.batch) {
      start[j] = a.cu ? a.cu[i] : i * a.per_seq;
      len[j] = a.cu ? a.cu[i + 1] - start[j] : a.per_seq;
      prefix[j] = a.prefix ? a.prefix[i] : 0;
      n[j] = max(min((len[j] + bq - 1) / bq, a.n_qtiles), 0);
      p[j] = max(prefix[j], 0) / bq;
    }
  }
  auto found = [&](int j, int at, int level) {
    t.b = 64 * j + at;
    t.qt = level - __builtin_amdgcn_readlane(p[j], at);
    t.start = __builtin_amdgcn_readlane(start[j], at);
    t.len = __builtin_amdgcn_readlane(len[j], at);
    t.prefix = __builtin_amdgcn_readlane(prefix[j], at);
  };
  const int pf = __builtin_amdgcn_readfirstlane(p[0]), nf = __builtin_amdgcn_readfirstlane(n[0]);
  if (G == 1 && __builtin_amdgcn_ballot_w64(lane < a.batch && (p[0] != pf || n[0] != nf)) == 0) {   // all alike
    const int lvl = u / a.batch;
    if (lvl >= nf) return false;
    found(0, u - lvl * a.batch, pf + nf - 1 - lvl);
    return true;
  }
  auto from_level = [&](int c) {   // tiles of level c and above
    int sum = 0;
#pragma unroll
    for (int j = 0; j < G; ++j) sum += max(min(p[j] + n[j] - c, n[j]), 0);
    return wave_sum(sum);
  };
  if (from_level(0) <= u) return false;
  int level = 0, above = a.levels, left = u;   // from_level(level) > u >= from_level(above) = u - left
  while (above - level > 1) {
    const int mid = (level + above) >> 1, m = from_level(mid);
    if (m > u) level = mid;
    else { above = mid; left = u - m; }
  }
#pragma unroll
  for (int j = 0; j < G; ++j) {   // which of the sequences that have a tile of this level
    const bool has = p[j] <= level && level < p[j] + n[j];
    const uint64_t mask = __builtin_amdgcn_ballot_w64(has);
    const int before = __builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0));
    const uint64_t it = __builtin_amdgcn_ballot_w64(has && before == left);
    if (it) found(j, __builtin_ctzll(it), level);
    left -= __builtin_popcountll(mask);
  }
  return true;
}

// Any number of ragged sequences: sequence b owns the ids from cu[b] / bq + b on, at least as many as it has tiles, longest
// first.  The wave narrows the batch down to the owner of `u` by a factor of 64 with every load.  False: an id too many.
// (Ranking with a walk over all offsets in each step: paper's layer 2048 x 20..200 tokens 2.82 ms, now 2.38.)
__device__ __forceinline__ bool tile_of_search(const AttnArgs &a, int bq, int u, QueryTile &t) {
  const int lane = threadIdx.x & 63;
  int b = 0;
  for (int count = a.batch; count > 1;) {
    const int step = (count + 63) >> 6, i = lane * step;
    const bool reached = i < count && a.cu[b + i] / bq + b + i <= u;
    const int k = max(__builtin_popcountll(__builtin_amdgcn_ballot_w64(reached)) - 1, 0) * step;
    b += k;
    count = min(step, count - k);
  }
  set_sequence(a, b, t);
  b = t.b;
  t.qt = min((t.len + bq - 1) / bq, a.n_qtiles) - 1 - (u - t.start / bq - b);
  return t.qt >= 0;
}

// Chunk mode: cached lengths, or the flags of skipped sequences (nothing in this or a later launch of the call reads them).
// By workgroups of their own: in the tiles' workgroups the arguments push scalars out of the registers of the main loop.  As many
// as have a thread per sequence: one for all took the launch 9 us longer at 4096 sequences (1B shape, chunks of 1 or 2 behind 30).
__device__ __forceinline__ void commit_chunk(const AttnArgs &a, int b) {
  if (b >= a.batch) return;
  const int slot = a.slots ? a.slots[b] : b, pre = a.prefix[b];
  if (slot < 0 || slot >= a.max_batch) return;
  if (pre >= 0) a.seq_lens[slot] = pre + (a.cu ? a.cu[b + 1] - a.cu[b] : a.per_seq);
  else a.status[slot] = GTA_ERR_CACHE_FULL;
}

// CHUNK: keys and latents in the caches.  Fresh prompts have a kernel without that code: in one for both they paid for it (calls of
// the paper's layers, both and now, 7 x 41..331 tokens 41.8 / 40.1 us, 32 x 20..100 68.6 / 66.0, 19 x 295 101.6 / 99.0).
template <class T, bool FUSE, bool CHUNK>
__global__ __launch_bounds__(T::NT, T::KS == 1 && T::DH == 64 && T::DLW == 128 ? 3 : 2) void attn_prefill_kernel(AttnArgs a) {
  if constexpr (!CHUNK) { a.prefix = nullptr; a.slots = nullptr; a.pm.table = nullptr; }
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, ln = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform: branches on it are scalar
  if constexpr (CHUNK)
    if ((int)blockIdx.x >= a.workgroups) { commit_chunk(a, ((int)blockIdx.x - a.workgroups) * T::NT + tid); return; }
  const int per = FUSE ? a.nq : a.nq * a.ndlc * a.splits;    // workgroups of a query tile
  int u, r;                                                  // rank of the tile, workgroup of the tile
  int id = !T::PAIRED || (int)blockIdx.x < a.ahead ? (int)blockIdx.x : a.back - (int)blockIdx.x;
  if (a.spread) {
    if (a.eighth && id < 8 * a.eighth) id = (id & 7) * a.eighth + (id >> 3);
    u = id / per; r = id % per;
  }
  else {   // eight tiles at a time, one per XCD, in turn from either end
    const int x = id & 7, at = id >> 3, round = at / per;
    r = at % per;
    u = round * 8 + (round & 1 ? 7 - x : x);
  }
  QueryTile tile;
  if (a.numbering == kEvery) {   // an id for every (level, sequence)
    const int lvl = u < a.batch ? 0 : u / a.batch;
    tile.qt = a.n_qtiles - 1 - lvl;
    if (tile.qt < 0) return;
    set_sequence(a, u - lvl * a.batch, tile);
    if (tile.qt * T::BQ >= tile.len) return;
  } else if (__builtin_expect(a.numbering == kSearched, 0)) {   // the rarer ways out of line: 4 chunks of 1200..2048 292.1 -> 291.3 us
    if (!tile_of_search(a, T::BQ, u, tile)) return;
  } else if (!(__builtin_expect(a.batch <= 64, 1) ? tile_of_rank<1>(a, T::BQ, u, tile) : tile_of_rank<kRankedBatch / 64>(a, T::BQ, u, tile))) return;
  constexpr bool ONE = FUSE && (!CHUNK || T::KS == 1);       // a workgroup per map (the main loop of the other kernel is slower with it)
  const int g = ONE ? r : r % a.nq, dlc = ONE ? 0 : r / a.nq % a.ndlc, split = ONE ? 0 : r / (a.nq * a.ndlc);
  const int64_t start = tile.start;
  const int Tb = tile.len, q0 = tile.qt * T::BQ;             // queries of this sequence, first of this tile
  const int P = CHUNK ? tile.prefix : 0;                     // keys cached before the first query
  const int kh = wave / T::QW, qw = wave % T::QW;            // key half and query rows of this wave
  const int splits = FUSE ? a.splits : a.splits == 1 || P < 0 ? 1 : splits_of(a, P + Tb);   // fused: 1
  auto stats = [&](int row) { return a.pml + (((int64_t)split * a.total + start + q0 + row) * a.nq + g) * a.ndlc + dlc; };
  if (!FUSE && split >= splits) {   // no share in the keys
    if (split == a.splits - 1 && tid < T::BQ && q0 + tid < Tb) *stats(tid) = make_float2(0.f, -(float)splits);
    return;
  }
  if (P < 0) {   // skipped sequence: zero rows
    if constexpr (FUSE) {
      const int64_t ldo = (int64_t)a.nh * a.dh;
      bf16 *Ob = a.out + (start + q0) * ldo + g * a.hpq * a.dh;
      for (int i = tid; i < T::BQ * 32; i += T::NT)
        if (q0 + i / 32 < Tb) *reinterpret_cast<u32x4 *>(Ob + (int64_t)(i / 32) * ldo + (i % 32) * 8) = u32x4{0u, 0u, 0u, 0u};
    } else {
      bf16 *Lb = a.L + (start + q0) * (int64_t)(a.nq * a.dl) + g * a.dl + dlc * T::DLW;
      for (int i = tid; i < T::BQ * (T::DLW / 8); i += T::NT)
        if (q0 + i / (T::DLW / 8) < Tb)
          *reinterpret_cast<u32x4 *>(Lb + (int64_t)(i / (T::DLW / 8)) * (a.nq * a.dl) + (i % (T::DLW / 8)) * 8) = u32x4{0u, 0u, 0u, 0u};
    }
    return;
  }
  const int Tk = P + Tb;                                     // keys of this sequence
  const int qw0 = q0 + qw * 32;                              // first query of this wave
  const int qa0 = P + qw0;                                   // its position among the keys
  const int kend = P + min(q0 + T::BQ, Tb);                  // keys [0, kend) are visible to this tile
  const int ntiles_all = (kend + T::BK - 1) / T::BK;
  const int tile0 = (int)((int64_t)ntiles_all * split / splits), tile1 = (int)((int64_t)ntiles_all * (split + 1) / splits);
  const int nsteps = (tile1 - tile0 + T::KS - 1) / T::KS;    // step t: key tiles tile0 + KS t (+ 1)
  const int kend_w = qw0 < Tb ? P + min(qw0 + 32, Tb) : 0;   // keys [0, kend_w) are visible to this wave
  int64_t krow0 = start;                                     // first key / latent row of the sequence
  int slot = 0;
  if (a.prefix) {
    slot = a.slots ? a.slots[tile.b] : tile.b;
    krow0 = a.pm.table ? 0 : (int64_t)slot * a.max_seq;      // block table: Kb / Cb are the pools, rows per tile
  }
  const int32_t *table = a.pm.table + (int64_t)__builtin_amdgcn_readfirstlane(slot) * a.pm.pages_per_slot;
  const char *Kb = reinterpret_cast<const char *>(a.k + krow0 * a.wk_w + (g / a.qpk) * T::DH);
  const char *Cb = reinterpret_cast<const char *>(a.c + krow0 * a.wc_w + (g / a.qpc) * a.dl + dlc * T::DLW);
  const unsigned wk2 = a.wk_w * 2, wc2 = a.wc_w * 2;

  // The wave's queries stay in registers for the whole kernel: the Q^T column operand of k-step ks is
  // the 16-byte chunk d = ks*16 + h*8 .. +8 of the lane's query (rows past the sequence re-read its
  // last row; their output is never written).
  bf16x8 qf[T::DH / 16];

  f32x16 acc[T::NDLB];
#pragma unroll
  for (int i = 0; i < T::NDLB; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;

  // Tile staging: this wave's load instructions of a tile are wave, wave + NW, .. of the keys and of the latents; where
  // there are fewer than waves (two tiles a step), one half of the waves loads a tile's keys, the other its latents.  Rows past the sequence read as zeros (such keys are in the future of every
  // valid query and are masked, and 0 x 0 adds nothing).
  const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char *)smem;
  constexpr int KI = T::K_INSTR >= T::NW ? T::K_INSTR / T::NW : 1, CI = T::C_INSTR >= T::NW ? T::C_INSTR / T::NW : 1;
  const int ki = wave % T::K_INSTR, ci = wave % T::C_INSTR;
  unsigned kv[KI], cv[CI];
  {
    const int i = lane / T::K_CPR;
#pragma unroll
    for (int j = 0; j < KI; ++j)
      kv[j] = (ki + T::NW * j + T::K_INSTR * i) * wk2 + ((lane % T::K_CPR) ^ (T::k_sel(i) * (T::K_CPR / 2))) * 16;
#pragma unroll
    for (int j = 0; j < CI; ++j) {
      const int q = ci + T::NW * j;
      cv[j] = (4 * (q / 4 * T::C_RPI + lane / T::C_CPR) + q % 4) * wc2 + (lane % T::C_CPR) * 16;
    }
  }
  auto k_loader = [&](int j) { return T::K_INSTR >= T::NW || wave / 4 == j; };        // KS = 2: one tile each
  auto c_loader = [&](int j) { return T::C_INSTR >= T::NW || wave / 4 == 1 - j; };
  // requests the next step: `fill` is its stage, j_next its first key
  unsigned fill = lds0;
  int j_next = tile0 * T::BK;
  const char *kp = Kb + (int64_t)j_next * wk2, *cp = Cb + (int64_t)j_next * wc2;
  auto issue = [&]() {
#pragma unroll
    for (int j = 0; j < T::KS; ++j) {
      const int j0 = j_next + j * T::BK, rows = min(Tk - j0, T::BK);   // rows < 1: past the end
      const char *kt = kp + j * T::BK * (int64_t)wk2, *ct = cp + j * T::BK * (int64_t)wc2;
      if (a.pm.table) {   // the tile's 32 rows sit in one page
        const int jt = min(j0, (Tk - 1) & ~(T::BK - 1));
        int pg = load_uniform(table + __builtin_amdgcn_readfirstlane(jt >> a.ps_shift));
        pg = (unsigned)pg >= (unsigned)a.pm.num_pages ? 0 : pg;
        const int64_t row0 = ((int64_t)pg << a.ps_shift) + (jt & (a.pm.page_size - 1));
        kt = Kb + row0 * wk2; ct = Cb + row0 * wc2;
      }
      if (k_loader(j)) {
        const u32x4 r = uniform_buffer_of(kt, rows > 0 ? (rows - 1) * wk2 + T::K_ROW : 0u);
#pragma unroll
        for (int i = 0; i < KI; ++i) load_to_lds(r, kv[i], fill + j * T::TILE + (ki + T::NW * i) * T::K_PITCH);
      }
      if (c_loader(j)) {
        const u32x4 r = uniform_buffer_of(ct, rows > 0 ? (rows - 1) * wc2 + T::C_ROW : 0u);
#pragma unroll
        for (int i = 0; i < CI; ++i) load_to_lds(r, cv[i], fill + j * T::TILE + T::K_BYTES + (ci + T::NW * i) * T::C_PITCH);
      }
    }
    j_next += T::KS * T::BK;
    kp += T::KS * T::BK * (int64_t)wk2; cp += T::KS * T::BK * (int64_t)wc2;
    fill = fill == lds0 + (T::NSTAGE - 1) * T::STAGE ? lds0 : fill + T::STAGE;
  };
  // load instructions of this wave per step; wait until at most `steps` steps of them are in flight, then meet
  constexpr int PER_STEP = (T::K_INSTR >= T::NW ? KI * T::KS : 1) + (T::C_INSTR >= T::NW ? CI * T::KS : 1);
  auto wait_meet = [&](auto steps_tag) {
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(decltype(steps_tag)::value * PER_STEP) : "memory");
  };
  // fragment addresses inside a stage (of this wave's tile)
  const int ksel = T::k_sel(ln / T::K_INSTR) * (T::K_ROW / 2);
  const int koff = kh * T::TILE + ln % T::K_INSTR * T::K_PITCH + ln / T::K_INSTR * T::K_ROW + h * 16;
  const int koff_lo = koff + ksel, koff_hi = koff - ksel;      // first, second half of a key row
  const int coff = kh * T::TILE + T::K_BYTES + ((lane & 15) >> 2) * T::C_PITCH + T::c_row(0) + h * (T::c_row(1) - T::c_row(0)) +
                   (((lane >> 4) & 1) * 16 + (lane & 3) * 4) * 2;
  auto c_frag = [&](int st, int mm, int dlb) {
    const char *p = smem + (st + coff) + T::c_row(4 * mm) + dlb * 64;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(p));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(p + T::c_row(2)));
    const s16x8 c8 = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, c8);
  };
  auto k_frag = [&](int st, int ks) {
    return *reinterpret_cast<const bf16x8 *>(smem + (st + (ks < T::DH / 32 ? koff_lo : koff_hi)) + ks * 32);
  };

  // scores S^T of one 32-key block (raw, unscaled); all key fragments are requested before the first
  // MFMA so that the chain of MFMAs pays one LDS round trip, not one per fragment
  auto scores = [&](int st, f32x16 &s) {
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = 0.f;
    bf16x8 kf[T::DH / 16];
#pragma unroll
    for (int ks = 0; ks < T::DH / 16; ++ks) kf[ks] = k_frag(st, ks);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ks = 0; ks < T::DH / 16; ++ks) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks], qf[ks], s, 0, 0, 0);
  };
  // keys after the lane's query are masked in a block that touches the diagonal
  auto mask = [&](f32x16 &s, int jb) {
    const int lim = qa0 + ln - jb;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int ko = 8 * (r >> 2) + 4 * h + (r & 3);
      s[r] = ko > lim ? -INFINITY : s[r];
    }
  };
  // softmax of one block: pn = exp2(scaled score - running maximum) as bf16 MFMA column operands
  // (k-slot i of lane half h  <->  key 16*mm + 8*(i/4) + 4*h + i%4); m_run / l_run are updated and
  // corr is the factor the accumulators still have to take before this block is added
  auto softmax = [&](const f32x16 &s, bf16x8 (&pn)[2], float &corr) {
    float bm = fmaxf(s[0], s[1]);
#pragma unroll
    for (int r = 2; r < 16; r += 2) bm = fmaxf(fmaxf(s[r], s[r + 1]), bm);   // v_max3
    const float m_cand = pair_max(bm) * a.scale_log2e;
    const float m_new = m_cand > m_run + kLazyThreshold ? fmaxf(m_run, m_cand) : m_run;
    // a query may see no key of this wave's first block (a block behind it, another wave's or workgroup's keys before it)
    const float ref = m_new > -INFINITY ? m_new : 0.f;
    corr = __builtin_amdgcn_exp2f(m_run - ref);
    m_run = m_new;
    const bf16x2 ones = {(bf16)1.0f, (bf16)1.0f};
    float ps = 0.f;
#pragma unroll
    for (int mm = 0; mm < 2; ++mm)
#pragma unroll
      for (int i = 0; i < 8; i += 2) {
        const float p0 = __builtin_amdgcn_exp2f(fmaf(s[mm * 8 + i], a.scale_log2e, -ref));
        const float p1 = __builtin_amdgcn_exp2f(fmaf(s[mm * 8 + i + 1], a.scale_log2e, -ref));
        bf16x2 pk;
        pk[0] = (bf16)p0; pk[1] = (bf16)p1;
        pn[mm][i] = pk[0]; pn[mm][i + 1] = pk[1];
        ps = __builtin_amdgcn_fdot2_f32_bf16(pk, ones, ps, false);   // the row sum uses the rounded values
      }
    l_run = fmaf(l_run, corr, ps);
  };
  // L^T += C^T . P^T, latent tile rows read through the transpose load with the same key order
  auto pv = [&](int st, const bf16x8 (&pf)[2]) {
    // key half outermost: consecutive MFMAs go to different accumulators
#pragma unroll
    for (int mm = 0; mm < 2; ++mm)
#pragma unroll
      for (int dlb = 0; dlb < T::NDLB; ++dlb)
        acc[dlb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(c_frag(st, mm, dlb), pf[mm], acc[dlb], 0, 0, 0);
  };

  // The waves of a workgroup meet at a barrier every tile and so run in phase: the overlap of softmax
  // arithmetic and MFMAs has to come from each wave's own instruction stream.  Iteration t issues the
  // score MFMAs of block t+1, then the map-times-latent MFMAs of block t with the softmax arithmetic
  // of block t+1 dealt out between them.
  // Step t reads the latents of its tile from stage t and the keys of the next from stage t + 1; the loads of step
  // t + NSTAGE - 1 go out at its start, into the stage that step t - 1 left.
  const int nb_all = (kend_w + 31) >> 5, nb_w = min(nb_all, tile1);   // this wave's blocks: tile0 + KS t + kh < nb_w
  auto blk = [&](int t) { return tile0 + T::KS * t + kh; };
  bf16x8 pf[2] = {};
  float corr = 1.f;
  issue();
  issue();
  {
    const bf16 *qg = a.q + (start + min(qw0 + ln, Tb - 1)) * a.wq_w + g * T::DH + h * 8;
#pragma unroll
    for (int ks = 0; ks < T::DH / 16; ++ks) qf[ks] = *reinterpret_cast<const bf16x8 *>(qg + ks * 16);
    // the compiler's wait for them belongs here, where it costs nothing, and not in front of their uses in the loops
#pragma unroll
    for (int ks = 0; ks < T::DH / 16; ++ks) asm volatile("" : "+v"(qf[ks]));
  }
#pragma unroll
  for (int t = 2; t < T::NSTAGE; ++t) issue();
  wait_meet(std::integral_constant<int, T::NSTAGE - 2>{});   // steps 0 and 1 have landed
  if (blk(0) < nb_w) {
    f32x16 s;
    scores(0, s);
    if (blk(0) * 32 + 31 > qa0) mask(s, blk(0) * 32);
    softmax(s, pf, corr);
    corr = 1.f;   // the accumulators are still zero
  }
  int cur = 0, nxt = T::STAGE;
  auto rotate = [&]() {
    cur = nxt;
    nxt = nxt == (T::NSTAGE - 1) * T::STAGE ? 0 : nxt + T::STAGE;
  };
  auto rescale = [&]() {
    if (__builtin_amdgcn_ballot_w64(corr != 1.f) != 0) {   // rare: the running maximum moved
#pragma unroll
      for (int i = 0; i < T::NDLB; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][r] *= corr;
    }
  };
  // Main part: steps whose next block lies below the wave's diagonal (up to t_main), and with latent tiles of 128 (DIAG) also those
  // where it touches the diagonal.  (256: the branch costs the longest chains what the diagonal gains; 16 prompts of 525..15071 tokens,
  // 8 x 128 + 1024 shape, 19.09 -> 19.18 ms; with 128 columns 1 x 500 tokens of the 1B shape 42.95 -> 42.39 us, 2 chunks of
  // 100..200 57.4 -> 56.6, 32 x 2048 tokens of the paper's layer 670 -> 662.)
  constexpr bool DIAG = T::PIPELINED && T::NDLB == 4;
  int t = 0;
  if constexpr (T::PIPELINED) {
  const int lim = min(nb_w, qa0 >> 5) - 1 - tile0 - kh, t_main = lim < 0 ? 0 : lim / T::KS;
#pragma unroll 1
  for (; DIAG ? blk(t + 1) < nb_w : t < t_main; ++t) {
    // The fragment reads of the first score MFMAs and of the first two map-times-latent MFMAs go out
    // before anything else, so that the MFMAs below do not each wait for an LDS round trip; the second
    // half of the key fragments follows behind the first two score MFMAs.
    constexpr int KS = T::DH / 16, KS1 = KS / 2;
    bf16x8 kf[KS];
#pragma unroll
    for (int ks = 0; ks < KS1; ++ks) kf[ks] = k_frag(nxt, ks);
    __builtin_amdgcn_sched_barrier(0);
    if (t > 0) issue();
    rescale();
    f32x16 s;
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = 0.f;
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      if (ks == 1) {
#pragma unroll
        for (int k2 = KS1; k2 < KS; ++k2) kf[k2] = k_frag(nxt, k2);
      }
      s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks], qf[ks], s, 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (DIAG && t >= t_main) mask(s, blk(t + 1) * 32);
    // 2 * NDLB steps, each one MFMA of block t (latent fragment i, read two steps earlier), the
    // transpose reads of fragment i+2 and a slice of the softmax arithmetic of block t+1 (16 slices
    // dealt evenly over the steps); the scheduling barrier after every step pins this order, so each
    // MFMA is followed by arithmetic that runs in its shadow
    constexpr int NS = 2 * T::NDLB, SPS = 16 / NS;   // steps, softmax slices per step
    auto cread = [&](int i) { return c_frag(cur, i / T::NDLB, i % T::NDLB); };
    constexpr int LA = 3;   // latent fragments in flight ahead of their MFMA
    bf16x8 cf[NS + LA], pn[2];
#pragma unroll
    for (int i = 0; i < LA; ++i) cf[i] = cread(i);
    // Below the diagonal the running maximum is left where it is and the block's own maximum is not
    // even formed: p = exp2(score - m_run) is taken as it comes and only its row sum is watched.  bf16
    // probabilities and fp32 sums carry any scale, so nothing is lost while p stays far from the top
    // of the fp32 range; a block whose row sum passes 2^32 (or is not finite) sends the whole wave
    // through the full online-softmax step once, which moves the maximum and redoes the block.
    float ps = 0.f;
    const float negm = -m_run;
    const bf16x2 ones = {(bf16)1.0f, (bf16)1.0f};
    auto soft_slice = [&](int k) {   // 16 slots; the 8 pairs of exponentials take the even ones
      if (k % 2 == 0) {
        const int e = k;   // elements e, e+1 -> k-slots e%8, e%8+1 of pn[e/8]
        const float p0 = __builtin_amdgcn_exp2f(fmaf(s[e], a.scale_log2e, negm));
        const float p1 = __builtin_amdgcn_exp2f(fmaf(s[e + 1], a.scale_log2e, negm));
        bf16x2 pk;
        pk[0] = (bf16)p0; pk[1] = (bf16)p1;
        pn[e >> 3][e & 7] = pk[0]; pn[e >> 3][(e & 7) + 1] = pk[1];
        ps = __builtin_amdgcn_fdot2_f32_bf16(pk, ones, ps, false);
      }
    };
#pragma unroll
    for (int i = 0; i < NS; ++i) {
      if (i + LA < NS) cf[i + LA] = cread(i + LA);
      acc[i % T::NDLB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(cf[i], pf[i / T::NDLB], acc[i % T::NDLB], 0, 0, 0);
#pragma unroll
      for (int k = i * SPS; k < (i + 1) * SPS; ++k) soft_slice(k);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (__builtin_amdgcn_ballot_w64(!(ps < kRowSumLimit)) != 0) {   // rare
      softmax(s, pn, corr);
    } else {
      l_run += ps;
      corr = 1.f;
    }
    pf[0] = pn[0]; pf[1] = pn[1];
    wait_meet(std::integral_constant<int, T::NSTAGE - 3>{});
    rotate();
  }
  }
  // the blocks that the loop above leaves (the last one has no next), then idle steps that only keep staging for the other waves
#pragma unroll 1
  for (; t < nsteps; ++t) {
    if (t > 0) issue();
    if (blk(t) < nb_w) {
      rescale();
      if constexpr (DIAG) {
        pv(cur, pf);
        corr = 1.f;
      } else {
        f32x16 s;
        bf16x8 pn[2];
        if (blk(t + 1) < nb_w) {
          scores(nxt, s);
          if (blk(t + 1) * 32 + 31 > qa0) mask(s, blk(t + 1) * 32);
        } else {   // no further block: all-masked scores leave the statistics unchanged and give P = 0
#pragma unroll
          for (int r = 0; r < 16; ++r) s[r] = -INFINITY;
        }
        softmax(s, pn, corr);
        pv(cur, pf);
        pf[0] = pn[0]; pf[1] = pn[1];
      }
    }
    wait_meet(std::integral_constant<int, T::NSTAGE - 3>{});
    rotate();
  }
  asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");   // no load may land in what follows

  float l_all = pair_sum(l_run);
  if constexpr (T::KS == 2) {
    // ---- the odd half's sums join the even half's: register r of lane i of wave w at (w, r, i).  A query whose keys
    // all lie in one half gets weight 0 from the other (maximum -inf).
    float *mg = reinterpret_cast<float *>(smem) + qw * (T::NDLB * 16 + 2) * 64 + lane;
    if (kh == 1) {
#pragma unroll
      for (int dlb = 0; dlb < T::NDLB; ++dlb)
#pragma unroll
        for (int r = 0; r < 16; ++r) mg[(dlb * 16 + r) * 64] = acc[dlb][r];
      mg[T::NDLB * 16 * 64] = m_run; mg[(T::NDLB * 16 + 1) * 64] = l_all;
    }
    __syncthreads();
    if (kh == 0) {
      const float mo = mg[T::NDLB * 16 * 64], lo = mg[(T::NDLB * 16 + 1) * 64], mx = fmaxf(m_run, mo);
      const float ref = mx > -INFINITY ? mx : 0.f;
      const float se = __builtin_amdgcn_exp2f(m_run - ref), so = __builtin_amdgcn_exp2f(mo - ref);
      l_all = l_all * se + lo * so;
      m_run = mx;
#pragma unroll
      for (int dlb = 0; dlb < T::NDLB; ++dlb)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[dlb][r] = acc[dlb][r] * se + mg[(dlb * 16 + r) * 64] * so;
    }
    __syncthreads();
  }
  if (!FUSE && splits > 1) {   // un-normalised sums and statistics for the merge
    const int row = qw * 32 + ln;
    if (kh == 0 && q0 + row < Tb) {
      float *pa = a.pacc + ((int64_t)split * a.total + start + q0 + row) * (a.nq * a.dl) + g * a.dl + dlc * T::DLW + 4 * h;
#pragma unroll
      for (int dlb = 0; dlb < T::NDLB; ++dlb)
#pragma unroll
        for (int rq = 0; rq < 4; ++rq)
          *reinterpret_cast<float4 *>(pa + dlb * 32 + rq * 8) =
              make_float4(acc[dlb][rq * 4], acc[dlb][rq * 4 + 1], acc[dlb][rq * 4 + 2], acc[dlb][rq * 4 + 3]);
      if (h == 0) *stats(row) = make_float2(m_run, l_all);
    }
    return;
  }

  if constexpr (FUSE) {
    // ---- value decoder on the tile (Sec. 3.2): the workgroup holds the whole latent width of its
    // group, so the heads of the group are finished here and L never goes to memory
    typedef FusedDecoder<T> F;
    const int head0 = g * a.hpq;
    const unsigned ldo = (unsigned)(a.nh * a.dh * 2);
    // this wave's heads; its rows of the gate and of the output, 8 lanes a row; rows past the sequence are beyond the buffers
    auto head_of = [&](int i) { return head0 + kh * F::HPW + i; };
    const int rows = min(Tb - qw0, 32);
    const unsigned row_bytes = rows > 0 ? (rows - 1) * ldo + 128u : 0u, io_off = (lane >> 3) * ldo + (lane & 7) * 16;
    auto rows_of = [&](const bf16 *p, int i) {
      return __builtin_amdgcn_make_buffer_rsrc((void *)(p + (start + qw0) * (int64_t)(a.nh * a.dh) + head_of(i) * 64), 0, row_bytes, 0x00020000);
    };
    u32x4 gt[2][4];
    auto ask_gate = [&](int i) {
      const __amdgpu_buffer_rsrc_t r = rows_of(a.gate, i);
#pragma unroll
      for (int j = 0; j < 4; ++j) gt[i % 2][j] = __builtin_amdgcn_raw_buffer_load_b128(r, io_off + j * 8 * ldo, 0, 0);
    };
    // matrix of head w of the group: 16 loads of 8 rows; 64-byte halves of a row swapped where bit 1 of the row is set, so that the
    // four rows of a transpose read lie in different 64-byte columns of 256 bytes
    const unsigned wv = (lane >> 3) * 128 + ((((lane & 7) >> 2) ^ ((lane >> 4) & 1)) * 4 + (lane & 3)) * 16;
    auto load_w = [&](int w) {
      const u32x4 r = uniform_buffer_of(a.wp + (int64_t)(head0 + w) * 128 * 64, F::W_BYTES);
#pragma unroll
      for (int j = 0; j < 16 / T::NW; ++j)
        load_to_lds(r, wv + (wave * (16 / T::NW) + j) * 1024, lds0 + w % F::WBUF * F::W_BYTES + (wave * (16 / T::NW) + j) * 1024);
    };
    constexpr int GATE = 4, STORES = 4;   // instructions of a wave and head
    auto request = [&](int w, bool gate) {   // in this order: the waits below count what is younger than a matrix
      load_w(w);
      asm volatile("" ::: "memory");
      if (gate && a.gate) ask_gate(w);
      asm volatile("" ::: "memory");
    };
#pragma unroll
    for (int w = 0; w < F::WBUF; ++w) request(w, w < 2);
    bf16x8 lf[8];
    if (kh == 0) {
      const float inv = 1.0f / l_all;
#pragma unroll
      for (int mm = 0; mm < 8; ++mm)
#pragma unroll
        for (int i = 0; i < 8; ++i) lf[mm][i] = (bf16)(acc[mm / 2][mm % 2 * 8 + i] * inv);
      // i holds column 16 mm + 8 (i/4) + 4 h + i%4 so far.  Swapped across the lane halves it is column 16 mm + 8 h + i, the order in
      // which the decoder's own kernels add up, and the results are theirs bit for bit.
#pragma unroll
      for (int mm = 0; mm < 8; ++mm) {
        u32x4 v = __builtin_bit_cast(u32x4, lf[mm]);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const u32x2 r = __builtin_amdgcn_permlane32_swap(v[i], v[i + 2], false, false);
          v[i] = r[0]; v[i + 2] = r[1];
        }
        lf[mm] = __builtin_bit_cast(bf16x8, u32x4{v[0], v[1], v[2], v[3]});
      }
    }
    if constexpr (T::KS == 2) {
      bf16x8 *lx = reinterpret_cast<bf16x8 *>(smem + F::L_OFF + qw * 8192) + lane;
      if (kh == 0) {
#pragma unroll
        for (int mm = 0; mm < 8; ++mm) lx[mm * 64] = lf[mm];
      }
      __syncthreads();
      if (kh == 1) {
#pragma unroll
        for (int mm = 0; mm < 8; ++mm) lf[mm] = lx[mm * 64];
      }
    }
    const int wrow = (lane & 15) >> 2;
    const int wfr = (8 * h + wrow) * 128 + ((lane >> 4) & 1) * 32 + (lane & 3) * 8, wsw = (wrow >> 1) * 64;
    char *io = smem + F::IO_OFF + wave * 4096;
#pragma unroll
    for (int i = 0; i < F::HPW; ++i) {
      // this head's matrix has landed (younger than it: gate values of one head and the stores of the last; before the first head
      // the next one's matrix and the gates of both); everyone has read the one before it
      if constexpr (T::KS == 2) {
        if (i == 0) asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
      } else if (i == 0) {
        if (a.gate) asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(2 * GATE + 16 / T::NW) : "memory");
        else asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(16 / T::NW) : "memory");
      } else {
        if (a.gate) asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(GATE + STORES) : "memory");
        else asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(STORES) : "memory");
      }
      if (T::KS == 1 && i > 0 && i + 1 < F::HPW) request(i + 1, true);
      f32x16 z[2];
#pragma unroll
      for (int tn = 0; tn < 2; ++tn)
#pragma unroll
        for (int r = 0; r < 16; ++r) z[tn][r] = 0.f;
      const char *wb = smem + (T::KS == 1 ? i % F::WBUF : kh * F::HPW + i) * F::W_BYTES + wfr;
#pragma unroll
      for (int mm = 0; mm < 8; ++mm)
#pragma unroll
        for (int tn = 0; tn < 2; ++tn) {
          const char *wp = wb + mm * 16 * 128 + (tn * 64 ^ wsw);
          const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(wp));
          const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(wp + 4 * 128));
          const s16x8 w8 = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
          z[tn] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, w8), lf[mm], z[tn], 0, 0, 0);
        }
      // chunk c of row r in slot c ^ (r % 8); lane: row ln, columns tn*32 + rq*8 + 4h .. +3
      if (a.gate) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int r = j * 8 + (lane >> 3);
          *reinterpret_cast<u32x4 *>(io + r * 128 + (((lane & 7) ^ (r & 7)) << 4)) = gt[i % 2][j];
        }
      }
      auto finish = [&](auto factor) {
#pragma unroll
        for (int tn = 0; tn < 2; ++tn)
#pragma unroll
          for (int rq = 0; rq < 4; ++rq) {
            bf16x4 *slot = reinterpret_cast<bf16x4 *>(io + ln * 128 + (((tn * 4 + rq) ^ (ln & 7)) << 4) + h * 8);
            const bf16x4 gz = *slot;
            bf16x4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = (bf16)(z[tn][rq * 4 + e] * factor((float)gz[e]));
            *slot = o;
          }
      };
      if (!a.gate) finish([](float) { return 1.f; });
      else if (a.gate_kind == kGateSigmoid) finish([](float x) { return gate_factor(kGateSigmoid, x); });
      else finish([&](float x) { return gate_factor(a.gate_kind, x); });
      const __amdgpu_buffer_rsrc_t ro = rows_of(a.out, i);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int r = j * 8 + (lane >> 3);
        __builtin_amdgcn_raw_buffer_store_b128(*reinterpret_cast<const u32x4 *>(io + r * 128 + (((lane & 7) ^ (r & 7)) << 4)), ro, io_off + j * 8 * ldo, 0, 0);
      }
    }
    return;
  }

  // ---- normalise, park the tile in LDS in output layout, write row-contiguous 16-byte chunks
  if (kh == 0) {
    const float inv = 1.0f / l_all;
    const int row = qw * 32 + ln;
#pragma unroll
    for (int dlb = 0; dlb < T::NDLB; ++dlb)
#pragma unroll
      for (int rq = 0; rq < 4; ++rq) {
        bf16x4 v;
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = (bf16)(acc[dlb][rq * 4 + i] * inv);
        *reinterpret_cast<bf16x4 *>(smem + row * T::OUT_PITCH + (dlb * 32 + rq * 8 + 4 * h) * 2) = v;
      }
  }
  __syncthreads();
  bf16 *Lb = a.L + (start + q0) * (int64_t)(a.nq * a.dl) + g * a.dl + dlc * T::DLW;
  constexpr int CPR = T::DLW / 8, RPP = T::NT / CPR;   // 16-byte chunks per output row, rows per pass
  const int r0 = tid / CPR, ch = tid % CPR;
#pragma unroll 4
  for (int it = 0; it < T::BQ / RPP; ++it) {
    const int r = it * RPP + r0;
    if (q0 + r < Tb)
      *reinterpret_cast<u32x4 *>(Lb + (int64_t)r * (a.nq * a.dl) + ch * 8) =
          *reinterpret_cast<const u32x4 *>(smem + r * T::OUT_PITCH + ch * 16);
  }
}

// Merge of the key splits of one token (blockIdx.x): thread = 4 columns of one map group; weights exp2(m_s - max) / sum.
__global__ __launch_bounds__(256) void attn_merge_kernel(AttnArgs a, int dlw) {
  const int64_t tok = blockIdx.x;
  const int nq = a.nq, dl = a.dl;
  for (int i = threadIdx.x; i < nq * dl / 4; i += 256) {
    const int col = i * 4, st = col / dl * a.ndlc + col % dl / dlw;
    auto stats = [&](int s) { return a.pml[(s * a.total + tok) * (nq * a.ndlc) + st]; };
    constexpr int U = 4;   // requested beside the last, before it is known whether they are used
    const float2 last = stats(a.splits - 1);
    float2 first[U];
#pragma unroll
    for (int s = 0; s < U; ++s) first[s] = stats(min(s, a.splits - 1));
    const int splits = last.y < 0.f ? (int)-last.y : a.splits;
    if (splits == 1) continue;   // written already
    float mx = -INFINITY;
#pragma unroll
    for (int s = 0; s < U; ++s) mx = s < splits ? fmaxf(mx, first[s].x) : mx;
    for (int s = U; s < splits; ++s) mx = fmaxf(mx, stats(s).x);
    const float ref = mx > -INFINITY ? mx : 0.f;
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    float ls = 0.f;
    for (int s = 0; s < splits; ++s) {
      const float2 ml = stats(s);
      if (ml.y != 0.f) {   // a split without visible keys has the sum 0; one of nothing but NaN has no maximum either
        const float w = __builtin_amdgcn_exp2f(ml.x - ref);
        const float4 p = *reinterpret_cast<const float4 *>(a.pacc + (s * a.total + tok) * (int64_t)(nq * dl) + col);
        ls = fmaf(w, ml.y, ls);
        v.x = fmaf(w, p.x, v.x); v.y = fmaf(w, p.y, v.y); v.z = fmaf(w, p.z, v.z); v.w = fmaf(w, p.w, v.w);
      }
    }
    const float inv = 1.0f / ls;
    bf16x4 o;
    o[0] = (bf16)(v.x * inv); o[1] = (bf16)(v.y * inv); o[2] = (bf16)(v.z * inv); o[3] = (bf16)(v.w * inv);
    *reinterpret_cast<bf16x4 *>(a.L + tok * (nq * dl) + col) = o;
  }
}

// latent columns per workgroup
int latent_tile(const Dims &d) { return d.dh == 128 ? (d.dl % 256 == 0 ? 256 : 128) : (d.dl % 128 == 0 ? 128 : 64); }

// From this many query tiles on a tile's workgroups stay on one XCD (they read the same keys and latents); fewer would
// leave XCDs idle or unevenly loaded, and their workgroups go to the XCDs in turn: 1 x 4000 tokens of 8 maps and 4 column
// slices (32 tiles) 454 us on one XCD each, 447 in turn; 1 x 500 of the 1B shape (4) 48.6 / 48.3; from 64 tiles on equal.
constexpr int kSpreadTiles = 64;

template <class T, bool FUSE>
void launch_tile(AttnArgs a, const Dims &d, int batch, int max_len, hipStream_t st) {
  a.n_qtiles = ((a.cu ? max_len : std::min(max_len, a.per_seq)) + T::BQ - 1) / T::BQ;
  a.ndlc = d.dl / T::DLW;
  a.levels = a.n_qtiles + (a.prefix ? a.max_seq / T::BQ : 0) + 1;
  // ids for every (level, sequence), and no more than this many query tiles whatever the lengths are
  const int64_t every = (int64_t)a.n_qtiles * batch;
  int64_t tiles = std::min(every, a.total / T::BQ + batch);
  // Where the chip holds every (level, sequence) at once, two workgroups of four waves or one of eight on a CU, the order means nothing
  // and tiles need no ranks: ragged calls, with and without ranks, paper's layer 7 x 41..331 tokens 53.4 / 53.1 us, 8 x 10..80
  // 32.7 / 32.6, 1B shape 4 x 10..40 behind 6000 67.3 / 66.5.  Heads of 64 with latent tiles of 128 have three workgroups of four waves on
  // a CU, but there the missing tiles of 513 to 768 ids cost more than the ranks (60 x 25..250 91.9 / 95.7, 20 x 80..800 102.3 /
  // 105.2, 18 x 100..1000 behind 3000 202 / 218, one length level).
  const bool fits = every * a.nq * a.ndlc * a.splits <= 512 / T::KS, at_once = batch > 1 && fits;
  // Nor do fresh prompts of one tile each or of one length: 4096 x 32 tokens of the 1B shape 4.46 -> 2.57 ms, 4096 x 2..16 behind 100
  // rows, paper's layer, 2.57 -> 1.12 (ranked with a walk over all offsets).  With offsets the lengths show in ids that are no more than
  // the bound (256 x 129 of the paper's layer with two latents 535 -> 525 us; a batch of one wave's lanes looks at them itself).  Where a
  // batch is too large to rank, ids that few tiles are missing from cost less than the search: 768 wide layer 300 x 20..200 (600 ids, bound
  // 558) 224.8 / 214.2 us, paper's layer 512 chunks of 20..200 (1.14 times the bound) 799 / 782, 300 x 20..130 (1.26) 287 / 273, equal
  // at 260 x 100..1000 (1.6).
  if (at_once || (!a.prefix && (!a.cu || a.n_qtiles == 1 || (batch > 64 && every == tiles))) ||
      (batch > kRankedBatch && 5 * every <= 8 * tiles)) {
    a.numbering = kEvery;
    tiles = every;
  } else a.numbering = batch <= kRankedBatch ? kRanked : kSearched;
  // One tile per sequence: the workgroups of a tile read the same rows.  Where the chip holds them all, an XCD takes an eighth of
  // the workgroups in a row (1B shape, in turn / eighths: 8 x 100 behind 4000 89.8 / 84.1 us, 3 x 100 70.3 / 68.1, 64 x 128 fresh 169.7
  // / 165.8).  Chunks beyond that are ranked by the rows they read, and eighths would give one XCD the longest: from 16 tiles on they are
  // dealt like many tiles (eighths / in turn / dealt: 1B shape 40 x 10..100 behind 1..3000 202 / 154 / 148 us, of one length 244 / 256 /
  // 240; 8 x 128 + 1024 shape 20 x 10..100 behind 1..4000 347 / 260 / 239, of one length 303 / 306 / 307), fewer in turn (12 x 10..100
  // behind 1..4000 249 / 181 / 180, of one length 225 / 228 / 233).
  a.spread = at_once || tiles < (a.prefix && a.n_qtiles == 1 ? 16 : kSpreadTiles);
  a.eighth = fits && a.n_qtiles == 1 ? (int)(tiles * a.nq * a.ndlc * a.splits / 8) : 0;
  if (!a.spread) tiles = (tiles + 7) / 8 * 8;
  int smem = T::SMEM;
  if constexpr (FUSE) smem = FusedDecoder<T>::SMEM;
  a.workgroups = (int)(tiles * a.ndlc * d.nq * a.splits);
  // Two workgroups of four waves share a CU: where the chip holds all of them, those behind the first 256 go backwards, so that the
  // longest shares its CU with the shortest of them (a tile's workgroups stay on one XCD): 1B shape 6 x 1100 172 -> 164 us, 7 x
  // 200..1000 113 -> 109, 8 x 1000 183 -> 180.  Not with narrower latent tiles (16 x 700 of the paper's layer 121.7 / 121.0, 8 x 100,
  // which has too few for it, 39.7 / 39.9).
  a.ahead = a.workgroups <= 512 ? 256 : a.workgroups;
  a.back = 255 + a.workgroups;
  auto launch = [&](auto kernel, int more) {
    allow_dynamic_lds((const void *)kernel, smem);
    kernel<<<(unsigned)(a.workgroups + more), T::NT, smem, st>>>(a);
  };
  if (a.prefix) launch(attn_prefill_kernel<T, FUSE, true>, (batch + T::NT - 1) / T::NT);
  else launch(attn_prefill_kernel<T, FUSE, false>, 0);
}

constexpr int kSplitTarget = 256;   // workgroups of 128 queries a launch with key splits aims at: one per CU

// Key splits of a launch of `half` workgroups in key halves (rule and figures at launch_attn).
int key_splits(const AttnArgs &a, int64_t half, int max_keys) {
  const int64_t most = (int64_t)(max_keys + 31) / 32 >> (a.prefix ? 4 : 5), n = std::min(kSplitTarget / half, most);
  return n < 1 ? 1 : (int)n;
}
int64_t half_workgroups(const Dims &d, int batch, int max_len, int dlw) { return (int64_t)((max_len + 127) / 128) * batch * d.nq * (d.dl / dlw); }

// max_keys: host bound of a sequence's keys.  part: scratch for key splits (attn_split_bytes) or NULL.
template <int DH, int DLW, bool FUSE>
void launch_attn(AttnArgs a, const Dims &d, int batch, int max_len, int max_keys, float *part, hipStream_t st) {
  // Workgroups of 128 queries, all keys walked by four waves, two workgroups per CU (heads of 64 and latent tiles of 128: three, for
  // which the lines lie in the same places).  Launches whose workgroups would all be on the chip at once (512) only wait for the longest chain of key tiles; there eight waves share a workgroup's
  // queries in two key halves: half the chain, at 2 us of merge and one workgroup per CU.  Measured whole calls, one
  // half against two, 1B shape: fresh 1 x 2000 127 against 122 us, 1 x 8192 404 / 360 (512 workgroups), 2 x 4096 281 /
  // 267 (512), 2 x 3000 ragged 213 / 197 (384), 3 x 4000 373 / 398 (768); chunks 8 x 300 behind 4000 189 / 172 (192),
  // 8 x 600 behind 4000 290 / 291 (320), 5 x 2000 ragged behind 5000 389 / 421 (640); paper's layer 1 x 8000 224 / 182 (320), 4 x 2048
  // 120 / 109 (320), 5 x 2000 143 / 138 (400), 6 x 2000 151 / 151 (480), of 200..2000 119 / 108, chunks 20 x 30..300 behind 2000 109 / 101
  // (300), of one length 125 / 145.  Up to 1024 keys the chain is too short for more than one round of the two halves: 8 x 1000
  // 191 / 196 (512), paper's layer 10 x 1000 126 / 130 (400), 16 x 700 128 / 136 (480), but 2 x 1000 75 / 70 (80); up to 256 keys it
  // gains little or nothing: paper's layer 1 x 128 26.4 / 26.4, 1 x 256 36.0 / 35.1, 1B shape 1 x 128 40.7 / 42.2.
  const int64_t half = half_workgroups(d, batch, max_len, DLW);
  a.splits = 1;
  // Fresh prompts of one length whose workgroups nearly fill the chip keep one half, the longest paired with the shortest on a CU
  // (launch_tile): 1B shape, two halves / one, 3 prompts 3 x 1900 173.2 / 177.0 us (360 workgroups), 3 x 2000 183.1 / 183.5 (384), 3 x
  // 2300 199.1 / 198.1 (432), 3 x 2600 226.5 / 220.9 (504); 4 x 1400 162.2 / 164.5 (352), 4 x 1600 180.3 / 177.9 (416), 4 x 2000 212.6 /
  // 203.9 (512); 5 x 1500 197.2 / 187.5 (480); 6 x 1100 174.8 / 165.6 (432).  Two prompts are ahead only from 480 on (2 x 3500 230.4 /
  // 233.5, 448; 2 x 4000 261.5 / 258.1), one never (1 x 8000 353.6 / 361.3).  Chunks of one length gain as much behind equal caches (8 x 600
  // behind 4000 315 / 271) and lose behind unequal ones, which the host does not see (behind 200..4000 226 / 246).
  const bool alike = DLW == 256 && !a.prefix && batch > 2 && a.total == (int64_t)batch * max_len && half > 384;
  if (half > 512 || max_keys <= 256 || (half > 256 && max_keys <= 1024) || alike) {
    launch_tile<AttnTile<DH, DLW, 1>, FUSE>(a, d, batch, max_len, st);
    return;
  }
  if (!FUSE && part) {
    // Still fewer workgroups than CUs: the key range is split over workgroups, too, as long as a split keeps 8 steps
    // of two tiles (16 for a fresh prompt, whose average tile is half as long).  1 x 40 behind 6000 145 us without,
    // 80 with up to 23 splits, 67 with 11; 4 x 40 behind 6000 153 / 76; 1 x 2000 fresh 124 / 120.  max_keys is only the
    // capacity of the slots: the kernels count a sequence's own keys (splits_of).
    a.split_shift = a.prefix ? 4 : 5;
    a.splits = key_splits(a, half, max_keys);
    const int64_t stats = a.total * d.nq * (d.dl / DLW) * 2;   // floats per split
    while (a.splits > 1 && (size_t)(a.splits * (stats + a.total * d.nq * d.dl) + 64) * 4 > attn_split_bytes(d)) --a.splits;
    a.pml = reinterpret_cast<float2 *>(part);
    a.pacc = part + ((a.splits * stats + 63) & ~(int64_t)63);
  }
  a.ndlc = d.dl / DLW;
  launch_tile<AttnTile<DH, DLW, 2>, FUSE>(a, d, batch, max_len, st);
  if (a.splits > 1)
    attn_merge_kernel<<<(unsigned)a.total, 256, 0, st>>>(a, DLW);
}

template <bool FUSE>
void launch_attn_any(const AttnArgs &a, const Dims &d, int batch, int max_len, int max_keys, float *part, hipStream_t st) {
  if constexpr (FUSE) { launch_attn<64, 128, true>(a, d, batch, max_len, max_keys, part, st); return; }
  const int dlw = latent_tile(d);
  // Tiles of 128 latent columns recompute the scores twice as often as tiles of 256, a third more matrix work at latents of
  // 512, but where the chip has room for twice the workgroups the chain of key steps that the call waits for has a third less
  // in it.  Whole calls, 256 against 128 columns (workgroups of 256): 1B shape fresh 1 x 500 47.2 / 43.7 us (32), 1 x 1000
  // 64.0 / 58.4 (64), 1 x 2000 110.6 / 100.7 (128), 1 x 3000 136 / 126 (192), 2 x 1500 ragged 121 / 115 (192), 1 x 4000 167.9 /
  // 165.9 (256), 24 x 128 97.0 / 97.5 (192); 8 x 128 + 1024 shape 1 x 512 76.5 / 72.6 (128), 1 x 1000 129.2 / 130.3 (256).
  // Chunks, whose chains are alike: 40 behind 6000 62.0 / 57.6 (88), 300 behind 1000 63.1 / 57.1, 2 x 500 behind 4000 91.1 /
  // 95.0 (256), 3 x 700 behind 4000 167 / 211 (144).
  const int64_t wide = dlw == 256 ? half_workgroups(d, batch, max_len, 256) : 0;
  if (wide && (!part || wide * key_splits(a, wide, max_keys) > (a.prefix ? 128 : 255)))
    launch_attn<128, 256, false>(a, d, batch, max_len, max_keys, part, st);
  else if (d.dh == 128) launch_attn<128, 128, false>(a, d, batch, max_len, max_keys, part, st);
  else if (dlw == 128) launch_attn<64, 128, false>(a, d, batch, max_len, max_keys, part, st);
  else launch_attn<64, 64, false>(a, d, batch, max_len, max_keys, part, st);
}

}  // namespace

// Scratch of the key splits, the same whatever the call's size (so that a workspace sized for many tokens also serves
// few): kSplitTarget workgroups of 128 rows x one latent tile, and two floats per row and tile.
size_t attn_split_bytes(const Dims &d) {
  return (size_t)kSplitTarget * 128 * (latent_tile(d) + 2) * 4 + 4096;
}

bool attn_prefill_supported(const Dims &d, int max_len) {
  // a sequence's K / C rows stay below 2 GiB: the limit the interface names for these kernels
  if ((int64_t)max_len * d.wc_w * 2 >= ((int64_t)1 << 31) || (int64_t)max_len * d.wk_w * 2 >= ((int64_t)1 << 31)) return false;
  if (d.dtype != GTA_BF16 || d.wq_w % 8 || d.wk_w % 8 || d.wc_w % 8) return false;
  return (d.dh == 128 && d.dl % 128 == 0) || (d.dh == 64 && d.dl % 64 == 0);
}

static AttnArgs attn_args(const Dims &d, const void *q, const void *k, const void *c, const int32_t *cu, int batch,
                          int64_t total) {
  AttnArgs a{};
  a.q = (const bf16 *)q; a.k = (const bf16 *)k; a.c = (const bf16 *)c;
  a.cu = cu; a.per_seq = (int)(total / batch);
  a.nq = d.nq; a.qpk = d.qpk; a.qpc = d.qpc; a.wq_w = d.wq_w; a.wk_w = d.wk_w; a.wc_w = d.wc_w; a.dl = d.dl;
  a.scale_log2e = d.scale * 1.4426950408889634f;
  a.batch = batch; a.total = total;
  return a;
}

void launch_attn_prefill_bf16(const Dims &d, const void *q, const void *k, const void *c, const int32_t *cu,
                              int batch, int64_t total, int max_len, void *L, float *part, hipStream_t st) {
  AttnArgs a = attn_args(d, q, k, c, cu, batch, total);
  a.L = (bf16 *)L;
  launch_attn_any<false>(a, d, batch, max_len, max_len, part, st);
}

// One workgroup covers the whole latent width and the group's heads fill one 256-wide tile
bool attn_decoder_fusable(const Dims &d, int max_len) {
  return attn_prefill_supported(d, max_len) && d.dh == 64 && d.dl == 128 && d.hpq * d.dh == 256;
}

void launch_attn_decoder_bf16(const Dims &d, const void *q, const void *k, const void *c, const int32_t *cu,
                              int batch, int64_t total, int max_len, const void *wp, const void *gate, void *out,
                              hipStream_t st) {
  AttnArgs a = attn_args(d, q, k, c, cu, batch, total);
  a.wp = (const bf16 *)wp; a.gate = d.gate ? (const bf16 *)gate : nullptr; a.out = (bf16 *)out;
  a.hpq = d.hpq; a.dh = d.dh; a.nh = d.nh; a.gate_kind = d.gate;
  launch_attn_any<true>(a, d, batch, max_len, max_len, nullptr, st);
}

void launch_attn_chunk_bf16(const Dims &d, const void *q, const gta_cache &cache, const int32_t *slots,
                            const int32_t *prefix, const int32_t *cu, int batch, int64_t total, int max_chunk,
                            void *L, const void *wp, const void *gate, void *out, bool fuse, float *part, hipStream_t st) {
  AttnArgs a = attn_args(d, q, cache.k, cache.c, cu, batch, total);
  a.prefix = prefix; a.slots = slots; a.max_seq = cache.max_seq;
  a.seq_lens = cache.seq_lens; a.status = cache.status; a.max_batch = cache.max_batch;
  a.pm = page_map_of(cache);
  a.ps_shift = 0;
  while (a.pm.table && (1 << a.ps_shift) < a.pm.page_size) ++a.ps_shift;
  a.L = (bf16 *)L;
  if (fuse) {
    a.wp = (const bf16 *)wp; a.gate = d.gate ? (const bf16 *)gate : nullptr; a.out = (bf16 *)out;
    a.hpq = d.hpq; a.dh = d.dh; a.nh = d.nh; a.gate_kind = d.gate;
    launch_attn_any<true>(a, d, batch, max_chunk, cache.max_seq, nullptr, st);
  } else {
    launch_attn_any<false>(a, d, batch, max_chunk, cache.max_seq, part, st);
  }
}

}  // namespace gta
