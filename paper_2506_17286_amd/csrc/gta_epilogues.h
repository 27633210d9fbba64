// Epilogues shared by the GEMM kernels that hand out groups of four finished columns (gta_f32.hip,
// gta_rows_bf16.hip), and the column tiles of the kernels for few rows.
#pragma once
#include <type_traits>

#include "gta_internal.h"
#include "gta_rope.h"

namespace gta {

typedef __attribute__((ext_vector_type(4))) float f32x4;

__device__ __forceinline__ void store4(float *p, f32x4 v) { *reinterpret_cast<f32x4 *>(p) = v; }
__device__ __forceinline__ void store4(__bf16 *p, f32x4 v) {
  typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
  bf16x4 o;
#pragma unroll
  for (int i = 0; i < 4; ++i) o[i] = (__bf16)v[i];
  *reinterpret_cast<bf16x4 *>(p) = o;
}

template <typename T>
struct Quad { typedef T type __attribute__((ext_vector_type(4))); };

// ------------------------------------------------------------------------------ epilogues
// A GEMM hands its epilogue groups of four columns in three calls: early(row, first column, rotated tile?) requests
// what the group reads itself, prepare() works out position, cache row and sines, store() takes the values and
// `partner`, which returns the four values half a head further (used by the rotation only).  The kernels for few
// rows call early() ahead of their operand loads and prepare() under them: behind them the two cost a decode step
// 6 us.  Columns are global (all segments).  In the launches for few rows, workgroups behind the tiles are
// for commit(): side_waves() waves of them.

// Projection (Sec. 3.2) with RoPE on q and k (App. B.1.1) and the cache write (App. B.1.3).
// TD: element type of the Q | K | C | gate rows (a decode step keeps q and gate in fp32), TC: of the caches.
// PREFILL: decode steps do not occur, FOLD false: nor does fold.batch > 0 (their sines would be held in registers all the same).
// With fold.batch > 0 a group of columns finds its token among the offsets, which are all requested at once, and takes the
// sines of its angles itself (the same values as the table's), and waves of their own set the lengths.
template <typename TD, typename TC, bool PREFILL = false, bool FOLD = false>
struct ProjEpi {
  TD *dst[4]; int width[4];                 // Q | K | C | gate rows (decode: K and C go to the caches only)
  int dh, rope;
  // prefill: position and sequence of every packed token and the (cos, sin) table
  const int32_t *seq_id, *pos; const float2 *table; int max_len, rope_by_token;
  // decode (seq_lens != NULL): row b is the new token of slot slots[b] at position seq_lens[slot]
  const int32_t *seq_lens; int32_t *oldlen; double freq[64];
  TC *kcache, *ccache; const int32_t *slots; int max_batch, max_seq; PageMap pm;   // kcache NULL: no cache write
  Fold fold; CacheView commit_to;

  int side_waves() const { return commit_to.k ? fold.batch : 0; }
  __device__ __forceinline__ void commit(int wave) const {
    if (FOLD && wave < fold.batch) prefill_commit_seq(commit_to, fold.cu, fold.per_seq, wave);
  }
  __device__ __forceinline__ bool folded() const { return FOLD && fold.batch; }
  __device__ __forceinline__ bool decode() const { return !PREFILL && seq_lens; }
  __device__ __forceinline__ void locate(int col, int &seg, int &local) const {
    seg = 0;
    while (seg < 3 && col >= width[seg]) { col -= width[seg]; ++seg; }
    local = col;
  }
  // does the tile of columns starting at `col` (one segment) hold rotated values?
  __device__ __forceinline__ bool rotates(int col) const { return rope && col < width[0] + width[1]; }
  __device__ __forceinline__ int head_dim() const { return dh; }
  // what a group of four columns reads on its own account, requested before anything else (early), and what follows
  // from it without the group's values (prepare)
  struct Early { int slot, p, seq; double f[4]; };
  struct Ctx { int seg, lc, half; int64_t cr; f32x4 cs, sn; };   // half: distance to the partner (signed), 0 = not rotated
  __device__ __forceinline__ Early early(int row, int col, bool rot) const {
    Early e{};
    if (decode()) {
      e.slot = slots ? slots[row] : row;
      const bool ok = e.slot >= 0 && e.slot < max_batch;
      e.p = seq_lens[ok ? e.slot : 0];
      if (!ok) e.p = -1;
      if (rot) {
        const int j = col % (dh / 2);
#pragma unroll
        for (int i = 0; i < 4; ++i) e.f[i] = freq[j + i];
      }
    } else if (folded()) {
      if (fold.cu) {
        int s[kFoldBatch], start = 0;
#pragma unroll
        for (int b = 0; b < kFoldBatch; ++b) s[b] = fold.cu[min(b, fold.batch - 1)];
#pragma unroll
        for (int b = 0; b < kFoldBatch; ++b)
          if (b < fold.batch && s[b] <= row) { e.seq = b; start = s[b]; }
        e.p = row - start;
      } else {
        e.seq = row / fold.per_seq;
        e.p = row - e.seq * fold.per_seq;
      }
      if (rot) {
        const int j = col % (dh / 2);
#pragma unroll
        for (int i = 0; i < 4; ++i) e.f[i] = freq[j + i];
      }
    } else {
      e.p = pos[row];
      if (kcache) e.seq = seq_id[row];
    }
    return e;
  }
  __device__ __forceinline__ Ctx prepare(const Early &y, int row, int col, bool rot) const {
    Ctx c;
    locate(col, c.seg, c.lc);
    int p = y.p;
    c.cr = -1;
    if (decode()) {
      if (p >= 0 && p < max_seq) c.cr = cache_row(pm, max_seq, y.slot, p);
      if (col == 0) oldlen[row] = c.cr >= 0 ? p : -1;
      if (c.cr < 0) p = 0;                      // slot full: nothing is appended, the tail zero-fills the sequence
    } else if (kcache && (c.seg == 1 || c.seg == 2)) {
      const int slot = slots ? slots[y.seq] : y.seq;
      if (slot >= 0 && slot < max_batch && p >= 0 && p < max_seq) c.cr = cache_row(pm, max_seq, slot, p);
    }
    c.half = 0;
    if (rot && (decode() || rope_by_token || p < max_len)) {
      const int half = dh / 2, e = c.lc % dh, j = e < half ? e : e - half;
      c.half = e < half ? half : -half;
      if (decode() || folded()) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {   // fp32 rows and prompts: the same values as a prefill's table
          const float2 t = PREFILL || std::is_same<TC, float>::value ? rope_cos_sin(p, y.f[i]) : rope_cos_sin_short(p, y.f[i]);
          c.cs[i] = t.x; c.sn[i] = t.y;
        }
      } else {
        const float4 *t = reinterpret_cast<const float4 *>(table + (int64_t)(rope_by_token ? row : p) * half + j);
        const float4 t0 = t[0], t1 = t[1];
        c.cs = f32x4{t0.x, t0.z, t1.x, t1.z}; c.sn = f32x4{t0.y, t0.w, t1.y, t1.w};
      }
    }
    return c;
  }
  template <class Partner>
  __device__ __forceinline__ void store(const Ctx &c, int row, f32x4 v, Partner partner) const {
    if (c.half) {
      const f32x4 o = partner(c.half);
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = c.half > 0 ? v[i] * c.cs[i] - o[i] * c.sn[i] : v[i] * c.cs[i] + o[i] * c.sn[i];
    }
    const bool cached = c.seg == 1 || c.seg == 2;
    if (!(decode() && cached)) store4(dst[c.seg] + (int64_t)row * width[c.seg] + c.lc, v);
    if (c.cr >= 0 && cached) store4((c.seg == 1 ? kcache : ccache) + c.cr * width[c.seg] + c.lc, v);
  }
};

// Value decoder (Sec. 3.2): times the gate factor of the same element.
template <typename T, typename TG = float>
struct GateEpi {
  T *out; const TG *g; int ld, gate;
  int side_waves() const { return 0; }
  __device__ __forceinline__ void commit(int) const {}
  __device__ __forceinline__ bool rotates(int) const { return false; }
  __device__ __forceinline__ int head_dim() const { return 0; }
  struct Early { typename Quad<TG>::type z; };
  struct Ctx { int col; typename Quad<TG>::type z; };
  __device__ __forceinline__ Early early(int row, int col, bool) const {
    Early e{};
    if (gate) e.z = *reinterpret_cast<const typename Quad<TG>::type *>(g + (int64_t)row * ld + col);
    return e;
  }
  __device__ __forceinline__ Ctx prepare(const Early &e, int, int col, bool) const { return Ctx{col, e.z}; }
  template <class Partner>
  __device__ __forceinline__ void store(const Ctx &c, int row, f32x4 v, Partner) const {
    const int64_t o = (int64_t)row * ld + c.col;
    if (gate) {
      const f32x4 z{(float)c.z[0], (float)c.z[1], (float)c.z[2], (float)c.z[3]};
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] *= gate == kGateSigmoid ? 1.0f / (1.0f + expf(-z[i])) : gate_factor(gate, z[i]);
    }
    store4(out + o, v);
  }
};

template <typename T>
struct StoreEpi {
  T *out; int ld;
  int side_waves() const { return 0; }
  __device__ __forceinline__ void commit(int) const {}
  __device__ __forceinline__ bool rotates(int) const { return false; }
  __device__ __forceinline__ int head_dim() const { return 0; }
  struct Early {};
  struct Ctx { int col; };
  __device__ __forceinline__ Early early(int, int, bool) const { return Early{}; }
  __device__ __forceinline__ Ctx prepare(const Early &, int, int col, bool) const { return Ctx{col}; }
  template <class Partner>
  __device__ __forceinline__ void store(const Ctx &c, int row, f32x4 v, Partner) const {
    store4(out + (int64_t)row * ld + c.col, v);
  }
};

// Column tile nt (BN columns) of the kernels for few rows: tile column c is global column col0 + c % (BN / 2) +
// (c / (BN / 2)) * step.  A rotated tile must hold both halves of its heads: with heads wider than BN it takes BN / 2
// columns of one half and those they pair with (`pair`), otherwise whole heads lie in BN columns in a row.
struct RowTile { int col0, step; bool pair; };
template <int BN = 32>
__device__ __forceinline__ RowTile row_tile(int nt, bool rot, int dh) {
  if (!rot || dh <= BN) return RowTile{nt * BN, BN / 2, false};
  const int tph = dh / BN;
  return RowTile{nt / tph * dh + nt % tph * (BN / 2), dh / 2, true};
}

}  // namespace gta
