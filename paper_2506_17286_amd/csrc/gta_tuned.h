// Tuned bf16 path for gfx950: MFMA GEMMs, MFMA prefill attention, streaming split-K decode.
#pragma once
#include "gta_internal.h"

namespace gta {

bool tuned_prefill_supported(const Dims &d);
bool tuned_decode_supported(const Dims &d);
int tuned_decode_target_workgroups(const Dims &d);      // split-K launch size the kernel of this shape wants
int tuned_decode_max_splits(const Dims &d, int batch);   // most splits the cheapest tail kernel of this call takes
bool tuned_decode_layout_ok(const gta_cache &cache);   // block-table layouts the streaming decode kernels take
bool tuned_chunk_layout_ok(const gta_cache &cache);    // ... and the MFMA attention kernel in cache mode

int tuned_prefill(const Dims &d, const gta_weights &w, const void *x, const int32_t *cu, int batch,
                  int64_t total, int max_len, const gta_cache *cache, const int32_t *slots, void *out,
                  const PrefillWs &ws, hipStream_t st);
// setup and projection of a fresh prefill: Q, K, C and gate rows to ws, cache rows and lengths
void tuned_project(const Dims &d, const gta_weights &w, const void *x, const int32_t *cu, int batch, int64_t total, int max_len,
                   const gta_cache *cache, const int32_t *slots, const PrefillWs &ws, hipStream_t st);
// chunked prefill: the chunk's tokens follow the rows the slots already hold (needs the MFMA attention kernel)
bool tuned_prefill_chunk_supported(const Dims &d, int max_seq);
int tuned_prefill_chunk(const Dims &d, const gta_weights &w, const void *x, const int32_t *cu, int batch,
                        int64_t total, int max_chunk, const gta_cache &cache, const int32_t *slots, void *out,
                        const PrefillWs &ws, hipStream_t st);
int tuned_decode(const Dims &d, const gta_weights &w, const void *x_new, int batch, const gta_cache &cache,
                 const int32_t *slots, void *out, const DecodeWs &ws, hipStream_t st);

void tuned_decode_attention(const Dims &d, const float *q, const int32_t *oldlen_in, int32_t *oldlen_out,
                            const gta_cache &cache, const int32_t *slots, int batch, int splits, float *part,
                            hipStream_t st);
void tuned_decode_combine(const Dims &d, const float *part, const int32_t *oldlen, int splits, int batch, float *L,
                          hipStream_t st);

// bf16 MFMA GEMMs (gta_gemm_bf16.hip)
bool gemm_shapes_supported(const Dims &d);
size_t proj_packed_bytes(const Dims &d);   // workspace for the packed [H, Wtot] weights, 0 if not used
PackWeights pack_of(const Dims &d, const gta_weights &w, int64_t M, const PrefillWs &ws);   // what launch_proj_gemm wants packed before it
void launch_proj_gemm(const Dims &d, const gta_weights &w, const void *x, int M, const PrefillWs &ws,
                      const gta_cache *cache, const int32_t *slots, int max_len, bool rope_by_token, const Fold &fold,
                      hipStream_t st);
bool proj_folds(const Dims &d, int batch, int64_t M);   // may launch_proj_gemm do without the setup launch?
void launch_decoder_gemm(const Dims &d, const void *L, const void *wp, const void *g, void *out, int M,
                         hipStream_t st);
int skinny_ksplit(const Dims &d, int M);
void launch_skinny_proj(const Dims &d, const gta_weights &w, const void *x, int M, float *part, int ksplit,
                        hipStream_t st);
void launch_plain_gemm(const void *A, int64_t lda, int M, int N, int K, const void *B, void *C, hipStream_t st);

// bf16 MFMA causal prefill attention (gta_prefill_bf16.hip)
bool attn_prefill_supported(const Dims &d, int max_len);
void launch_attn_prefill_bf16(const Dims &d, const void *q, const void *k, const void *c, const int32_t *cu,
                              int batch, int64_t total, int max_len, void *L, float *part, hipStream_t st);
// scratch `part` of the two that can split the key range (NULL: no splits)
size_t attn_split_bytes(const Dims &d);
// attention with the value decoder and gate fused into its epilogue (narrow shapes): writes the heads
bool attn_decoder_fusable(const Dims &d, int max_len);
void launch_attn_decoder_bf16(const Dims &d, const void *q, const void *k, const void *c, const int32_t *cu,
                              int batch, int64_t total, int max_len, const void *wp, const void *gate, void *out,
                              hipStream_t st);
// The same two against the caches: sequence b's keys / latents are rows 0 .. prefix[b] + T_b - 1 of its
// slot, its queries sit at positions prefix[b] .. (prefix[b] < 0: zero rows).  L may be NULL when fused.  Sets the
// cached lengths, and the flags of skipped sequences (a launch of its own for that took 4 us).
void launch_attn_chunk_bf16(const Dims &d, const void *q, const gta_cache &cache, const int32_t *slots,
                            const int32_t *prefix, const int32_t *cu, int batch, int64_t total, int max_chunk,
                            void *L, const void *wp, const void *gate, void *out, bool fuse, float *part, hipStream_t st);

// bf16 GEMMs for few rows, K split inside the workgroup (gta_rows_bf16.hip)
bool rows_gemm_ok(const Dims &d);
void launch_rows_proj_decode(const Dims &d, const gta_weights &w, const void *x, int batch, const gta_cache &cache,
                             const int32_t *slots, const DecodeWs &ws, hipStream_t st);
void launch_short_proj(const Dims &d, const gta_weights &w, const void *x, int M, const PrefillWs &ws, const gta_cache *cache,
                       const int32_t *slots, int max_len, bool rope_by_token, const Fold &fold, hipStream_t st);
bool short_proj_folds(const Dims &d, int64_t M);
void launch_short_decoder(const Dims &d, const void *L, const void *wp, const void *g, void *out, int M, hipStream_t st);
void launch_short_plain(const void *A, int64_t lda, int M, int N, int K, const void *B, void *C, hipStream_t st);
void launch_rows_plain(const void *A, int64_t lda, int M, int N, int K, const void *B, void *C, hipStream_t st);

// fp32 MFMA kernels (gta_f32.hip).  They serve the shape-generic entry path where the shape allows; each condition
// covers its own kernels.
bool f32_gemms_ok(const Dims &d, int64_t M);                                  // projection, output projection
bool f32_decoder_ok(const Dims &d, int64_t M);                                // value decoder
bool f32_attn_ok(const Dims &d, int batch, int max_len);                      // prefill attention
bool f32_decode_ok(const Dims &d, const gta_cache &cache, int batch);         // decode step
void launch_proj_f32(const Dims &d, const gta_weights &w, const void *x, int M, const PrefillWs &ws, const gta_cache *cache,
                     const int32_t *slots, int max_len, bool rope_by_token, const Fold &fold, hipStream_t st);
bool f32_proj_folds(const Dims &d, int batch, int64_t M);                     // may it do without the setup launch?
void launch_decoder_f32(const Dims &d, const float *L, const void *wp, const float *gate, float *out, int M, hipStream_t st);
void launch_out_proj_f32(const Dims &d, const float *O, const void *wo, float *out, int M, hipStream_t st);
void launch_attn_prefill_f32(const Dims &d, const float *q, const float *k, const float *c, const int32_t *cu, int batch,
                             int64_t total, int max_len, float *L, hipStream_t st);
// partials in the layout of tuned_decode_attention (merged by tuned_decode_combine or the tail)
void launch_decode_attn_f32(const Dims &d, const float *q, const int32_t *oldlen, const gta_cache &cache, const int32_t *slots,
                            int batch, int splits, float *part, hipStream_t st);
int f32_decode(const Dims &d, const gta_weights &w, const void *x_new, int batch, const gta_cache &cache, const int32_t *slots,
               void *out, const DecodeWs &ws, hipStream_t st);
// the narrow decode tail on fp32 weights (gta_decode_bf16.hip); false where it does not take the call
bool launch_decode_tail_f32(const Dims &d, const DecodeWs &ws, int batch, const float *wp, float *out, const gta_cache &cache,
                            const int32_t *slots, hipStream_t st);

}  // namespace gta
