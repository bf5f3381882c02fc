// Internal declarations shared by the HIP translation units of libhistospec.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <atomic>
#include <string>
#include <vector>

#include "histospec.h"

typedef uint16_t bf16_t;  // storage type: upper half of an fp32

// Keys per split-KV partition of the verify attention when nothing else is known (hs_create picks 128, 256, 512 or 1024
// from the context's limits).  Partitions are keyed to absolute position, so a row's reduction order does not
// depend on how many draft rows share its sequence.
constexpr int HS_ATT_PART_DEFAULT = 512;
// History segment scanned by one workgroup of the draft kernel.
constexpr int HS_DRAFT_SEG = 4096;
constexpr int HS_MAX_NODES = 64;  // ancestor masks are 64-bit

// Rejection sampling: the vocabulary is summed in slices of this many tokens; per row and slice the largest logit and the
// sum of exp((logit - largest) / temperature) are kept in the workspace, with a word that says which call wrote them
// (calls of one context may overlap on different streams).
constexpr int HS_REJECT_SLICE = 4096;
struct alignas(16) hs_reject_stat { float m; uint32_t check; double s; };
static inline int hs_reject_slices(int vocab) { return (vocab + HS_REJECT_SLICE - 1) / HS_REJECT_SLICE; }

struct hs_workspace_layout {
    size_t x, xn, qkv, q, attn, act, part_o, part_ml, logits, logits_bytes, rowmax, draft_best, gemm_part, gemm_part_bytes, err, pf_len, row_info, att_work, att_list, reject_stats, reject_walk, total;
};

struct hs_ctx {
    hs_model_desc desc;
    hs_limits lim;
    const bf16_t *embed, *lm_head;
    const float *norm_f, *rope_cs;
    std::vector<const bf16_t*> wqkv, wo, wgate, wup, wdown;
    std::vector<const float*> norm1, norm2;
    uint32_t flags = 0;
    char* capture = nullptr;  // hs_debug_capture: snapshots of the last layer's projection inputs
    char* ws = nullptr;
    size_t ws_bytes = 0;
    hs_workspace_layout lay;
    int att_part = HS_ATT_PART_DEFAULT;
    int max_parts = 0;
    int max_segs = 0;
    mutable std::atomic<uint32_t> reject_calls{0};   // numbers the rejection-sampling calls (any host thread)
    int n_cu = 256;  // compute units of the device the context was created on
    std::string err;
    // profiling
    int profile = 0;
    std::vector<hipEvent_t> ev;  // pairs
    std::vector<int> ev_class;
    int ev_used = 0;
    int ev_last = 0;
};

static inline __host__ __device__ float bf16_to_f32(bf16_t b) {
    union { uint32_t u; float f; } c;
    c.u = (uint32_t)b << 16;
    return c.f;
}

// Round to nearest even (inputs here are never NaN).
static inline __host__ __device__ bf16_t f32_to_bf16(float f) {
    union { uint32_t u; float f; } c;
    c.f = f;
    uint32_t u = c.u;
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (bf16_t)(u >> 16);
}

// hs_set_flags: plain kernels (either flag), and with them activations and KV cache in fp32.
static inline bool hs_fp32_activations(const hs_ctx* ctx) { return (ctx->flags & HS_FLAG_FP32_ACTIVATIONS) != 0; }
static inline bool hs_plain_kernels(const hs_ctx* ctx) {
    return (ctx->flags & (HS_FLAG_REFERENCE_KERNELS | HS_FLAG_FP32_ACTIVATIONS)) != 0;
}
int hs_gemm_chunks(int n, int k);
int hs_gemm_chunks(int n, int k, bool narrow);   // with groups of 64 (narrow) or 128 weight rows
// Must the logits exist as an [rows][vocab] array?  Yes if the caller asks for them (a destination in the step, or
// HS_FLAG_WORKSPACE_LOGITS), with the plain kernels, and when the LM head splits K (a small vocabulary).  Otherwise the
// LM head reduces every row to its argmax in its epilogue and hs_accept finishes the reduction.
static inline bool hs_logits_in_workspace(const hs_ctx* ctx) {
    return (ctx->flags & HS_FLAG_WORKSPACE_LOGITS) != 0 || hs_plain_kernels(ctx) ||
           hs_gemm_chunks(ctx->desc.vocab, ctx->desc.d_model) > 1;
}
static inline bool hs_head_fused(const hs_ctx* ctx, const hs_step* step) {
    return !step->logits && !hs_logits_in_workspace(ctx);
}

// Grid of a row-strided kernel (workgroup i takes rows i, i + grid, ...) whose workgroups have `threads` threads and
// of which `per_row` work on one row: what the device holds at once (2048 threads per compute unit), at most one
// set per row.  The row count itself is only known on the device.
static inline int hs_row_grid(const hs_ctx* ctx, int threads, int per_row = 1) {
    const int resident = ctx->n_cu * (2048 / threads) / per_row;
    return resident < 1 ? 1 : (resident < ctx->lim.max_rows ? resident : ctx->lim.max_rows);
}

// A zero that the compiler does not know: an index with it makes a load that all lanes share a vector load.  Such loads
// return in the order of their issue, so that a row's data can be asked for behind the row count and both are waited for at
// once; a scalar load's wait would hold up whatever is addressed by another scalar load.
__device__ __forceinline__ unsigned hs_opaque_zero() {
    unsigned z;
    asm volatile("v_mov_b32 %0, 0" : "=v"(z));
    return z;
}
// What has been asked for above stays above.
__device__ __forceinline__ void hs_loads_issued() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}
__device__ __forceinline__ int hs_uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// ---- launchers (each enqueues on `st`; shapes have been validated by the caller) ----

// GEMM family: C[M,N] (+)= A[M,K] . W[N,K]^T, A and W bf16, fp32 accumulation in a fixed k order.
// Activation buffers (a, and c of the SwiGLU epilogue) are bf16, or float in the fp32-activation mode.
// m_dev points at the row count M on the device; the grid covers m_max rows and tiles beyond M exit.
// HS_EPI_ROWMAX (LM head only, unsplit K): nothing of the product is stored; every workgroup reduces its columns of
// each row to one 64-bit key, (order-preserving bits of the largest value) << 32 | ~column, smallest column on ties,
// written to c as unsigned long long [m_max][hs_gemm_rowmax_groups(n)] -- the maximum over a row's keys is its argmax.
enum { HS_EPI_STORE_F32 = 0, HS_EPI_ADD_F32 = 1, HS_EPI_SWIGLU_BF16 = 2, HS_EPI_ROWMAX = 3 };
// rows_hint (host-side estimate of the live row count) selects the tile height and the split execution
// (one workgroup per K chunk + an ordered reduce); results are identical whatever it is.
// pending: if not null and the split execution was chosen, the ordered reduce is NOT launched: *pending receives the
// number of chunk partials left in the workspace ([chunk][m_max][n] floats at lay.gemm_part) for the next kernel in
// line to add up in chunk order and apply the epilogue (store / add to c) -- if there are at most `rows` rows; with more,
// the epilogue has been applied.  No partials: chunks = 0.
// fold: K chunks may run one after the other in a workgroup where that is expected to be so much faster, HS_FOLD_KNOWN or
// HS_FOLD_GUESSED for row counts that are known to the caller or swing around rows_hint; 0 (never) where rows_hint is only a limit.
struct hs_pending { int chunks = 0, rows = 0; };
constexpr double HS_FOLD_KNOWN = 1.08, HS_FOLD_GUESSED = 1.2;
void hs_launch_gemm(const hs_ctx* ctx, int epi, const void* a, const bf16_t* w, const bf16_t* w2, void* c,
                    const int32_t* m_dev, int m_max, int n, int k, int rows_hint, hipStream_t st,
                    hs_pending* pending = nullptr, double fold = 0.);
int hs_gemm_rowmax_groups(int n);   // column groups (= keys per row) of an HS_EPI_ROWMAX launch over n columns

// What a row's place in its sequence comes to, written once per pass (beside the attention's unit lists, or by the launch
// that lays out a prefill's rows) and read by every layer: the row's K/V slot (page * 16 + slot in the page; -1: nothing is written), its position and the number of
// attention partitions of its sequence.
struct alignas(16) hs_row_info { int32_t slot, pos, parts, unused; };
struct hs_row_places {
    const int32_t *pos, *block_table;
    int max_blocks, max_pos, n_blocks;
    hs_row_info* info;
};
static inline hs_row_places hs_row_places_of(const hs_ctx* ctx, const hs_kv_cache* cache, const hs_seq_state* seq, const hs_step* step) {
    return {step->pos, seq->block_table, ctx->lim.max_blocks_per_seq, ctx->lim.max_pos, cache->n_blocks,
            reinterpret_cast<hs_row_info*>(ctx->ws + ctx->lay.row_info)};
}
// The row at `at` tokens from its sequence's start (a position flagged by the draft step, a slot beyond the block table, a
// missing page: nothing is written).
__device__ __forceinline__ hs_row_info hs_place_row(const int32_t* pages, int max_blocks, int n_blocks, int max_pos, int at,
                                                    int pos, int parts) {
    const int page = at >= 0 && (at >> 4) < max_blocks ? pages[at >> 4] : -1;
    const bool none = pos < 0 || pos >= max_pos || page < 0 || page >= n_blocks;
    return {none ? -1 : page * 16 + (at & 15), pos, parts, 0};
}

// In the row kernels below, `expected` is the host's estimate of the row count (0: none).  Up to HS_EARLY_ROWS of it, a workgroup whose
// row lies below it asks for the row's data before the count has arrived from memory (in bounds: never more than max_rows);
// with more, the count comes first: where there are fewer rows than expected, each of the others would be read for nothing.
// The result does not depend on it.  us at 64 rows with 1078 expected, early, counted first and with 64 expected: 1.5B shape, norms
// 8.7 and 12.6, 4.1 and 4.9, 3.7 and 4.0, rotary kernel 10.4, 5.2, 4.0; 7B norm after down 14.7, 5.7, 5.2.  At 7 rows with 64
// expected what is read for nothing costs no time; at 128 and 220 rows counting first costs 0.1 to 0.3 a launch.
constexpr int HS_EARLY_ROWS = 64;
static inline int hs_early_rows(int expected) { return expected <= HS_EARLY_ROWS ? expected : 0; }

// Embedding gather into the residual stream and its first RMSNorm; with lists (hs_verify), the rows' hs_row_info and the
// unit lists of the step's attention are written by further workgroups of the same launch.
void hs_launch_embed_norm(const hs_ctx* ctx, const hs_kv_cache* cache, const hs_seq_state* seq, const hs_step* step,
                          bool lists, float* x, const float* w, void* out, hipStream_t st);
// RMSNorm of the residual stream; with partials pending it first adds the chunk partials of the
// preceding projection (in chunk order) to x.
void hs_launch_rmsnorm(const hs_ctx* ctx, float* x, const float* w, void* out, const int32_t* m_dev,
                       hs_pending pending, int expected, hipStream_t st);
// Rotary embedding + KV write; with partials pending the QKV values are the chunk-ordered sums of the pending
// partials instead of qkv.
void hs_launch_rope_kv(const hs_ctx* ctx, int layer, const hs_kv_cache* cache, const hs_seq_state* seq,
                       const hs_step* step, const float* qkv, void* q, hs_pending pending, int expected,
                       hipStream_t st);
void hs_launch_attention(const hs_ctx* ctx, int layer, const hs_kv_cache* cache, const hs_seq_state* seq,
                         const hs_step* step, const void* q, void* out, hipStream_t st);
// Chunked prefill: row arrays of one call (rows of sequence b = its next tokens from the token log) and the causal
// attention over [0, kv_done + i] for token i of the chunk.  len_plus1[b] = cached positions + 1.
void hs_launch_prefill_rows(const hs_ctx* ctx, const hs_kv_cache* cache, const hs_seq_state* seq, int32_t* kv_done, int chunk, hs_step* step,
                            int32_t* len_plus1, hipStream_t st);
void hs_launch_attention_prefill(const hs_ctx* ctx, int layer, const hs_kv_cache* cache, const hs_seq_state* seq,
                                 const int32_t* len_plus1, const hs_step* step, const bf16_t* q, bf16_t* out, int chunk,
                                 hipStream_t st);
// Unit lists of the verify attention (hs_worklist.h) and their capacity.
struct hs_attn_lists {
    int32_t* work;
    int4 *list_a, *list_b;
    int part_keys, G, hkv, max_parts, n_layers;
};
hs_attn_lists hs_attention_lists(const hs_ctx* ctx);
size_t hs_attention_max_units(const hs_ctx* ctx);
void hs_launch_attention_merge(const hs_ctx* ctx, const hs_seq_state* seq, const hs_step* step, void* out,
                               int expected, hipStream_t st);
void hs_launch_argmax(const hs_ctx* ctx, const float* logits, int32_t* argmax, const int32_t* m_dev,
                      int expected, hipStream_t st);
void hs_launch_draft(const hs_ctx* ctx, const hs_draft_args* args, const hs_seq_state* seq, hs_step* step,
                     hipStream_t st);
// hs_draft_static: segment winners in a static device array of HS_DRAFT_STATIC_ENTRIES slots.  Returns false (with the
// HIP error) if the array's address on the current device cannot be had.  hs_draft_static_error_word: the error word
// kept inside that array (used when no workspace is bound).
constexpr int HS_DRAFT_STATIC_ENTRIES = 1 << 16;
bool hs_launch_draft_static(const hs_ctx* ctx, const hs_draft_args* args, const hs_seq_state* seq, hs_step* step,
                            hipStream_t st, hipError_t* why);
uint32_t* hs_draft_static_error_word(hipError_t* why);
void hs_launch_draft_group(const hs_ctx* ctx, const hs_group_draft_args* args, const hs_seq_state* seq,
                           hs_step* step, hipStream_t st);
// Acceptance and/or commit of one step in one launch (rejection sampling: after one for its sums).  args == nullptr: no acceptance; policy == nullptr: no commit.
// keys != nullptr: the rows' argmax is first reduced from the LM head's row-maximum keys (n_keys per row).
void hs_launch_accept_commit(const hs_ctx* ctx, const hs_accept_args* args, const hs_kv_cache* cache,
                             const hs_seq_state* seq, const hs_step* step, const float* logits,
                             const unsigned long long* keys, int n_keys, const hs_policy* policy, hipStream_t st);
