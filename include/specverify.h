/*
 * specverify -- C ABI of the batched speculative-verification step on one
 * MI355X (gfx950).
 *
 * The operation.  The paper states it in words (Introduction, "This work";
 * Section 3, "Opportunity: speculative decoding for rollout"): a verifier
 * instance holding the trained model receives, for every request of a batch,
 * the tokens a drafter proposed; it checks all of them in ONE parallel forward
 * pass against the request's KV cache; the first rejected token and every
 * draft after it are dropped and the verifier supplies the token for that
 * position; accepted tokens count as generated by the trained model and the
 * result is lossless with respect to plain decoding.  "Acceptance length" is
 * the number of tokens one verification emits, the supplied token included
 * (Section 4.1).  Drafter and verifier exchange nothing but these messages
 * (Section 4.3), which is what verify_step() carries.  The accept / residual /
 * bonus rule is speculative sampling as in the works the paper cites for it;
 * it is restated at verify_step() below.
 *
 * Conventions.
 *  - "device" pointers are HIP device memory on the GPU that was current at
 *    verify_init(); "host" pointers are ordinary process memory.
 *  - The caller owns every device buffer (weights, KV pool, workspace, inputs,
 *    outputs); they must stay valid until the work enqueued on them is done.
 *    The library allocates host bookkeeping only and never frees caller memory.
 *  - All device work is enqueued on the stream given to verify_init();
 *    functions return after enqueueing unless stated otherwise.
 *  - Every function returns SV_OK (0) or a negative sv_status.  Host arguments
 *    (shapes, ids, limits, page demand) are checked before anything is enqueued
 *    or any bookkeeping changes: a call they fail leaves the context as it was.
 *    If a HIP runtime call fails after that (SV_EHIP), the sequences' live
 *    lengths are unchanged, but pages already reserved for the batch stay with
 *    their sequences (verify_seq_len returns them to the pool) and work already
 *    enqueued runs.  verify_last_error() gives the text.
 *  - Matrices are [out_features, in_features], in_features contiguous.
 */
#ifndef SPECVERIFY_H
#define SPECVERIFY_H

#include <stddef.h>
#include <stdint.h>

#ifdef __cplusplus
extern "C" {
#endif

typedef struct sv_ctx sv_ctx; /* opaque; created by verify_init, destroyed by verify_destroy */

typedef enum {
    SV_OK = 0,
    SV_EINVAL = -1,       /* null pointer, shape or range violation */
    SV_ENOPAGES = -2,     /* KV page pool exhausted */
    SV_ENOSEQ = -3,       /* unknown / duplicate sequence id */
    SV_EUNSUPPORTED = -4, /* shape the kernels do not cover */
    SV_EHIP = -5          /* a HIP runtime call failed */
} sv_status;

enum { SV_FP32 = 0, SV_BF16 = 1 };          /* storage type of weights, KV, GEMM operands */
enum { SV_GREEDY = 0, SV_STOCHASTIC = 1, SV_MATCH = 2 };  /* verify_mode */
enum { SV_INVERSE_CDF = 0, SV_EXP_RACE = 1 }; /* sample_mode */

/* Decoder geometry: pre-norm decoder, RMSNorm, grouped-query attention with
 * rotary embedding (rotate-half pairing i <-> i + head_dim/2, angle
 * pos * rope_theta^(-2i/head_dim)), SwiGLU FFN (n_experts == 0) or softmax
 * router + top_k experts with renormalised weights (n_experts > 0), no biases,
 * untied LM head. */
typedef struct {
    int32_t n_layers, d_model, n_q_heads, n_kv_heads, head_dim, d_ff, vocab;
    int32_t n_experts, top_k, d_expert; /* 0,0,0 = dense */
    int32_t dtype;                      /* SV_FP32 or SV_BF16 */
    float rope_theta, rms_eps;
} sv_model;

/* Weights: device pointers, borrowed for the life of the context.  The
 * per-layer members are HOST arrays of n_layers device pointers.
 *   embed, lm_head [vocab, d_model]; final_norm, ln1[l], ln2[l] [d_model];
 *   wqkv[l] [(n_q_heads + 2 n_kv_heads) head_dim, d_model], rows = q heads, k heads, v heads;
 *   wo[l] [d_model, n_q_heads head_dim];
 *   dense: w_gate_up[l] [2 d_ff, d_model] (gate rows, then up rows), w_down[l] [d_model, d_ff];
 *   MoE:   w_router[l] [n_experts, d_model], w_gate_up[l] [n_experts, 2 d_expert, d_model],
 *          w_down[l] [n_experts, d_model, d_expert].
 * Element type = sv_model.dtype.
 * packed != 0 (bf16 only): lm_head, wqkv, wo, w_gate_up and w_down are given in the fragment order that
 * sv_op_pack_weight() produces (same size as the row-major matrix): the projection kernels then read each
 * weight panel as one contiguous stream.  embed and the norm gains are row-major either way. */
typedef struct {
    const void *embed, *lm_head, *final_norm;
    const void *const *ln1, *const *wqkv, *const *wo, *const *ln2;
    const void *const *w_gate_up, *const *w_down, *const *w_router; /* w_router NULL if dense */
    int32_t packed;
} sv_weights;

/* Run-time limits and caller-provided device memory.
 * kv_pool must hold verify_kv_pool_bytes(), workspace verify_workspace_bytes();
 * both 256-byte aligned.  page_size: tokens per KV page, a multiple of 32. */
typedef struct {
    int32_t max_batch;         /* requests per verify_step */
    int32_t max_k;             /* drafts per chain */
    int32_t max_chains;        /* draft chains per request */
    int32_t max_seqs;          /* sequence ids are 0 .. max_seqs-1 */
    int32_t page_size;
    int32_t num_pages;
    int32_t max_pages_per_seq;
    int32_t verify_mode;       /* SV_GREEDY / SV_STOCHASTIC / SV_MATCH */
    int32_t sample_mode;       /* SV_INVERSE_CDF / SV_EXP_RACE (stochastic mode only) */
    float temperature;         /* divides the target logits; the paper's rollouts use 1.0 (Section 5.1) */
    void *kv_pool;             /* device */
    size_t kv_pool_bytes;
    void *workspace;           /* device */
    size_t workspace_bytes;
} sv_runtime;

/* One verification request batch.  A request b contributes n = 1 + N*k new
 * rows: x0 (its last committed token, not yet in the cache) at position L_b,
 * and draft i (1..k) of chain c at position L_b + i. */
typedef struct {
    int32_t B, k, N;
    const int32_t *seq_ids;     /* host   [B]  distinct ids of cached sequences */
    const int32_t *last_tokens; /* device [B]  x0 */
    const int32_t *draft_lens;  /* device [B]  or NULL: per-request draft window <= k (all chains) */
} sv_batch;

typedef struct {
    int32_t *accepted_len; /* device [B]       a_b in 0..k                                  */
    int32_t *out_tokens;   /* device [B, k+1]  a_b accepted drafts, then the supplied token; rest -1 */
    int32_t *best_chain;   /* device [B]       chain that was kept                          */
    float *logits;         /* device [B*n, vocab] or NULL: receives the target logits (row order = b, then x0, chain 0 drafts, chain 1 ...) */
} sv_out;

/* Sizes of the two caller-provided device buffers for (model, runtime). 0 on invalid arguments.  The workspace is what the
 * verification steps need; a larger one is used for wider prefill passes (sv_workspace_bytes gives the size for a number of
 * rows). */
size_t verify_kv_pool_bytes(const sv_model *, const sv_runtime *);
size_t verify_workspace_bytes(const sv_model *, const sv_runtime *);

/* Create a context on the current device.  hip_stream: a hipStream_t (NULL = the null stream).
 * Enqueues initialisation of the workspace.  SV_EUNSUPPORTED for geometries outside the kernels'
 * cover: head_dim 64 or 128, d_model a multiple of 4 up to 8192, and for bf16 every projection's output width a
 * multiple of 128 and input width a multiple of 64.  Mixture-of-experts models: bf16 with packed weights only,
 * n_experts a multiple of 64 up to 256, top_k <= 64, d_model and d_expert multiples of 128. */
int verify_init(const sv_model *, const sv_weights *, const sv_runtime *, void *hip_stream, sv_ctx **out);
void verify_destroy(sv_ctx *);
const char *verify_last_error(const sv_ctx *); /* never NULL; valid until the next call on ctx */

/* Sequence bookkeeping (the per-request KV cache that persists across steps and grows with the
 * generated tokens, Section 4.3 "KVCache-scale").  seq_add claims pages for cached_len entries whose
 * contents the caller then provides with verify_kv_write or verify_prefill.  seq_set_len truncates or
 * re-extends the live length (rollback to an earlier point; entries beyond are dead).  seq_len reads
 * the true length back: it SYNCHRONISES the stream, and lets the host release pages it had reserved
 * for drafts that were rejected. */
int verify_seq_add(sv_ctx *, int32_t seq_id, int32_t cached_len);
int verify_seq_remove(sv_ctx *, int32_t seq_id);
int verify_seq_set_len(sv_ctx *, int32_t seq_id, int32_t len);
int verify_seq_len(sv_ctx *, int32_t seq_id, int32_t *len_out /* host */);

/* Copy cache entries [pos0, pos0+n) of one layer from / to dense device arrays
 * k, v of shape [n, n_kv_heads, head_dim] in the storage type (the paged layout is internal). */
int verify_kv_write(sv_ctx *, int32_t seq_id, int32_t layer, int32_t pos0, int32_t n, const void *k, const void *v);
int verify_kv_read(sv_ctx *, int32_t seq_id, int32_t layer, int32_t pos0, int32_t n, void *k, void *v);

/* Plain causal pass over n tokens (device int32) appended to the sequence; every token is cached.
 * last_logits (device [vocab] fp32, may be NULL) receives the logits of the last token.  A batch of one prompt
 * for verify_prefill_batch (see there). */
int verify_prefill(sv_ctx *, int32_t seq_id, const int32_t *tokens, int32_t n, float *last_logits);

/* The same for B sequences at once (HOST arrays seq_ids[B], n[B]; all distinct and live): prompt b is row b of
 * the device int32 matrix tokens [B, ld], n[b] <= ld tokens long, and the prompts must come longest first.
 * The prompts go through packed, in prompt order, in as few passes of equal size as hold all their tokens: a pass takes
 * as many rows as the workspace has room for, up to 4096 (never fewer than a step of the context, nor more than the cache
 * holds; fewer for mixture-of-experts models with many experts and for row-major weights), and streams the weights once for
 * all of them.  max_pages_per_seq must cover cached length
 * + prompt.  last_logits (device [B, vocab] fp32, may be NULL) receives each
 * prompt's last-token logits.  Errors leave lengths and pages as they were before the failing pass. */
int verify_prefill_batch(sv_ctx *, const int32_t *seq_ids, int32_t B, const int32_t *tokens, int32_t ld,
                         const int32_t *n, float *last_logits);

/* The verification step.
 *   drafts      device int32 [B, N, k]
 *   draft_probs device fp32  [B, N, k, vocab], q_i(.) the drafter sampled d_i from; NULL = one-hot drafts
 *   uniforms    device fp32  [B, N, k+1], each in [0,1); ignored (may be NULL) in greedy mode; match mode reads
 *               chain 0's row only
 * Per request and chain, with p_i = softmax(target logits of slot i / temperature):
 *   greedy:     accept d_i while d_i == argmax p_i (lowest id on ties); supply argmax p_{a+1}.
 *   stochastic: accept d_i while u_i * q_i(d_i) < p_i(d_i); at the first rejection r supply a draw
 *               from max(p_r - q_r, 0) (from p_r if that is identically 0); with no rejection supply
 *               a draw from p_{k+1}.  The draw consumes u_{k+1}: sample_mode SV_INVERSE_CDF takes the
 *               smallest id whose running weight sum exceeds u * total; SV_EXP_RACE takes
 *               argmax_v (ln w_v - ln e_v), e_v = -log1p(-U_v), U_v = (float(z >> 32) + 0.5) * 2^-32,
 *               z = SplitMix64-finalise(((b*N + c) << 32 | bits(u_{k+1})) + (v+1) * 0x9E3779B97F4A7C15).
 *   match:      (sampled exact match) for every slot i the target's own token t_i is drawn from p_i by the
 *               sample_mode's rule with randomness that depends on the request and the slot only: the uniform
 *               u[b, 0, i-1] of chain 0, and in SV_EXP_RACE the key (b << 32 | bits(u)) with b the request's
 *               index in the batch.  Accept d_i while d_i == t_i; supply t_{a+1}.  Every chain that agrees with
 *               the sampled tokens so far sees the same p_i and is held to the same t_i, so the emitted tokens
 *               are those of plain sampling with the same keys whichever chain is kept: the longest-chain rule
 *               below loses nothing for any N (the stochastic rule is lossless for N = 1 only).  draft_probs
 *               is not read.
 * Token ids reach the step in device memory and are not checked on the host.  A draft id outside [0, vocab) is
 * rejected in every mode without being used as an index: its row is embedded as the nearest valid id (the row's
 * results are dead, the chain ends before it), and the token supplied for its slot is drawn from p_r itself
 * (q_r taken as zero).  A last_tokens id outside the vocabulary is embedded as the nearest valid id.
 * The chain with the largest accepted length is kept (lowest chain id on ties).  The cache then holds
 * x0 and the a accepted drafts at positions L_b .. L_b + a, its length is L_b + a + 1, and the supplied
 * token is the next step's x0.  k = 0 is plain decoding of one token. */
int verify_step(sv_ctx *, const sv_batch *, const int32_t *drafts, const float *draft_probs,
                const float *uniforms, const sv_out *);

#ifdef __cplusplus
}
#endif
#endif /* SPECVERIFY_H */
