// Host-callable launchers of the gfx950 kernels (internal to the library).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "common.h"

namespace sv {

// ---- gemm.hip ----
int gemm_bf16_shape_ok(int N, int K, int splits);
int gemm_bf16_variant_ok(int variant, int N);
hipError_t gemm_bf16(const bf16_t* A, const bf16_t* W, float* out, int M, int N, int K, int splits, int variant,
                     hipStream_t st);
hipError_t pack_weight(const bf16_t* src, bf16_t* dst, int N, int K, hipStream_t st);
hipError_t pack_rows(const bf16_t* src, bf16_t* dst, int M, int K, hipStream_t st);
// row_tiles: 32-row tiles per work-group (1..5; 0 = as few work-groups along the rows as five tiles each allow); cold, here and below: the
// weights come from HBM (see kCacheBytes)
hipError_t gemm_bf16_ws(const bf16_t* Ap, const bf16_t* Wp, float* out, int M, int N, int K, int splits, bool wide, bool cold,
                        hipStream_t st, int row_tiles = 0);
int gemm_bf16_ws_row_tiles(int M);
// Tall tiles, 64 rw rows (rw 3..5) x 256 features, both operands through LDS: n of them along the rows, then nt of 64 rwt
// rows (rwt < rw).  glu: N = 2 F gate and up rows, out = packed bf16 activations [ceil(M/32)*32, F]
struct TallTiles { int rw, n, rwt, nt; };
struct TallPlan { int splits; TallTiles tiles; double us; };
hipError_t gemm_bf16_tall(const bf16_t* Ap, const bf16_t* Wp, float* out, int M, int N, int K, int splits, bool glu, const TallTiles& tiles, hipStream_t st);
// Narrow strips: one work-group of 32 `tiles` rows (tiles 1..5, 6, 8 or 10) x 32 fs features (fs 4, 5 or 7); the rest as above
struct StripTile { int tiles, fs; };
struct StripPlan { int splits; StripTile tile; double us; };
constexpr int kStripRows = 320;             // most rows of a strip
inline int gemm_bf16_strips(int N, const StripTile& s) { return (N / 2 + 16 * s.fs - 1) / (16 * s.fs); }    // strips of N features
hipError_t gemm_bf16_strip(const bf16_t* Ap, const bf16_t* Wp, float* out, int M, int N, int K, int splits, bool glu, const StripTile& tile, bool cold, hipStream_t st);
StripPlan gemm_bf16_strip_plan(int M, int N, int K, int min_splits, int max_splits, bool glu);
TallPlan gemm_bf16_tall_plan(int M, int N, int K, int max_splits);
TallTiles gemm_bf16_tall_256(int M);
hipError_t gemm_bf16_ws_glu(const bf16_t* Ap, const bf16_t* Wp, bf16_t* act_out, int M, int F, int K, hipStream_t st);
// fp32.  norm.gain != null: A are residual rows, a * rsqrt(mean(a^2) + eps) * gain is what is multiplied (rows 16-byte aligned; where
// gemm_f32_fuses says so).  add: out += the product
struct F32Norm { const float* gain; float eps; };
enum F32Form { kF32Plain, kF32Glu, kF32Qkv };
bool gemm_f32_fuses(int M, int N, int K, F32Form form);
hipError_t gemm_f32(const float* A, const float* W, float* out, int M, int N, int K, bool add, const F32Norm& norm, hipStream_t st);
// W [2F][K] (gate rows, then up rows): act [M][F] = silu(gate) * up
hipError_t gemm_f32_glu(const float* A, const float* W, float* act, int M, int F, int K, const F32Norm& norm, hipStream_t st);
// QKV projection, rotary embedding and append in one (rope.qkv_part unused); norm.gain != null
struct RopeAppend;
hipError_t gemm_f32_qkv(const float* h, const float* W, int K, const F32Norm& norm, const RopeAppend& rope, hipStream_t st);

// ---- elementwise.hip ----
// One pass of rows, described by the host in one staged block (ints): per request kReqInts of
//   first row t0, rows n, keys per split-KV piece, pieces, first row of the request's attention partials, partial rows
//   per kv head, partial rows per piece, sequence id, prompt index and first column (prefill; else 0), 2 unused.
// Rows of a request are consecutive; requests may have different numbers of rows (prefill).
constexpr int kReqInts = 12;
struct RowPrep {
    const int32_t* req;         // [B][kReqInts]
    const int32_t* seq_len;     // [max_seqs] live lengths
    const int32_t* page_table; int max_pages_per_seq, page_size;
    const int32_t* last_tokens; // [B]
    const int32_t* drafts;      // [B, N*k] (may be null when k == 0)
    const int32_t* tok_matrix; int tok_ld;   // prefill: the prompts instead of last_tokens / drafts
    const void* embed; int dtype; float* h; int d;   // embed != null: h[t,:] = the row's embedding (fp32)
    int32_t* row_slot;          // [T] physical cache slot: page * page_size + position in the page
    int32_t* row_info;          // [T][4] sequence id, index among the request's rows, the request's rows, its cached length
    int32_t* row_part;          // [T][4] row of the first attention partial (kv head 0, piece 0, q head 0 of the group), partial
                                //        rows per kv head, per piece, pieces to merge (0: the attention writes the row itself)
    float* rope;                // [T, head_dim/2, 2] cos, sin
    int T, B, n, k, head_dim, vocab, group;  // n > 0: every request has n rows; 0: look t0 / n up.  group = q heads per kv head
    float rope_theta;
};
hipError_t prep_rows(const RowPrep& p, hipStream_t st);
// h[t,:] += sum_s part[s][t,:] (S may be 0), then a[t,:] = storage(h * rsqrt(mean(h^2)+eps) * w)
// last.of != null (the end of a prefill): only the last row of each of last.n requests of that table is normalised, to rows last.row0,
// last.row0 + 1, ... of a.  dense: what is added has one row for each of these and no others
struct LastRows { const int32_t* of; int n; bool dense; int row0; };
hipError_t add_rmsnorm(float* h, const float* part, int S, const void* w, void* a, int dtype, int T, int d, float eps,
                       bool packed, hipStream_t st, const LastRows& last = LastRows{});
// the same with the addend = weighted sum of the row's top_k expert outputs y[inv[t*top_k + j]] (bf16 models)
hipError_t add_rmsnorm_experts(float* h, const float* y, const int32_t* inv, const float* wts, int top_k, const void* w, void* a,
                               int T, int d, float eps, bool packed, hipStream_t st, const LastRows& last = LastRows{});
struct RopeAppend {
    const float* qkv_part; int S;       // [S][T][(Hq+2Hkv)*hd]
    const float* rope;                  // [T][hd/2][2]
    const int32_t* row_slot;            // [T] physical cache slots
    void* q_out;                        // [T][Hq][hd] storage type
    void* pool; KvGeom geom; int layer;
    int T, Hq, Hkv, hd, dtype;
};
hipError_t rope_append(const RopeAppend& p, hipStream_t st);
hipError_t swiglu(const float* gu_part, int S, void* act, int T, int F, bool packed, hipStream_t st);   // bf16
hipError_t kv_copy(void* pool, const KvGeom& geom, int layer, const int32_t* page_table_row, int pos0, int n,
                   void* k, void* v, int dtype, bool to_pool, hipStream_t st);
hipError_t set_i32(int32_t* p, int32_t v, hipStream_t st);
// seq_len[request's sequence] += the request's rows (end of a prefill pass)
hipError_t add_rows(int32_t* seq_len, const int32_t* req, int B, hipStream_t st);

// ---- few.hip ----
// Projections of up to 16 rows (packed weights that start at 16 bytes).  norm.gain != null: `in` are up to 8 fp32 residual rows, normalised
// on the way in; else packed operands.  few_rows_ok: the shapes that each form takes (N features of the matrix)
struct FewNorm { const bf16_t* gain; float eps; };
enum FewForm { kFewAdd, kFewGlu, kFewQkv };
bool few_rows_ok(int M, int N, int K, FewForm form, bool norm);
// QKV projection, rotary embedding and append (rope.qkv_part unused)
hipError_t few_rows_qkv(const void* in, const bf16_t* W, int K, const FewNorm& norm, const RopeAppend& rope, bool cold, hipStream_t st);
// h [M][N] += act W^T
hipError_t few_rows_add(const bf16_t* act, const bf16_t* W, float* h, int M, int N, int K, bool cold, hipStream_t st);
// act = silu(gate) * up of the normalised rows, packed
hipError_t few_rows_glu(const float* h, const bf16_t* W, bf16_t* act, int M, int F, int K, const FewNorm& norm, bool cold, hipStream_t st);

// ---- attention.hip ----
constexpr int kItemInts = 8;
struct AttnArgs {
    const void* q;                      // [T][Hq][hd] storage type
    const void* pool; KvGeom geom; int layer;
    const int32_t* page_table; int max_pages_per_seq;
    const int32_t* seq_len;             // [max_seqs]
    const int32_t* row_info;            // [T][4], see RowPrep
    const int32_t* row_part;            // [T][4]
    void* out;                          // [T][Hq*hd] storage type
    float* part_o;                      // split-KV partials [partial row][hd]
    float* part_ml;                     // [partial row][2] reference maximum, sum
    int row_groups;                     // set by attention(): work-groups that share one (item, head)
    int T, n_max, k, Hq, Hkv, hd, dtype;   // n_max: most rows of a request
    // items of the bf16 kernels, kItemInts ints each: sequence id, first key, end, rows n of the request; its first row t0,
    // first stacked row of the item (row_items), first partial row of the piece (kv head 0; -1: the request has one piece,
    // the kernel writes the output itself), partial rows per kv head
    const int32_t* work; int n_work;
    const int32_t* n_work_dev;          // when set: the item count lives here (a captured launch cannot carry it)
    int grid_items;                     // when > 0: items the grid is sized for (an upper bound of the item count)
    bool row_items;                     // prefill: an item is 64 stacked rows of a request, whose keys end at the last one it sees
    bool merge;                         // some request has several pieces
    bool four_waves;                    // prefill: four waves a work-group instead of two
    bool cold;                          // the keys and values come from HBM (see kCacheBytes)
    const int32_t* last_of; int n_last; // when set (the last layer of a prefill): only the last rows of the first n_last requests of that
    void* last_out;                     //       table are wanted, in rows 0 .. n_last - 1 of this buffer, which is not `out` (work: items that hold them)
    int min_row_tiles;                  // lower bound on the 16-row tiles of the bf16 kernel (tuning)
    int max_row_tiles;                  // most 16-row tiles one work-group takes (1..4); more rows -> row groups
    bool out_packed;                    // write `out` in the packed activation order (see act_index)
    bool force_generic;                 // take the generic path (a work-group per row and head) whatever the shape
};
constexpr int kItemRows = 64;               // stacked rows of a prefill item
constexpr int kStepRows = 256;              // most stacked rows per kv head of a step's request that the bf16 kernels take
// the bf16 kernels cover the shape; step_rows: stacked rows per kv head of a step's request, 0 for a prefill
bool attn_mfma_ok(int dtype, int hd, int page_size, bool force_generic, int step_rows);
// do a prefill's work-groups take four waves?  (keys of its items, longest first)
bool prefill_four_waves(const int* keys, int items, int Hkv);
hipError_t attention(const AttnArgs& a, hipStream_t st);

// ---- moe.hip ----
struct MoeArgs {
    const bf16_t* a;          // activations, packed [ceil(T/32)][d/16][64][8]
    const bf16_t* w_router;   // [E][d] row-major
    const bf16_t* w_gate_up;  // [E][2F][d] packed as one (E*2F) x d matrix
    const bf16_t* w_down;     // [E][d][F] packed as one (E*d) x F matrix
    float* router_logits;     // [parts][T][E] partial router logits (parts of the reduction)
    int router_parts = 4;     // parts it has room for, at least 4
    int32_t* top_ids;         // [T][top_k] experts in descending probability
    float* top_w;             // [T][top_k] renormalised weights
    int32_t* live;            // [2 + 2 E] number of experts that have rows, -; of each: id | tiles << 16, first tile
    int32_t* tile_off;        // [E+1] first 32-row tile of each bucket
    int32_t* perm;            // [32 * max_tiles] source row of a padded row
    int32_t* inv;             // [T * top_k] padded row of an assignment
    bf16_t* act;              // [max_tiles][F/16][64][8] SwiGLU outputs as operand tiles
    float* y;                 // [32 * max_tiles][d] expert outputs (until the first product has read them: the buckets' rows as bf16 operand tiles)
    float* out;               // [T][d] combined result
    int T, d, E, top_k, F;
    bool cold;                // the expert weights come from HBM (see kCacheBytes)
};
int moe_shape_ok(int T, int d, int E, int top_k, int F);
size_t moe_group_lds_bytes(int T, int E);
int moe_max_tiles(int T, int E, int top_k);
hipError_t moe_ffn(const MoeArgs& a, hipStream_t st);

// ---- sampler.hip ----
struct SampleArgs {
    const float* logits;                // [T][V]
    const int32_t* drafts;              // [B][N][k]
    const float* draft_probs;           // [B][N][k][V] or null
    const float* uniforms;              // [B][N][k+1] or null (greedy)
    const int32_t* draft_lens;          // [B] or null
    float* stat_part;                   // [sample_part_entries(T)][4] a row part's max, sum exp((x-max)/temp), argmax id (as int bits)
    float* draw_part;                   // [sample_part_entries(T)][4] winners of the parts of a race
    int32_t* accepted_len;              // [B]
    int32_t* out_tokens;                // [B][k+1]
    int32_t* best_chain;                // [B]
    int B, N, k, V, verify_mode, sample_mode;
    float temperature;
    int32_t* seq_len; const int32_t* batch_seq;   // when set: live lengths, advanced by accepted + 1
    int stat_parts, draw_parts;         // set by sample_verify()
};
constexpr int kDrawParts = 8;
size_t sample_part_entries(int rows);
hipError_t sample_verify(const SampleArgs& a, hipStream_t st);
struct RollbackArgs {
    void* pool; KvGeom geom; int n_layers, dtype;
    const int32_t* page_table; int max_pages_per_seq;
    const int32_t* batch_seq;
    int32_t* seq_len;
    const int32_t* accepted_len;
    const int32_t* best_chain;
    int B, N, k;
};
// move the kept chain's accepted K/V entries next to x0 (N > 1 only); committed: the live lengths have been advanced already
hipError_t compact_kept(const RollbackArgs& a, bool committed, hipStream_t st);
// advance the live lengths by accepted + 1
hipError_t commit_lens(const RollbackArgs& a, hipStream_t st);

}  // namespace sv
