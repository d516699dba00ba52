// C ABI of the verification step: context, host-side page bookkeeping, and the sequence of kernel
// launches that makes up one parallel verification pass (declared in include/specverify.h).
#include <hip/hip_runtime.h>
#include <stdarg.h>
#include <stdio.h>
#include <string.h>
#include <algorithm>
#include <functional>
#include <cmath>
#include <string>
#include <vector>

#include "../../include/specverify.h"
#include "../../include/specverify_ops.h"
#include "kernels.h"

using namespace sv;

namespace {

constexpr int kRing = 8;              // pinned staging slots for per-step host -> device metadata
constexpr int kMaxSplits = 8;
constexpr int kMaxSplitsWs = 16;       // weight-streaming kernel: any divisor of the slice count up to this
constexpr int kChunkKeys = 1024;      // keys per split-KV chunk of the bf16 attention
// Most rows of a prefill pass.  A pass streams every weight once, so a prompt that goes through in passes of a step's few dozen
// rows pays for that stream again and again: one prompt of 777 tokens through a context sized for 40 rows took 22 passes,
// 29.2 ms over 7 layers of the 7B shape; in one pass 4.7 ms (with the first token's step, 1.2 ms of it).  24 prompts of
// 100-500 tokens, 7 layers: 47.4 ms in 14 passes with the LM head on every row, 26.4 ms in two passes with it on the
// prompts' last rows.  From about a thousand rows on the projections are bound by their products.
// The rows of a pass are the caller's choice, by the size of the workspace: a step's rows where it holds no more (on the 7B
// shape 5 rows 7 MB, 1024 rows 170, 4096 rows 501).
constexpr int kPrefillRows = 4096;
constexpr int kPrefillPlaces = 512;   // work-groups of a prefill's attention that run at once: two per CU
constexpr int kHeadInputs = 2048;      // LM heads of so many inputs or more: see plan_wide
constexpr int kStripInputs = 4096;    // split reductions of no more inputs take strips at some numbers of rows only: see plan_packed
constexpr int kPlans = 64;            // launch plans a context remembers (five shapes per number of rows)
constexpr int kCausalK = 1 << 20;     // "drafts per chain" of a prefill pass: one chain, never ending

struct SeqState {
    bool live = false;
    int len_ub = 0;                   // host upper bound of the live length
    std::vector<int32_t> pages;
};

size_t align_up(size_t x, size_t a = 256) { return (x + a - 1) / a * a; }

int pick_splits(int M, int N, int K) {
    // enough work-groups to cover the 256 CUs about twice; the reduction range stays a multiple of 64
    const int tiles = ((M + 127) / 128) * (N / 128);
    int s = 1;
    while (s < kMaxSplits && tiles * s < 512 && K % (64 * s * 2) == 0) s *= 2;
    return s;
}

// Launch plan of the weight-streaming projection kernel: 32-row tiles per work-group, strip width and reduction
// splits, by an estimate of the run time in microseconds.  The estimate plays the launch through: work-groups are
// dealt to the 256 CUs in rounds (one work-group per CU for the 128- and 160-row x 256-feature tiles, two for the
// smaller ones); a CU works its share off at a rate that grows with the rows it holds (the weight stream is
// shared by more products), no faster than a lone work-group can walk its reduction slices; the chip as a whole
// sustains about 1.2 PFLOP/s on random data (it is power-limited well below the MFMA peak) and 5 TB/s of
// weights (ordinary loads; streamed, as one row tile reads cold ones, 5.4 to 6.5: what this estimate decides by itself, splits and widths, was not
// fitted again); a partial plane costs its bytes, written here and read again by the consumer.  The constants are a
// fit to a sweep of every (tiles, width, splits) over thirty shapes of the benchmark models on MI355X (rows 5 to
// 2304), except the lone work-group's pace, which is taken from whole steps (cold weights); on the sweep the plan
// chosen was within 0.3 % of the best on average and 4.5 % at worst.
// strip.tiles > 0: a strip; tall.n > 0: the tall kernel.  ws_us: the weight-streaming kernel's estimate, whichever it is
struct WsPlan { int splits; bool wide; int row_tiles; double us, ws_us; TallTiles tall; StripTile strip; };
WsPlan plan_ws(int M, int N, int K, bool allow_split, int max_splits = kMaxSplitsWs) {
    const int slices_all = K / 16;
    const int tiles = (M + 31) / 32;
    WsPlan best{1, false, gemm_bf16_ws_row_tiles(M), 1e30, 1e30, {}, {}};
    // up to 160 rows: one work-group along the rows (cutting so few rows only multiplies the readers of a strip)
    const int mt_lo = tiles <= 5 ? tiles : 1, mt_hi = tiles <= 5 ? tiles : 5;
    for (int mt = mt_lo; mt <= mt_hi; ++mt)
        for (int wide = 0; wide < 2; ++wide) {
            if (wide && N % 256 != 0) continue;
            const int cols = wide ? 256 : 128;
            const int tiles_m = (tiles + mt - 1) / mt;
            const int per_cu = (wide && mt >= 4) ? 1 : 2;                     // work-groups resident per CU
            const double base = wide ? 5.19 : 4.14;                           // TFLOP/s of a CU at full tile height
            // us per slice a lone work-group cannot beat: inside a step a layer's weights come cold from HBM (32 KB in
            // flight per work-group against ~1 us of latency), twice what a sweep of one projection in a loop shows
            const double lone = wide ? 0.17 : 0.13;
            // share of that rate a CU reaches with one resp. two work-groups of mt tiles
            static const double kOne[6] = {0, 0.56, 0.97, 0.94, 0.93, 0.98}, kTwo[6] = {0, 0.58, 0.82, 0.90, 0.96, 0.95};
            auto cu_rate = [&](int g) { return base * (g == 1 ? kOne[mt] : kTwo[mt]) * 1e6; };   // flop per microsecond
            for (int s = 1; s <= (allow_split ? max_splits : 1); ++s) {
                if (slices_all % (4 * s) != 0) continue;
                // splits whose fills are short: beyond five tiles of rows only the five-tile form of them is considered (up to
                // there a narrow strip has a form for every height; a wide one runs the five-tile form whatever its height)
                if ((K / s) % 128 != 0 && tiles > 5 && mt != 5) continue;
                const double slices = (double)slices_all / s;
                const double wg_flop = 2.0 * 32 * mt * cols * 16 * slices;
                const long long blocks = (long long)tiles_m * (N / cols) * s;
                auto round_time = [&](long long n) {                          // n work-groups dealt to the 256 CUs at once
                    const int g = (int)((n + 255) / 256);
                    return std::max(g * wg_flop / cu_rate(g), slices * lone * (1.0 + 0.373 * (g - 1)));
                };
                const long long cap = 256LL * per_cu, full = blocks / cap, rem = blocks % cap;
                double t = full * round_time(cap) + (rem ? round_time(rem) : 0.0);
                t = std::max(t, 2.0 * M * (double)N * K / 1198.0e6);          // the chip's sustained rate
                t = std::max(t, (double)N * K * 2.0 / 4.98e6);                // the weights, as ordinary loads bring them
                if (s > 1) t += (double)s * M * N * 4.0 / 5.4e6 + (double)(s - 1) * M * N * 4.0 / 4.0e6;   // planes written here, read by the consumer
                t += 2.3;
                if (t < best.us - 1e-9) best = WsPlan{s, wide != 0, mt, t, t, {}, {}};
            }
        }
    return best;
}

// The tall kernel and the strips request their operands straight into LDS, 16 bytes a lane; the weight-streaming kernel loads them into
// registers, which may start at any element.  It keeps operands that do not start at 16 bytes, at any number of rows.
bool direct_loads(const void* p) { return reinterpret_cast<uintptr_t>(p) % 16 == 0; }

// Launch plan of a packed projection: the weight-streaming kernel, or from more rows than one of its work-groups holds on the
// tall kernel where that is expected to take less.  Inside a step the weight-streaming launches
// take 1.10 times the estimate above, which was fitted to single projections in a loop (7B at 2304 rows: QKV 89 us against 78,
// down 282 against 263); the tall ones take theirs.
// Where the reduction is not split (LM heads) they take 1.1 to 1.3: every work-group along the rows reads its strip again.  us alone,
// weight-streaming against tall: 152064 x 3584 at 330 / 400 / 500 / 640 rows 445 / 498 / 549 / 681 against 392 / 411 / 446 / 543, 152064 x
// 5120 558 / 668 / 770 / 942 against 564 / 567 / 614 / 725.  Shorter ones (kHeadInputs) lie by the other line, as the weights read again are
// little beside the logits written: 151936 x 1024 at 161 / 192 / 256 rows 101 / 105 / 120 against 104 / 109 / 123, x 896 inside a step 20 less.
// us in a loop, weight-streaming against tall, 7B: QKV at 320 / 512 / 1280 / 2304 rows 21 / 30 / 52 / 98 against
// 24 / 23 / 43 / 71, down 48 / 83 / 180 / 282 against 54 / 65 / 152 / 243.
// tile_mode: -1 = this rule, 0 = the weight-streaming kernel only, 1 = 256-row tall tiles wherever the width allows.
// direct: weights that direct_loads takes.
WsPlan plan_wide(int M, int N, int K, bool allow_split, int tile_mode, bool direct, int max_splits = kMaxSplitsWs) {
    if (direct && tile_mode == 1 && N % 256 == 0) return WsPlan{1, true, 0, 0.0, 0.0, gemm_bf16_tall_256(M), {}};
    const WsPlan ws = plan_ws(M, N, K, allow_split, max_splits);
    if (!direct || tile_mode == 0 || M <= 128) return ws;
    const TallPlan t = gemm_bf16_tall_plan(M, N, K, allow_split ? std::min(max_splits, kMaxSplits) : 1);
    return t.us < (allow_split || K < kHeadInputs ? 1.10 : 1.25) * ws.us ? WsPlan{t.splits, true, 0, t.us, ws.us, t.tiles, {}} : ws;
}

// Up to 320 rows the narrow strips come in between.  Their estimate was fitted to launches on an idle chip; what they give inside a
// step, us of a layer against weight-streaming at 5 / 42 / 96 / 160 rows:
//   down 3584 x 18944 2.5 / 2.9 / 1.1 / 0.6 less, 5120 x 27648 1.7 / 5.7 / 8.9 / 1.4, 2048 x 11008 6.5 / 5.3 / 2.2 / 1.0, 896 x 4864 3.0 / 2.3 / 2.0 / 0.3; at
//   192 / 256 / 288 / 320 3584 x 18944 1.3 less / 1.2 more / 2.5 less / 0.2 more, 4096 x 14336 3.5 less / 3.0 more / - / 1.9 more.  From 161 rows
//   on a strip has to be expected ahead (8192 x 29568 at 320 rows 38 less; 8192 x 8192 and 4096 x 14336 there, 2.9 and 1.9 more of about 50,
//   are still among them)
//   QKV and O together, before the attention of 1 to 8 thousand keys, at 5 / 40 / 65 / 96 / 128 / 130 / 160 / 190 rows: 3584 inputs 0.4 / 0.9 / 0.8
//   less, 0.8 / 0.7 more, 2.1 / 2.6 less, 5.4 more; 4096 inputs 0.5 / 0.4 / 2.4 less, 1.0 more, 0.6 / 3.3 / 4.4 less, 2.0 more; 5120 inputs 1.4 / 1.0 / 0.1
//   less, 2.6 / 0.6 more, 2.4 / 1.9 less, 1.2 more; 2048 inputs (10 and 21 MB of QKV) 1.5 / 1.2 / 0.0 / 0.3 / 0.2 more, 0.6 less, 0.5 / 8.4 more and
//   0.3 less, 0.9 / 0.0 / 0.9 / 0.4 more, 0.3 less, 0.5 / 4.7 more
// so reductions of up to kStripInputs take strips for one, two and five row tiles, if their weights are a stream worth the name.
// LM heads of 97 to 320 rows: 152064 x 3584 at 112 / 160 / 192 / 320 7.9 / 5.9 / 51 / 39 less (up to 96 rows 0.8 to 4.4 less and, over 2048
// inputs, 1 to 4 more), where tall tiles are 48 and 12 less at 192 and 320; 151936 x 2048 within 2 of the tall tiles up to 256 rows and 7
// less at 320, 151936 x 1024 alone 5 to 13 less from 192 rows on, whatever the estimates say; where the strips are one round (225 of 50304 x
// 1024) and the tall estimate is lower, 6 to 8 more.
// Once more with weights read and planes left as streams, us a launch inside a step, weight-streaming against strip at 5 / 65 / 96 / 128 / 147 rows: LM heads
// 152064 x 3584 161 / 199 / 201 / 217 / - against 162 / 206 / 207 / 216 / 225, x 5120 229 / 276 / 279 / 288 / - against 227 / 285 / 290 / 297 / 312, 32000 x
// 2048 21.7 / 28.2 / 27.1 / 30.2 / 34.1 against 21.6 / 28.7 / 26.4 / 30.1 / 33.4; down 3584 x 18944 26.4 / 34.1 / 34.5 / 39.4 / - against 23.0 / 29.7 / 29.2 / 33.4 /
// -; QKV 4608 x 3584 7.4 / 12.4 / 12.7 / 14.0 / 16.2 against 7.3 / 12.3 / 14.3 / 16.6 / 17.4.  Those lines stand.  Not where strips lose now and are still
// taken: QKV 7168 x 5120 13.3 / 19.5 / 20.5 / 22.5 / 23.9 against 13.0 / 20.4 / 22.1 / 23.8 / 25.0, O 5120 x 5120 at 147 rows 18.0 against 20.7; down 2048 x 5632
// 6.7 / 9.1 / 9.4 / 13.0 / 12.0 against 6.4 / 11.0 / 11.6 / 14.0 / 14.6 (as before the streams).
// Other tall tiles: see plan_gate_up.
// experts: a model with a router, whose choices turn on the last bits of the rows: a strip keeps the splits of the launch that it
// replaces, and with them the bits.
bool strip_pays(int M, int N, int K) { return K > kStripInputs || ((int64_t)N * K >= 12000000 && (M <= 64 || (M > 128 && M <= 160))); }

WsPlan plan_packed(int M, int N, int K, bool allow_split, int tile_mode, bool experts, bool direct = true, int max_splits = kMaxSplitsWs) {
    WsPlan best = plan_wide(M, N, K, allow_split, tile_mode, direct, max_splits);
    if (direct && tile_mode != 0 && M >= 1 && M <= kStripRows && (!allow_split || strip_pays(M, N, K))) {
        const StripPlan s = gemm_bf16_strip_plan(M, N, K, experts ? best.splits : 1, experts ? best.splits : allow_split ? max_splits : 1, false);
        const bool tall_head = best.tall.n > 0 && gemm_bf16_strips(N, s.tile) <= 256 && s.us > 1.05 * best.us;
        const double limit = !allow_split ? (M <= 96 || tall_head ? 0.0 : 1.25 * best.ws_us) : best.tall.n > 0 ? 0.80 * best.us : (M <= 160 ? 1.15 : 0.93) * best.us;
        if (s.us < limit) best = WsPlan{s.splits, false, 0, s.us, best.ws_us, {}, s.tile};
    }
    return best;
}

// Gate/up projection with SwiGLU of T rows (N = 2 d_ff): up to five 32-row tiles strips or the weight-streaming kernel, from then on
// strips or tall tiles (one work-group of the weight-streaming kernel along the rows no longer holds them, and every further one
// reads the strip again).  Strips where they come to no more than the CUs and, from 161 rows on, are expected to be well ahead.  us of a
// layer inside steps, strip against weight-streaming at 5 / 96 / 160 rows: 18944 x 3584 1.6 / 8.6 / 9.6 less, 27648 x 5120 0.4 more / 1.2 / 3.4
// less, 14336 x 4096 11 / 14 / 48 less, 11008 x 2048 7 / 6 / 11 less; against tall at 192 / 256 / 320 18944 x 3584 11.9 / 6.0 / 5.0 less,
// 27648 x 5120 1.1 / 1.6 / 0.4 more, 14336 x 4096 14.2 / 2.8 less / 6.0 more (ten row tiles are estimated too low: 0.77 for 0.80 there).
// Two exceptions up to 160 rows.  More strips than CUs where the weight-streaming kernel's own strips of 128 features are still one
// round: 29568 x 8192 (462 against 231) 5.3 / 23 / 32 more, 30720 x 4096 alone 87 / 97 / 114 us against 86 / 90 / 101; with a second round in both,
// 33792, 40960 and 53248 x 4096 101 / 114 / 126, 115 / 122 / 139 and 151 / 161 / 174 against 128 / 140 / 124, 131 / 144 / 154 and 152 / 161 / 179.
// And 129 to 160 rows of so few features that the weight-streaming kernel's five 32-row tiles of every strip run at once: 4864 x 896 3.3
// more, alone 5120 and 6400 x 2048 26.4 and 25.9 against 23.2 and 23.4, but 7168 (56 strips) 26.8 against 31.1.
// The tall tiles against the weight-streaming kernel at 147 / 192 / 256 / 320 / 512 / 800 rows (in a loop): 65 / 66 / 77 / 98 / 144 / 218
// against 65 / 86 / 104 / 100 / 160 / 221.
struct GateUp { TallTiles tall; StripTile strip; };       // neither: the weight-streaming kernel
GateUp plan_gate_up(int T, int N, int K, int tile_mode, bool direct) {
    GateUp g{};
    if (!direct || tile_mode == 0 || N % 256 != 0) return g;
    if (tile_mode == 1) return GateUp{gemm_bf16_tall_256(T), {}};
    const StripPlan s = T <= kStripRows ? gemm_bf16_strip_plan(T, N, K, 1, 1, true) : StripPlan{1, {0, 4}, 1e30};
    const bool one_round = gemm_bf16_strips(N, s.tile) <= 256;
    bool strip;
    if (T > 160) {
        const TallPlan t = gemm_bf16_tall_plan(T, N, K, 1);
        g.tall = t.tiles;
        strip = one_round && s.us < (T > 256 ? 0.77 : 0.80) * t.us;
    } else {
        strip = s.us < 1e29 && (one_round || N / 256 > 256) && (T <= 128 || 5 * (N / 256) > 256);
    }
    return strip ? GateUp{{}, s.tile} : g;
}

struct Layout {                       // byte offsets into the workspace
    size_t seq_len, page_table, stage, row_info, row_part, row_slot, stat_part, draw_part;
    size_t rope, h, a_norm, q, attn, part, act, logits, part_o, part_ml, total;
    size_t moe_ids, moe_w, moe_live, moe_off, moe_perm, moe_inv, moe_act, moe_y, moe_logits;   // mixture-of-experts scratch
    int T, P;                         // rows of a step, rows of a pass (a prefill pass may hold more)
    int max_chunks, max_items, max_upd;
    size_t part_floats;               // capacity of part
    long long part_rows;              // capacity of part_o / part_ml
    int st_seq, st_req, st_work, st_upd;   // ints from the start of the staged block: sequence ids, requests, work items, page updates
    int st_total;
};

// Rows of partial router logits: four parts of a pass, and sixteen of one operand tile (see moe_ffn).
long long router_rows(int pass_rows) { return std::max(4LL * pass_rows, 16LL * 32); }

// prefill_rows: rows that a prefill pass shall hold, where the cache, the limit above and the expert kernels allow
bool make_layout(const sv_model& m, const sv_runtime& r, int prefill_rows, Layout& L) {
    if (r.max_batch <= 0 || r.max_k < 0 || r.max_chains <= 0 || r.max_seqs <= 0 || r.page_size <= 0 ||
        r.page_size % kVBlk != 0 || r.num_pages <= 0 || r.max_pages_per_seq <= 0 || r.max_batch > 32767 ||
        (size_t)r.max_pages_per_seq * r.page_size / kChunkKeys > 65535)
        return false;
    const size_t es = m.dtype == SV_BF16 ? 2 : 4;
    const int T = r.max_batch * (1 + r.max_chains * r.max_k);
    const int qw = m.n_q_heads * m.head_dim, qkvw = (m.n_q_heads + 2 * m.n_kv_heads) * m.head_dim;
    const int F = m.n_experts ? m.d_expert : m.d_ff;
    const int G = m.n_q_heads / std::max(1, m.n_kv_heads);
    int extra = (int)std::min<long long>(std::min(kPrefillRows, prefill_rows), (long long)r.num_pages * r.page_size);   // no more than the cache holds
    if (m.n_experts > 0)
        while (extra > T && !moe_shape_ok(extra, m.d_model, m.n_experts, m.top_k, m.d_expert)) extra -= std::min(extra - T, 256);
    const int P = std::max(T, extra);
    size_t o = 0;
    auto take = [&](size_t bytes) { size_t at = o; o += align_up(bytes); return at; };
    L.T = T;
    L.P = P;
    L.seq_len = take(sizeof(int32_t) * r.max_seqs);
    L.page_table = take(sizeof(int32_t) * (size_t)r.max_seqs * r.max_pages_per_seq);
    L.max_chunks = (int)(((size_t)r.max_pages_per_seq * r.page_size + kChunkKeys - 1) / kChunkKeys);
    L.max_items = r.max_batch * L.max_chunks + P * G / kItemRows + r.max_batch + 2048;
    L.max_upd = std::max(8 * r.max_batch, P / r.page_size + 2 * r.max_batch);
    L.st_seq = 4;                                          // (the first int: the number of work items)
    L.st_req = L.st_seq + (r.max_batch + 3) / 4 * 4;
    L.st_work = L.st_req + kReqInts * r.max_batch;
    L.st_upd = L.st_work + kItemInts * L.max_items;
    L.st_total = L.st_upd + 3 * L.max_upd;
    L.stage = take(sizeof(int32_t) * (size_t)L.st_total);
    L.row_info = take(sizeof(int32_t) * 4 * (size_t)P);
    L.row_part = take(sizeof(int32_t) * 4 * (size_t)P);
    L.row_slot = take(sizeof(int32_t) * P);
    L.stat_part = take(sizeof(float) * 4 * sample_part_entries(T));
    L.draw_part = take(sizeof(float) * 4 * sample_part_entries(T));
    L.rope = take(sizeof(float) * (size_t)P * m.head_dim);
    L.h = take(sizeof(float) * (size_t)P * m.d_model);
    const size_t Tp = (size_t)(P + 31) / 32 * 32;          // packed activations come in 32-row tiles
    L.a_norm = take(es * Tp * m.d_model);
    L.q = take(es * (size_t)P * qw);
    L.attn = take(es * Tp * qw);
    // split-K partial products: the most splits * rows * features a projection's plan asks for at any number of row
    // tiles (a plan between two of these sizes that would ask for more is made again with fewer splits).  The gate/up
    // product passes through here in row-major bf16 models only, the others have SwiGLU in its epilogue: it is given room
    // for a step's rows, and a prefill pass of such a model takes as many as that holds (see pass_rows).
    size_t part = 0;
    const int shapes[3][2] = {{qkvw, m.d_model}, {m.d_model, qw}, {m.d_model, F}};
    for (int tm = 1; tm <= (P + 127) / 128; ++tm) {
        const int M = std::min(tm * 128, P);
        for (auto& sh : shapes)
            part = std::max(part, (size_t)(m.dtype == SV_BF16 ? pick_splits(M, sh[0], sh[1]) : 1) * M * sh[0]);
        if (m.dtype == SV_BF16 && m.n_experts == 0) {
            const int Ms = std::min(M, T);
            part = std::max(part, (size_t)pick_splits(Ms, 2 * F, m.d_model) * Ms * 2 * F);
        }
    }
    if (m.dtype == SV_BF16)                                 // the same for the plans of packed weights
        for (int tm = 1; tm <= (P + 31) / 32; ++tm) {
            const int M = std::min(tm * 32, P);
            for (auto& sh : shapes)
                if (sh[1] % 64 == 0) part = std::max(part, (size_t)plan_packed(M, sh[0], sh[1], true, -1, m.n_experts > 0).splits * M * sh[0]);
        }
    L.part_floats = part;
    L.part = take(sizeof(float) * part);
    L.act = take(es * Tp * F);
    L.logits = take(sizeof(float) * (size_t)T * m.vocab);
    // the MFMA attention stacks G * n rows per kv head and keeps the partials of a request cut into pieces
    const int rows_pad = std::max(64, std::min(kStepRows, (G * (1 + r.max_chains * r.max_k) + 15) / 16 * 16));
    L.part_rows = (long long)r.max_batch * m.n_kv_heads * L.max_chunks * rows_pad;
    // a prefill cuts keys only where its items are few: kPrefillPlaces of them at most, pieces counted (see build_work)
    if (attn_mfma_ok(m.dtype, m.head_dim, r.page_size, false, 0))
        L.part_rows = std::max(L.part_rows, std::min(2LL * (P * m.n_q_heads + kItemRows * m.n_kv_heads), (long long)kPrefillPlaces * kItemRows));
    if (L.part_rows > 0x7fffffffLL) return false;          // partial rows are numbered in 32 bits
    L.part_o = take(sizeof(float) * (size_t)L.part_rows * m.head_dim);
    L.part_ml = take(sizeof(float) * (size_t)L.part_rows * 2);
    L.moe_ids = L.moe_w = L.moe_live = L.moe_off = L.moe_perm = L.moe_inv = L.moe_act = L.moe_y = L.moe_logits = 0;
    if (m.n_experts > 0) {
        const size_t tiles = (size_t)moe_max_tiles(P, m.n_experts, m.top_k);
        L.moe_ids = take(sizeof(int32_t) * (size_t)P * m.top_k);
        L.moe_w = take(sizeof(float) * (size_t)P * m.top_k);
        L.moe_live = take(sizeof(int32_t) * (2 + 2 * (size_t)m.n_experts));
        L.moe_off = take(sizeof(int32_t) * (m.n_experts + 1));
        L.moe_perm = take(sizeof(int32_t) * 32 * tiles);
        L.moe_inv = take(sizeof(int32_t) * (size_t)P * m.top_k);
        L.moe_act = take(es * 32 * tiles * m.d_expert);
        L.moe_y = take(sizeof(float) * 32 * tiles * m.d_model);
        L.moe_logits = take(sizeof(float) * (size_t)router_rows(P) * m.n_experts);
    }
    L.total = o;
    return true;
}

bool model_ok(const sv_model& m) {
    return m.n_layers > 0 && m.d_model > 0 && m.n_q_heads > 0 && m.n_kv_heads > 0 && m.head_dim > 0 &&
           m.head_dim % 2 == 0 && m.vocab > 0 && m.n_q_heads % m.n_kv_heads == 0 &&
           (m.dtype == SV_FP32 || m.dtype == SV_BF16) && (m.n_experts > 0 || m.d_ff > 0);
}

__global__ void apply_page_updates_kernel(int32_t* page_table, int mpps, const int32_t* upd, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) page_table[(int64_t)upd[3 * i] * mpps + upd[3 * i + 1]] = upd[3 * i + 2];
}

constexpr int kLenPairs = 240;        // (sequence, length) pairs that travel as one launch's arguments
struct LenPairs { int32_t v[2 * kLenPairs]; };
__global__ void set_lens_kernel(int32_t* seq_len, LenPairs pairs, int n) {
    const int i = threadIdx.x;
    if (i < n) seq_len[pairs.v[2 * i]] = pairs.v[2 * i + 1];
}

}  // namespace

struct sv_ctx {
    sv_model model;
    sv_runtime rt;
    std::vector<const void*> ln1, wqkv, wo, ln2, wgu, wdown, wrouter;
    const void *embed, *lm_head, *final_norm;
    hipStream_t stream;
    Layout lay;
    KvGeom geom;
    char* ws;
    std::vector<SeqState> seqs;
    std::vector<int32_t> free_pages;
    int32_t* staging[kRing];
    hipEvent_t staged[kRing];
    bool staged_valid[kRing];
    int ring_pos;
    int n_work;                                           // attention work items staged for the current pass
    int n_last_work;                                      // prefill: items behind them that hold the last rows asked for; -1: no room for the list
    bool pass_merge;                                      // some request of it has its keys cut into several pieces
    bool four_waves, last_four_waves;                     // prefill: waves of the work-groups over these items, over those behind them
    size_t weight_bytes, expert_bytes;                    // of all layers and the LM head; of one expert in all layers
    bool cold;                                            // what the current pass reads once comes from HBM (see kCacheBytes)
    int gemm_variant;                                     // -1 = choose per shape
    int gemm_tile;                                        // packed projections: -1 = by the plans, 0 = weight-streaming kernel only, 1 = tall tiles wherever the shape allows
    struct PlannedShape { int M, N, K; bool allow_split, direct; WsPlan plan; };
    std::vector<PlannedShape> plans;                      // launch plans of packed projections made so far, at most kPlans
    struct PlannedGateUp { int T; bool direct; GateUp launch; };
    std::vector<PlannedGateUp> gate_up;                   // the same for the gate/up projection
    bool packed;                                          // projection weights are in fragment order
    int pass_rows;                                        // most rows of a prefill pass
    bool attn_generic;
    int attn_min_rt;
    int attn_max_rt;
    bool use_graph;                                       // replay verify_step's device work from captured graphs
    bool graph_launch_shape;                              // launches take shapes that do not depend on the lengths
    struct GraphEntry {
        int B, k, N;
        const void* ptr[9];
        hipGraphExec_t exec;
        unsigned long long used;
    };
    std::vector<GraphEntry> graphs;
    unsigned long long graph_clock;
    int attn_chunk_opt;                                   // 0 = chosen per batch, else fixed by option
    unsigned prof_mask;                                   // kinds of kernels to time with events
    struct ProfRec { int kind; hipEvent_t a, b; };
    std::vector<ProfRec> prof_recs;                       // recorded, not yet read
    std::vector<hipEvent_t> prof_free;                    // event pool
    std::string err;

    template <typename T> T* at(size_t off) const { return reinterpret_cast<T*>(ws + off); }
    int fail(int code, const char* fmt, ...) {
        char buf[512];
        va_list ap;
        va_start(ap, fmt);
        vsnprintf(buf, sizeof buf, fmt, ap);
        va_end(ap);
        err = buf;
        return code;
    }
    int hip(hipError_t e, const char* what) {
        if (e == hipSuccess) return SV_OK;
        return fail(SV_EHIP, "%s: %s", what, hipGetErrorString(e));
    }
};

// Brackets the launches of one kind with a pair of events on the context's stream when that kind is
// being profiled.
struct ProfScope {
    sv_ctx* c; int kind; bool on; hipEvent_t a;
    ProfScope(sv_ctx* c_, int kind_) : c(c_), kind(kind_), on(((c_->prof_mask >> kind_) & 1u) != 0), a(nullptr) {
        if (!on) return;
        a = take();
        if (a) (void)hipEventRecord(a, c->stream); else on = false;
    }
    ~ProfScope() {
        if (!on) return;
        hipEvent_t b = take();
        if (!b) { c->prof_free.push_back(a); return; }
        (void)hipEventRecord(b, c->stream);
        c->prof_recs.push_back({kind, a, b});
    }
    hipEvent_t take() {
        if (!c->prof_free.empty()) { hipEvent_t e = c->prof_free.back(); c->prof_free.pop_back(); return e; }
        hipEvent_t e = nullptr;
        return hipEventCreate(&e) == hipSuccess ? e : nullptr;
    }
};

#define SV_TRY(expr)                    \
    do {                                \
        int _rc = (expr);               \
        if (_rc != SV_OK) return _rc;   \
    } while (0)
#define SV_HIP(ctx, expr) SV_TRY((ctx)->hip((expr), #expr))

// Rows of a prefill pass: what the workspace is laid out for, in row-major bf16 models no more than leave the gate/up product
// room in the split-K planes.
static int pass_rows(const sv_ctx* c) {
    const sv_model& m = c->model;
    if (m.dtype != SV_BF16 || c->packed) return c->lay.P;
    int rows = c->lay.T;
    for (int tm = 1; rows < c->lay.P; ++tm) {
        const int M = std::min(tm * 128, c->lay.P);
        if (M > c->lay.T && (size_t)pick_splits(M, 2 * m.d_ff, m.d_model) * M * 2 * m.d_ff > c->lay.part_floats) break;
        rows = std::max(rows, M);
    }
    return rows;
}

static KvGeom make_geom(const sv_model& m, const sv_runtime& r) {
    KvGeom g;
    g.n_kv_heads = m.n_kv_heads;
    g.head_dim = m.head_dim;
    g.page_size = r.page_size;
    g.page_elems = (int64_t)2 * m.n_kv_heads * r.page_size * m.head_dim;
    g.layer_elems = (int64_t)r.num_pages * g.page_elems;
    return g;
}

extern "C" size_t verify_kv_pool_bytes(const sv_model* m, const sv_runtime* r) {
    if (!m || !r || !model_ok(*m) || r->num_pages <= 0 || r->page_size <= 0) return 0;
    const KvGeom g = make_geom(*m, *r);
    return (size_t)m->n_layers * g.layer_elems * (m->dtype == SV_BF16 ? 2 : 4);
}

extern "C" size_t sv_workspace_bytes(const sv_model* m, const sv_runtime* r, int32_t prefill_rows) {
    Layout L;
    if (!m || !r || !model_ok(*m) || !make_layout(*m, *r, std::max(0, prefill_rows), L)) return 0;
    return L.total;
}

extern "C" size_t verify_workspace_bytes(const sv_model* m, const sv_runtime* r) { return sv_workspace_bytes(m, r, 0); }

// The layout with the most prefill rows, in whole 32-row tiles, that a workspace of the given size holds; false if it does
// not hold a step's rows.
static bool fit_layout(const sv_model& m, const sv_runtime& r, size_t bytes, Layout& L) {
    if (make_layout(m, r, kPrefillRows, L) && L.total <= bytes) return true;
    if (!make_layout(m, r, 0, L) || L.total > bytes) return false;
    int fits = 0, over = kPrefillRows / 32;
    while (over - fits > 1) {
        const int mid = (fits + over) / 2;
        Layout t;
        if (make_layout(m, r, 32 * mid, t) && t.total <= bytes) { fits = mid; L = t; } else over = mid;
    }
    return true;
}

extern "C" int verify_init(const sv_model* m, const sv_weights* w, const sv_runtime* r, void* hip_stream, sv_ctx** out) {
    if (!m || !w || !r || !out) return SV_EINVAL;
    *out = nullptr;
    Layout L;
    if (!model_ok(*m) || !fit_layout(*m, *r, r->workspace_bytes, L)) return SV_EINVAL;
    if (!r->kv_pool || !r->workspace || r->kv_pool_bytes < verify_kv_pool_bytes(m, r) ||
        ((uintptr_t)r->kv_pool & 255) || ((uintptr_t)r->workspace & 255))
        return SV_EINVAL;
    if (!(r->temperature > 0.f) || r->verify_mode < 0 || r->verify_mode > 2 || r->sample_mode < 0 || r->sample_mode > 1)
        return SV_EINVAL;
    if (!w->embed || !w->lm_head || !w->final_norm || !w->ln1 || !w->wqkv || !w->wo || !w->ln2 || !w->w_gate_up || !w->w_down)
        return SV_EINVAL;
    if (m->n_experts > 0) {
        // mixture-of-experts FFN: bf16 with packed weights only, within the expert kernels' shape cover
        if (m->dtype != SV_BF16 || !w->packed || !w->w_router) return SV_EUNSUPPORTED;
        if (!moe_shape_ok(L.T, m->d_model, m->n_experts, m->top_k, m->d_expert)) return SV_EUNSUPPORTED;
    }
    if (w->packed && m->dtype != SV_BF16) return SV_EINVAL;        // only bf16 projections have a packed form
    if (m->head_dim != 64 && m->head_dim != 128) return SV_EUNSUPPORTED;
    if (m->d_model % 4 != 0 || m->d_model > 8192) return SV_EUNSUPPORTED;   // RMSNorm kernel: float4 pieces, <= 8 per thread
    if (m->dtype == SV_BF16) {
        const int qw = m->n_q_heads * m->head_dim, qkvw = (m->n_q_heads + 2 * m->n_kv_heads) * m->head_dim;
        if (!gemm_bf16_shape_ok(qkvw, m->d_model, 1) || !gemm_bf16_shape_ok(m->d_model, qw, 1) ||
            (m->n_experts == 0 && (!gemm_bf16_shape_ok(2 * m->d_ff, m->d_model, 1) || !gemm_bf16_shape_ok(m->d_model, m->d_ff, 1))) ||
            !gemm_bf16_shape_ok(m->vocab, m->d_model, 1))
            return SV_EUNSUPPORTED;                                // GEMM N must be a multiple of 128, K of 64
    }
    sv_ctx* c = new sv_ctx();
    c->model = *m;
    c->rt = *r;
    c->lay = L;
    c->geom = make_geom(*m, *r);
    c->ws = reinterpret_cast<char*>(r->workspace);
    c->stream = reinterpret_cast<hipStream_t>(hip_stream);
    c->embed = w->embed; c->lm_head = w->lm_head; c->final_norm = w->final_norm;
    for (int l = 0; l < m->n_layers; ++l) {
        if (!w->ln1[l] || !w->wqkv[l] || !w->wo[l] || !w->ln2[l] || !w->w_gate_up[l] || !w->w_down[l] ||
            (m->n_experts > 0 && !w->w_router[l])) {
            delete c;
            return SV_EINVAL;
        }
        c->ln1.push_back(w->ln1[l]); c->wqkv.push_back(w->wqkv[l]); c->wo.push_back(w->wo[l]);
        c->ln2.push_back(w->ln2[l]); c->wgu.push_back(w->w_gate_up[l]); c->wdown.push_back(w->w_down[l]);
        c->wrouter.push_back(w->w_router ? w->w_router[l] : nullptr);
    }
    c->seqs.resize(r->max_seqs);
    c->free_pages.resize(r->num_pages);
    for (int i = 0; i < r->num_pages; ++i) c->free_pages[i] = r->num_pages - 1 - i;   // pop_back yields 0,1,2..
    {
        const size_t es = m->dtype == SV_BF16 ? 2 : 4, layers = m->n_layers, d = m->d_model;
        c->expert_bytes = m->n_experts > 0 ? es * layers * 3 * m->d_expert * d : 0;
        c->weight_bytes = es * (layers * (2 * (size_t)(m->n_q_heads + m->n_kv_heads) * m->head_dim + (m->n_experts > 0 ? 0 : 3 * (size_t)m->d_ff)) * d + (size_t)m->vocab * d);
    }
    c->cold = false;
    c->ring_pos = 0;
    c->gemm_variant = -1;
    c->gemm_tile = -1;
    c->packed = w->packed != 0;
    c->pass_rows = pass_rows(c);
    c->attn_generic = false;
    c->attn_min_rt = 1;
    c->use_graph = false;
    c->graph_launch_shape = false;
    c->graph_clock = 0;
    c->attn_max_rt = 4;
    c->attn_chunk_opt = 0;
    c->prof_mask = 0;
    const size_t slot_ints = L.st_total;
    for (int i = 0; i < kRing; ++i) { c->staging[i] = nullptr; c->staged[i] = nullptr; c->staged_valid[i] = false; }
    for (int i = 0; i < kRing; ++i) {
        if (hipHostMalloc(reinterpret_cast<void**>(&c->staging[i]), slot_ints * sizeof(int32_t), hipHostMallocDefault) != hipSuccess ||
            hipEventCreateWithFlags(&c->staged[i], hipEventDisableTiming) != hipSuccess) {
            verify_destroy(c);
            return SV_EHIP;
        }
    }
    // lengths and page table start at zero; an uninitialised pool could hold NaN patterns, which a
    // masked-out key would still feed into the PV product (0 * NaN), so the pool is cleared once.
    if (hipMemsetAsync(c->ws, 0, L.rope, c->stream) != hipSuccess ||
        hipMemsetAsync(r->kv_pool, 0, verify_kv_pool_bytes(m, r), c->stream) != hipSuccess) {
        verify_destroy(c);
        return SV_EHIP;
    }
    *out = c;
    return SV_OK;
}

static void drop_graphs(sv_ctx* c);

extern "C" void verify_destroy(sv_ctx* c) {
    if (!c) return;
    (void)hipStreamSynchronize(c->stream);
    drop_graphs(c);
    for (auto& r : c->prof_recs) { (void)hipEventDestroy(r.a); (void)hipEventDestroy(r.b); }
    for (hipEvent_t e : c->prof_free) (void)hipEventDestroy(e);
    for (int i = 0; i < kRing; ++i) {
        if (c->staging[i]) (void)hipHostFree(c->staging[i]);
        if (c->staged[i]) (void)hipEventDestroy(c->staged[i]);
    }
    delete c;
}

extern "C" const char* verify_last_error(const sv_ctx* c) { return c ? c->err.c_str() : "null context"; }

// ------------------------------------------------------------ sequences ---

static int pages_for(const sv_ctx* c, int len) { return (len + c->rt.page_size - 1) / c->rt.page_size; }

extern "C" int verify_seq_add(sv_ctx* c, int32_t id, int32_t cached_len) {
    if (!c) return SV_EINVAL;
    if (id < 0 || id >= c->rt.max_seqs) return c->fail(SV_ENOSEQ, "sequence id %d out of range", id);
    if (c->seqs[id].live) return c->fail(SV_ENOSEQ, "sequence id %d already live", id);
    const int need = pages_for(c, cached_len);
    if (cached_len < 0 || need > c->rt.max_pages_per_seq)
        return c->fail(SV_EINVAL, "cached_len %d exceeds max_pages_per_seq", cached_len);
    if (need > (int)c->free_pages.size()) return c->fail(SV_ENOPAGES, "need %d pages, %zu free", need, c->free_pages.size());
    SeqState& s = c->seqs[id];
    std::vector<int32_t> pages;
    for (int i = 0; i < need; ++i) { pages.push_back(c->free_pages.back()); c->free_pages.pop_back(); }
    hipError_t e = hipSuccess;
    if (need) e = hipMemcpyAsync(c->at<int32_t>(c->lay.page_table) + (size_t)id * c->rt.max_pages_per_seq, pages.data(),
                                 need * sizeof(int32_t), hipMemcpyHostToDevice, c->stream);
    if (e == hipSuccess) e = set_i32(c->at<int32_t>(c->lay.seq_len) + id, cached_len, c->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(c->stream);     // `pages` is a temporary
    if (e != hipSuccess) {
        for (int32_t p : pages) c->free_pages.push_back(p);
        return c->hip(e, "verify_seq_add");
    }
    s.live = true; s.len_ub = cached_len; s.pages.swap(pages);
    return SV_OK;
}

extern "C" int verify_seq_remove(sv_ctx* c, int32_t id) {
    if (!c) return SV_EINVAL;
    if (id < 0 || id >= c->rt.max_seqs || !c->seqs[id].live) return c->fail(SV_ENOSEQ, "sequence id %d not live", id);
    SeqState& s = c->seqs[id];
    for (int32_t p : s.pages) c->free_pages.push_back(p);
    s = SeqState();
    return SV_OK;
}

extern "C" int verify_seq_set_len(sv_ctx* c, int32_t id, int32_t len) {
    if (!c) return SV_EINVAL;
    if (id < 0 || id >= c->rt.max_seqs || !c->seqs[id].live) return c->fail(SV_ENOSEQ, "sequence id %d not live", id);
    SeqState& s = c->seqs[id];
    if (len < 0 || len > (int)s.pages.size() * c->rt.page_size)
        return c->fail(SV_EINVAL, "length %d beyond the %zu pages held", len, s.pages.size());
    SV_HIP(c, set_i32(c->at<int32_t>(c->lay.seq_len) + id, len, c->stream));
    s.len_ub = len;
    return SV_OK;
}

extern "C" int verify_seq_len(sv_ctx* c, int32_t id, int32_t* len_out) {
    if (!c || !len_out) return SV_EINVAL;
    if (id < 0 || id >= c->rt.max_seqs || !c->seqs[id].live) return c->fail(SV_ENOSEQ, "sequence id %d not live", id);
    int32_t len = 0;
    SV_HIP(c, hipMemcpyAsync(&len, c->at<int32_t>(c->lay.seq_len) + id, sizeof len, hipMemcpyDeviceToHost, c->stream));
    SV_HIP(c, hipStreamSynchronize(c->stream));
    SeqState& s = c->seqs[id];
    s.len_ub = len;
    const int keep = pages_for(c, len);
    while ((int)s.pages.size() > keep) { c->free_pages.push_back(s.pages.back()); s.pages.pop_back(); }
    *len_out = len;
    return SV_OK;
}

static int kv_io(sv_ctx* c, int32_t id, int32_t layer, int32_t pos0, int32_t n, void* k, void* v, bool to_pool) {
    if (!c || !k || !v) return SV_EINVAL;
    if (id < 0 || id >= c->rt.max_seqs || !c->seqs[id].live) return c->fail(SV_ENOSEQ, "sequence id %d not live", id);
    if (layer < 0 || layer >= c->model.n_layers || pos0 < 0 || n < 0 ||
        pos0 + n > (int)c->seqs[id].pages.size() * c->rt.page_size)
        return c->fail(SV_EINVAL, "kv range [%d,%d) of layer %d outside the pages held", pos0, pos0 + n, layer);
    SV_HIP(c, kv_copy(c->rt.kv_pool, c->geom, layer, c->at<int32_t>(c->lay.page_table) + (size_t)id * c->rt.max_pages_per_seq,
                      pos0, n, k, v, c->model.dtype, to_pool, c->stream));
    return SV_OK;
}
extern "C" int verify_kv_write(sv_ctx* c, int32_t id, int32_t layer, int32_t pos0, int32_t n, const void* k, const void* v) {
    return kv_io(c, id, layer, pos0, n, const_cast<void*>(k), const_cast<void*>(v), true);
}
extern "C" int verify_kv_read(sv_ctx* c, int32_t id, int32_t layer, int32_t pos0, int32_t n, void* k, void* v) {
    return kv_io(c, id, layer, pos0, n, k, v, false);
}

// ---------------------------------------------------------- forward pass ---

// What a pass takes from one request: n rows of its sequence; in a prefill they are columns col0 .. col0+n-1 of prompt pb.
struct PassReq { int32_t seq; int n, pb, col0; };
struct Pass {
    const PassReq* rq; int B;
    int n;                            // rows of every request; 0: they differ (prefill)
    int n_max, T, k;
    int last;                         // prefill: requests, the first ones, whose last rows' logits are wanted; else -1
};

// A slot of the pinned staging ring, free to be written.
static int take_slot(sv_ctx* c, int& slot) {
    slot = c->ring_pos;
    if (c->staged_valid[slot]) SV_HIP(c, hipEventSynchronize(c->staged[slot]));
    return SV_OK;
}
static int release_slot(sv_ctx* c, int slot) {
    SV_HIP(c, hipEventRecord(c->staged[slot], c->stream));
    c->staged_valid[slot] = true;
    c->ring_pos = (slot + 1) % kRing;
    return SV_OK;
}

// Pieces of less than kChunkKeys are for the last few requests of a rollout, and at most kFinePieces of them each (a
// captured launch has its grid sized for the most pieces there can be).
constexpr int kFinePieces = 64;
static bool fine_pieces_ok(const sv_ctx* c, int B) { return B * c->model.n_kv_heads <= 128; }
static int pieces_of(const sv_ctx* c, int total, int chunk) {
    return std::max(1, std::min((total + chunk - 1) / chunk, chunk < kChunkKeys ? kFinePieces : c->lay.max_chunks));
}

// Microseconds of an attention launch over pieces of the given keys, each standing for `alike` work-groups (the kv heads and
// row groups of a piece), longest first.  The work-groups that are resident share the stream (11500 keys of one head per us over
// the chip, 5.9 TB/s; a row group's second reader finds them in L2), none of them faster than it streams by itself; whenever
// one ends the next starts.  So a launch that begins with all its pieces in place is not as long as its longest piece at an
// even share: what ends leaves its share to the others.  Since all resident pieces advance alike, one clock of keys per piece
// serves them all.
// Constants by row tiles, fitted to 182 launches of 14 batches and, from four tiles on, 58 of seven handfuls of requests on
// MI355X: places (work-groups resident), keys per us of a work-group with a CU to itself and of two on a CU, keys' worth of
// start-up and merge per piece.  The sizes chosen were within 0.3 % of the best measured on average (2.3 % at most); list
// scheduling of even shares, before, 3.4 % (8.8): 64 requests of 1024-8192 keys 150 -> 138 us, 21 of 2000-9000 with 8 kv heads
// 136 -> 126, 96 with one row each 178 -> 172.
struct AttnPace { int places; double alone, paired, extra, stream; };
static AttnPace attn_pace(int row_tiles) {
    static const AttnPace k[4] = {{512, 70, 35, 75, 11500}, {256, 70, 70, 150, 11500}, {256, 70, 70, 400, 11500}, {512, 51, 40, 300, 11500}};
    AttnPace p = k[std::min(row_tiles, 4) - 1];
    const int groups = (row_tiles + 3) / 4;
    p.stream *= groups;
    if (groups > 1 && (row_tiles + groups - 1) / groups == 3) { p.alone *= 1.27; p.paired *= 1.27; }      // three tiles a work-group
    return p;
}
static double attn_launch_us(const std::vector<int>& lens, int alike, const AttnPace& pace, std::vector<double>& ends) {
    const size_t room = std::max(1, pace.places / alike);
    const auto later = std::greater<double>();
    ends.clear();
    double clock = 0.0, t = 0.0;
    size_t i = 0;
    while (i < lens.size() && ends.size() < room) { ends.push_back(lens[i++] + pace.extra); std::push_heap(ends.begin(), ends.end(), later); }
    while (!ends.empty()) {
        const double wgs = (double)ends.size() * alike;
        std::pop_heap(ends.begin(), ends.end(), later);
        const double end = ends.back();
        t += (end - clock) / std::min(wgs <= 256 ? pace.alone : pace.paired, pace.stream / wgs);
        clock = end;
        if (i < lens.size()) { ends.back() = clock + lens[i++] + pace.extra; std::push_heap(ends.begin(), ends.end(), later); }
        else ends.pop_back();
    }
    return t;
}

// The same by list scheduling, in keys of a CU's share of the stream: every piece goes to the place that frees up first.
static double attn_list_keys(const std::vector<int>& lens, int kv_heads, std::vector<double>& places) {
    const auto later = std::greater<double>();
    places.assign(std::max(1, 256 / kv_heads), 0.0);
    for (int len : lens) {
        std::pop_heap(places.begin(), places.end(), later);
        places.back() += len + 300.0;
        std::push_heap(places.begin(), places.end(), later);
    }
    return *std::max_element(places.begin(), places.end());
}

// Keys per piece for a step's attention, unless fixed by option: each candidate's launch is played through and the shortest
// wins.
//  - Up to 128 (request, kv head) pairs of up to three row tiles, the last few requests of a rollout, a launch of 256
//    work-groups at most does not share the stream with enough others to be bound by it: a lone one works off some 98 keys
//    per us, so fine pieces are better.  Estimate, in keys of a CU's share (46 per us): 300 per launch for start-up and merge.
//    One request of 6000 keys: pieces of 1024 take 22.2 + 7.2 us per layer (attention + merge), fine ones 13.4 + 5.2; seven
//    requests of 900-5000 keys 23.8 + 6.0 against 21.4 + 4.9.
//  - Else as above; a cut costs the merge launch as well.
//  - Models with experts keep the pieces of 1024 keys and more and the coarser estimate that they were first run with.  Neither
//    order of the sums is the more exact one, but where a row's last kept and first dropped expert are close another order
//    picks the other expert, and with the few rows of such a step that is 1-3 % of the logits (20 rows over 406-486 keys,
//    eight inputs: 0.005-0.030 between pieces of 128 and of 1024 keys, 0.000-0.009 with the same pieces), as much as the
//    path's results are held to from one version of the kernels to the next.  The price is 6 us of a layer's attention
//    at five requests of 700-3000 keys (14.9 -> 20.7).
static int pick_chunk(const sv_ctx* c, const Pass& ps) {
    if (c->attn_chunk_opt) return c->attn_chunk_opt;
    const int Hkv = c->model.n_kv_heads, G = c->model.n_q_heads / Hkv;
    const int row_groups = (G * ps.n_max + kItemRows - 1) / kItemRows, alike = Hkv * row_groups;
    const int row_tiles = (G * ps.n_max + 15) / 16;
    const AttnPace pace = attn_pace(row_tiles);
    const bool experts = c->model.n_experts > 0, few = !experts && fine_pieces_ok(c, ps.B);
    int chunk = kChunkKeys;
    double best = 1e300;
    std::vector<int> lens;
    std::vector<double> ends;
    for (int cand : {128, 256, 384, 512, 768, 1024, 1280, 1536, 2048, 2560, 3072, 4096, 5120, 6144, 8192, 12288, 16384, 24576, 32768}) {
        if ((cand < kChunkKeys && !few) || (experts && (cand == 1280 || cand == 2560 || cand == 5120))) continue;
        lens.clear();
        int most = 0;
        for (int b = 0; b < ps.B; ++b) {
            const int total = c->seqs[ps.rq[b].seq].len_ub + ps.rq[b].n;
            const int nch = pieces_of(c, total, cand);
            most = std::max(most, nch);
            for (int ch = 0; ch < nch; ++ch) lens.push_back((total + nch - 1) / nch);
        }
        const double wgs = (double)lens.size() * alike;
        double us;
        if (few && row_tiles <= 3 && wgs <= 256) {
            us = (300.0 + *std::max_element(lens.begin(), lens.end()) * std::max(0.47, wgs / 256.0) + 7.0 * (most > 1 ? most : 0)) / 46.0;
        } else if (experts) {
            std::sort(lens.begin(), lens.end(), std::greater<int>());
            us = attn_list_keys(lens, Hkv, ends);
        } else {
            if (most > 1 && wgs > 6.0 * pace.places && cand < 32768) continue;       // so many rounds of pieces only cost
            std::sort(lens.begin(), lens.end(), std::greater<int>());
            us = attn_launch_us(lens, alike, pace, ends) + (most > 1 ? 6.0 + 0.1 * most : 0.0);
        }
        if (us < best) { best = us; chunk = cand; }
        if (most == 1) break;                              // coarser candidates cut nothing either
    }
    return chunk;
}

// The attention's work list: every (request, piece of its keys) -- in a prefill (request, 64 stacked rows, piece) --
// that can exist given the upper bounds of the lengths, longest first (the hardware hands work-groups to CUs in order, so
// this is longest-processing-time-first list scheduling).  An item carries all a work-group needs to start streaming, so
// that its first K/V load is two dependent reads away (item, then page table; the live length is read beside it and
// only clips the end).  A request is cut into equal parts of whole 32-key tiles.  Fills the requests' piece fields
// beside the items.
static void build_work(sv_ctx* c, const Pass& ps, int32_t* req, int32_t* work) {
    const sv_model& m = c->model;
    const Layout& L = c->lay;
    const int G = m.n_q_heads / m.n_kv_heads;
    const bool prefill = ps.n == 0;
    int chunk = 0, cut = 1;
    if (prefill) {
        // 64-row groups make the parallelism; where they are too few for two work-groups per CU the keys are cut as well
        long long groups = 0;
        for (int b = 0; b < ps.B; ++b) groups += (G * ps.rq[b].n + kItemRows - 1) / kItemRows;
        cut = (int)std::max(1LL, kPrefillPlaces / (groups * m.n_kv_heads));
    } else {
        chunk = pick_chunk(c, ps);
    }
    struct Item { int len, v[kItemInts]; bool last; };
    std::vector<Item> items;
    long long prow = 0;
    c->pass_merge = false;
    int t0 = 0;
    for (int b = 0; b < ps.B; ++b) {
        const PassReq& r = ps.rq[b];
        const int start = c->seqs[r.seq].len_ub, total = start + r.n;
        const int rows_pad = (G * r.n + 15) / 16 * 16, groups = prefill ? (G * r.n + kItemRows - 1) / kItemRows : 1;
        int nch = prefill ? std::min(cut, pieces_of(c, total, kChunkKeys)) : pieces_of(c, total, chunk);
        if (prow + (long long)nch * m.n_kv_heads * rows_pad > L.part_rows || (long long)items.size() + (long long)nch * groups + (ps.B - b) > L.max_items)
            nch = 1;                                       // no room for partials: one piece, written directly
        const int clen = ((total + nch - 1) / nch + 31) / 32 * 32;
        int32_t* q = req + b * kReqInts;
        q[2] = clen; q[3] = nch; q[4] = (int32_t)prow; q[5] = nch * rows_pad; q[6] = rows_pad;
        for (int g = 0; g < groups; ++g) {
            const int last_key = prefill ? start + (std::min((g + 1) * kItemRows, G * r.n) - 1) / G + 1 : total;
            for (int ch = 0; ch < nch && ch * clen < total; ++ch) {
                const int kbeg = ch * clen, kend = std::min(kbeg + clen, total);
                items.push_back({std::min(kend, last_key) - kbeg,
                                 {r.seq, kbeg, kend, r.n, t0, g * kItemRows, nch > 1 ? (int32_t)(prow + ch * rows_pad) : -1, nch * rows_pad},
                                 b < ps.last && (g + 1) * kItemRows > G * (r.n - 1)});
            }
        }
        if (nch > 1) { prow += (long long)nch * m.n_kv_heads * rows_pad; c->pass_merge = true; }
        t0 += r.n;
    }
    std::stable_sort(items.begin(), items.end(), [](const Item& x, const Item& y) { return x.len > y.len; });
    for (size_t i = 0; i < items.size(); ++i) memcpy(work + i * kItemInts, items[i].v, sizeof(items[i].v));
    c->n_work = (int)items.size();
    c->n_last_work = 0;
    for (const Item& it : items) c->n_last_work += it.last;
    if (prefill && m.n_experts == 0) {                    // (models with experts keep their waves: see pick_chunk)
        std::vector<int> keys, last_keys;
        for (const Item& it : items) {
            keys.push_back(it.len);
            if (it.last) last_keys.push_back(it.len);
        }
        c->four_waves = prefill_four_waves(keys.data(), c->n_work, m.n_kv_heads);
        c->last_four_waves = prefill_four_waves(last_keys.data(), c->n_last_work, m.n_kv_heads);
    }
    if (c->n_work + c->n_last_work > L.max_items) { c->n_last_work = -1; return; }
    int at = c->n_work;
    for (const Item& it : items)
        if (it.last) memcpy(work + at++ * kItemInts, it.v, sizeof(it.v));
}

// Does the pass read more than the memory-side cache holds?  (All weights, experts as many as its rows can choose, all cached keys and values.
// A captured step keeps what held when it was captured: the results are the same bits either way.)
static bool reads_past_cache(const sv_ctx* c, const Pass& ps) {
    const sv_model& m = c->model;
    const size_t token = (size_t)2 * m.n_kv_heads * m.head_dim * (m.dtype == SV_BF16 ? 2 : 4) * m.n_layers;
    size_t bytes = c->weight_bytes + c->expert_bytes * std::min<long long>(m.n_experts, (long long)ps.T * m.top_k);
    for (int b = 0; b < ps.B; ++b) bytes += token * (c->seqs[ps.rq[b].seq].len_ub + ps.rq[b].n);
    return bytes > kCacheBytes;
}

// Make sure every request's sequence holds pages for its new rows; describe the pass (requests, attention work list,
// new page-table entries) to the device in one copy.  Nothing changes if the pool cannot cover the whole batch.
static int stage_pass(sv_ctx* c, const Pass& ps) {
    const Layout& L = c->lay;
    int need_total = 0;
    for (int b = 0; b < ps.B; ++b) {
        const int id = ps.rq[b].seq;
        if (id < 0 || id >= c->rt.max_seqs || !c->seqs[id].live) return c->fail(SV_ENOSEQ, "sequence id %d not live", id);
        for (int b2 = 0; b2 < b; ++b2)
            if (ps.rq[b2].seq == id) return c->fail(SV_ENOSEQ, "sequence id %d appears twice in the batch", id);
        const int need = pages_for(c, c->seqs[id].len_ub + ps.rq[b].n);
        if (need > c->rt.max_pages_per_seq) return c->fail(SV_ENOPAGES, "sequence %d would exceed max_pages_per_seq", id);
        need_total += std::max(0, need - (int)c->seqs[id].pages.size());
    }
    if (need_total > (int)c->free_pages.size())
        return c->fail(SV_ENOPAGES, "need %d more pages, %zu free", need_total, c->free_pages.size());
    if (need_total > L.max_upd) return c->fail(SV_EINVAL, "more than %d new pages in one pass", L.max_upd);

    int slot;
    SV_TRY(take_slot(c, slot));
    int32_t* st = c->staging[slot];
    int t0 = 0;
    for (int b = 0; b < ps.B; ++b) {
        const PassReq& r = ps.rq[b];
        st[L.st_seq + b] = r.seq;
        int32_t* q = st + L.st_req + b * kReqInts;
        const int32_t v[kReqInts] = {t0, r.n, 1, 1, 0, 0, 0, r.seq, r.pb, r.col0, 0, 0};
        memcpy(q, v, sizeof(v));
        t0 += r.n;
    }
    c->n_work = c->n_last_work = 0;
    c->four_waves = c->last_four_waves = false;
    c->pass_merge = false;
    c->cold = reads_past_cache(c, ps);
    if (attn_mfma_ok(c->model.dtype, c->model.head_dim, c->rt.page_size, c->attn_generic,
                     ps.n == 0 ? 0 : c->model.n_q_heads / c->model.n_kv_heads * ps.n))
        build_work(c, ps, st + L.st_req, st + L.st_work);
    st[0] = c->n_work;                                    // read by launches that were captured into a graph
    int nupd = 0;
    const int upd_at = L.st_work + kItemInts * (c->n_work + std::max(0, c->n_last_work));
    int32_t* upd = st + upd_at;
    for (int b = 0; b < ps.B; ++b) {
        SeqState& s = c->seqs[ps.rq[b].seq];
        const int need = pages_for(c, s.len_ub + ps.rq[b].n);
        while ((int)s.pages.size() < need) {
            const int32_t p = c->free_pages.back();
            c->free_pages.pop_back();
            upd[3 * nupd] = ps.rq[b].seq; upd[3 * nupd + 1] = (int32_t)s.pages.size(); upd[3 * nupd + 2] = p;
            s.pages.push_back(p);
            ++nupd;
        }
    }
    int32_t* dev = c->at<int32_t>(L.stage);
    SV_HIP(c, hipMemcpyAsync(dev, st, sizeof(int32_t) * (size_t)(upd_at + 3 * nupd), hipMemcpyHostToDevice, c->stream));
    if (nupd) {
        hipLaunchKernelGGL(apply_page_updates_kernel, dim3((nupd + 63) / 64), dim3(64), 0, c->stream,
                           c->at<int32_t>(L.page_table), c->rt.max_pages_per_seq, dev + upd_at, nupd);
        SV_HIP(c, hipGetLastError());
    }
    return release_slot(c, slot);
}

// The requests of a step or of a single-operation call: n rows each.
static int stage_batch(sv_ctx* c, const int32_t* ids, int B, int n, int k, std::vector<PassReq>& rq, Pass& ps) {
    rq.resize(B);
    for (int b = 0; b < B; ++b) rq[b] = {ids[b], n, 0, 0};
    ps = {rq.data(), B, n, n, B * n, k, -1};
    return stage_pass(c, ps);
}

// Work-group tile of the row-major projection kernel for M rows: 64, 128 or 256 tokens x 128 features.
static int pick_variant(const sv_ctx* c, int M) {
    if (c->gemm_variant >= 0) return c->gemm_variant;
    return M <= 64 ? 1 : M >= 512 ? 2 : 0;
}

// The plan of a packed projection, made once per shape (some microseconds of host arithmetic).
static WsPlan planned(sv_ctx* c, int M, int N, int K, bool allow_split, bool direct) {
    for (const auto& p : c->plans)
        if (p.M == M && p.N == N && p.K == K && p.allow_split == allow_split && p.direct == direct) return p.plan;
    const bool experts = c->model.n_experts > 0;
    WsPlan p = plan_packed(M, N, K, allow_split, c->gemm_tile, experts, direct);
    while (p.splits > 1 && (size_t)p.splits * M * N > c->lay.part_floats) p = plan_packed(M, N, K, allow_split, c->gemm_tile, experts, direct, p.splits - 1);
    if (c->plans.size() >= kPlans) c->plans.clear();
    c->plans.push_back({M, N, K, allow_split, direct, p});
    return p;
}

// The launch of the gate/up projection of T rows, made once per row count as well.
static GateUp gate_up_launch(sv_ctx* c, int T, bool direct) {
    for (const auto& g : c->gate_up)
        if (g.T == T && g.direct == direct) return g.launch;
    const GateUp g = plan_gate_up(T, 2 * c->model.d_ff, c->model.d_model, c->gemm_tile, direct);
    if (c->gate_up.size() >= kPlans) c->gate_up.clear();
    c->gate_up.push_back({T, direct, g});
    return g;
}

static int gemm(sv_ctx* c, const void* A, const void* W, float* out, int M, int N, int K, int* splits_out, bool allow_split = true) {
    ProfScope prof(c, SV_PROF_GEMM);
    if (c->model.dtype == SV_BF16) {
        if (c->packed) {
            const WsPlan p = planned(c, M, N, K, allow_split, direct_loads(W));
            *splits_out = p.splits;
            if (p.strip.tiles > 0) SV_HIP(c, gemm_bf16_strip((const bf16_t*)A, (const bf16_t*)W, out, M, N, K, p.splits, false, p.strip, c->cold, c->stream));
            else if (p.tall.n > 0) SV_HIP(c, gemm_bf16_tall((const bf16_t*)A, (const bf16_t*)W, out, M, N, K, p.splits, false, p.tall, c->stream));
            else SV_HIP(c, gemm_bf16_ws((const bf16_t*)A, (const bf16_t*)W, out, M, N, K, p.splits, p.wide, c->cold, c->stream, p.row_tiles));
        } else {
            const int s = allow_split ? pick_splits(M, N, K) : 1;
            *splits_out = s;
            SV_HIP(c, gemm_bf16((const bf16_t*)A, (const bf16_t*)W, out, M, N, K, s, pick_variant(c, M), c->stream));
        }
    } else {
        *splits_out = 1;
        SV_HIP(c, gemm_f32((const float*)A, (const float*)W, out, M, N, K, false, F32Norm{}, c->stream));
    }
    return SV_OK;
}

// What prep_rows reads of a prefill's prompts (null: a step's last_tokens and drafts).
struct Prompts { const int32_t* tokens; int ld; };

// Row preparation of a pass: cache slots, rotary table, where the attention partials lie; with_embed: also the rows'
// embeddings as the residual stream.
static int prepare_rows(sv_ctx* c, const Pass& ps, const int32_t* last_tokens, const int32_t* drafts, const Prompts* pr, bool with_embed) {
    const sv_model& m = c->model;
    const Layout& L = c->lay;
    RowPrep rp;
    rp.req = c->at<int32_t>(L.stage) + L.st_req; rp.seq_len = c->at<int32_t>(L.seq_len);
    rp.page_table = c->at<int32_t>(L.page_table); rp.max_pages_per_seq = c->rt.max_pages_per_seq; rp.page_size = c->rt.page_size;
    rp.last_tokens = last_tokens; rp.drafts = drafts; rp.tok_matrix = pr ? pr->tokens : nullptr; rp.tok_ld = pr ? pr->ld : 0;
    rp.embed = with_embed ? c->embed : nullptr; rp.dtype = m.dtype; rp.h = c->at<float>(L.h); rp.d = m.d_model;
    rp.row_slot = c->at<int32_t>(L.row_slot); rp.row_info = c->at<int32_t>(L.row_info); rp.row_part = c->at<int32_t>(L.row_part);
    rp.rope = c->at<float>(L.rope);
    rp.T = ps.T; rp.B = ps.B; rp.n = ps.n; rp.k = ps.k; rp.head_dim = m.head_dim; rp.vocab = m.vocab;
    rp.group = m.n_q_heads / m.n_kv_heads; rp.rope_theta = m.rope_theta;
    SV_HIP(c, prep_rows(rp, c->stream));
    return SV_OK;
}

// Residual add of what the previous projection left behind, then RMSNorm into the packed operand buffer.
// pending > 0: that many split-K planes in `part`; 0: nothing to add; -1: the expert outputs of a
// mixture-of-experts layer, still to be combined with the routing weights and added.
// last: see LastRows; a_out: where the rows go instead of the operand buffer.
static int add_norm(sv_ctx* c, int T, int pending, const void* gain, const LastRows& last = LastRows{}, void* a_out = nullptr) {
    const sv_model& m = c->model;
    const Layout& L = c->lay;
    float* h = c->at<float>(L.h);
    void* a_norm = a_out ? a_out : c->at<void>(L.a_norm);
    if (pending < 0)
        SV_HIP(c, add_rmsnorm_experts(h, c->at<float>(L.moe_y), c->at<int32_t>(L.moe_inv), c->at<float>(L.moe_w), m.top_k, gain, a_norm,
                                      T, m.d_model, m.rms_eps, c->packed, c->stream, last));
    else
        SV_HIP(c, add_rmsnorm(h, c->at<float>(L.part), pending, gain, a_norm, m.dtype, T, m.d_model, m.rms_eps, c->packed, c->stream, last));
    return SV_OK;
}

static AttnArgs attn_args(const sv_ctx* c, const Pass& ps, int layer, const void* q, void* out, bool out_packed) {
    const sv_model& m = c->model;
    const Layout& L = c->lay;
    AttnArgs aa;
    aa.q = q; aa.pool = c->rt.kv_pool; aa.geom = c->geom; aa.layer = layer;
    aa.page_table = c->at<int32_t>(L.page_table); aa.max_pages_per_seq = c->rt.max_pages_per_seq;
    aa.seq_len = c->at<int32_t>(L.seq_len); aa.row_info = c->at<int32_t>(L.row_info); aa.row_part = c->at<int32_t>(L.row_part);
    aa.out = out; aa.part_o = c->at<float>(L.part_o); aa.part_ml = c->at<float>(L.part_ml); aa.row_groups = 1;
    aa.T = ps.T; aa.n_max = ps.n_max; aa.k = ps.k; aa.Hq = m.n_q_heads; aa.Hkv = m.n_kv_heads; aa.hd = m.head_dim; aa.dtype = m.dtype;
    aa.work = c->at<int32_t>(L.stage) + L.st_work; aa.n_work = c->n_work;
    aa.last_of = nullptr; aa.n_last = 0; aa.last_out = nullptr;
    aa.row_items = ps.n == 0; aa.merge = c->pass_merge; aa.four_waves = c->four_waves; aa.cold = c->cold;
    aa.n_work_dev = nullptr; aa.grid_items = 0;
    if (c->graph_launch_shape) {      // nothing in the launch may depend on the lengths
        aa.n_work_dev = c->at<int32_t>(L.stage);
        aa.grid_items = ps.B * (fine_pieces_ok(c, ps.B) ? std::max(L.max_chunks, kFinePieces) : L.max_chunks);
        aa.merge = true;
    }
    aa.out_packed = out_packed;
    aa.force_generic = c->attn_generic; aa.min_row_tiles = c->attn_min_rt; aa.max_row_tiles = c->attn_max_rt;
    return aa;
}

// Does the last layer of this prefill pass go on with the prompts' last rows only, once K and V of all rows are in the cache?  Their
// attention outputs are gathered in the place of q, in whole 32-row tiles.
static bool last_rows_only(const sv_ctx* c, const Pass& ps) {
    const int tiles = (ps.last + 31) / 32 * 32;
    return ps.last > 0 && c->n_last_work >= 0 && tiles <= c->lay.P && 2 * tiles <= ps.T;
}

// Does a layer send this projection of M rows to the launch that takes norm, rotary, append or residual along?  (norm: rows that it normalises itself)
static bool takes_few_rows(int M, int N, int K, FewForm form, bool norm, int tile_mode, bool experts, bool aligned) {
    return !experts && tile_mode < 0 && aligned && few_rows_ok(M, N, K, form, norm);
}

// One decoder layer over the prepared rows.  On entry the residual stream h lacks `pending` (see add_norm) of
// the previous layer; on exit it lacks this layer's feed-forward output, described by the new `pending`.
static int layer_rows(sv_ctx* c, int l, const Pass& ps, int& pending) {
    const sv_model& m = c->model;
    const Layout& L = c->lay;
    int T = ps.T;
    const int d = m.d_model, qw = m.n_q_heads * m.head_dim, qkvw = (m.n_q_heads + 2 * m.n_kv_heads) * m.head_dim;
    hipStream_t st = c->stream;
    float* h = c->at<float>(L.h);
    float* part = c->at<float>(L.part);
    void* a_norm = c->at<void>(L.a_norm);
    // fp32: the projections write the residual themselves, and where their rows are few they take the norms and rotary with them
    const bool end = l == m.n_layers - 1 && ps.last >= 0, few = end && last_rows_only(c, ps);
    const bool f32 = m.dtype == SV_FP32;
    const bool f32_qkv = f32 && gemm_f32_fuses(T, qkvw, d, kF32Qkv);
    const bool f32_up = f32 && !few && gemm_f32_fuses(T, m.d_ff, d, kF32Glu);
    auto norm_by = [&](const void* gain) { return F32Norm{(const float*)gain, m.rms_eps}; };
    // a few rows of a packed dense model: likewise
    auto lean_ok = [&](const void* W, int N, int K, FewForm form, bool norm) {
        return c->packed && takes_few_rows(T, N, K, form, norm, c->gemm_tile, m.n_experts > 0, direct_loads(W));
    };
    auto few_norm = [&](const void* gain) { return FewNorm{(const bf16_t*)gain, m.rms_eps}; };

    RopeAppend ra;
    ra.qkv_part = part; ra.S = 1; ra.rope = c->at<float>(L.rope); ra.row_slot = c->at<int32_t>(L.row_slot);
    ra.q_out = c->at<void>(L.q); ra.pool = c->rt.kv_pool; ra.geom = c->geom; ra.layer = l;
    ra.T = T; ra.Hq = m.n_q_heads; ra.Hkv = m.n_kv_heads; ra.hd = m.head_dim; ra.dtype = m.dtype;
    if (f32_qkv) {
        ProfScope prof(c, SV_PROF_GEMM);
        SV_HIP(c, gemm_f32_qkv(h, (const float*)c->wqkv[l], d, norm_by(c->ln1[l]), ra, st));
    } else if (lean_ok(c->wqkv[l], qkvw, d, kFewQkv, false)) {
        const bool fused = pending == 0 && few_rows_ok(T, qkvw, d, kFewQkv, true);
        if (!fused) SV_TRY(add_norm(c, T, pending, c->ln1[l]));
        ProfScope prof(c, SV_PROF_GEMM);
        SV_HIP(c, few_rows_qkv(fused ? (const void*)h : a_norm, (const bf16_t*)c->wqkv[l], d, fused ? few_norm(c->ln1[l]) : FewNorm{}, ra, c->cold, st));
    } else {
        SV_TRY(add_norm(c, T, pending, c->ln1[l]));
        SV_TRY(gemm(c, a_norm, c->wqkv[l], part, T, qkvw, d, &ra.S));
        SV_HIP(c, rope_append(ra, st));
    }
    pending = 0;

    if (end && ps.last == 0) return SV_OK;                 // nobody asks for more than the cache entries
    AttnArgs aa = attn_args(c, ps, l, ra.q_out, c->at<void>(L.attn), c->packed);
    LastRows last{};
    if (few) {
        aa.last_of = c->at<int32_t>(L.stage) + L.st_req; aa.n_last = ps.last; aa.last_out = c->at<void>(L.q);
        aa.work += (size_t)kItemInts * c->n_work; aa.n_work = c->n_last_work; aa.four_waves = c->last_four_waves;
        if (!attn_mfma_ok(m.dtype, m.head_dim, c->rt.page_size, c->attn_generic, 0)) aa.last_out = c->at<void>(L.attn);   // (reads q, writes nothing but these rows)
        last = LastRows{aa.last_of, ps.last, true, 0};
    }
    {
        ProfScope prof(c, SV_PROF_ATTENTION);
        SV_HIP(c, attention(aa, st));
    }
    if (few) {                                             // from here on the rows are the last ones
        T = ps.last;
        aa.out = aa.last_out;
    }

    int s_o = 0;
    if (f32 && !few) {
        ProfScope prof(c, SV_PROF_GEMM);
        SV_HIP(c, gemm_f32((const float*)aa.out, (const float*)c->wo[l], h, T, d, qw, true, F32Norm{}, st));
    } else if (!few && lean_ok(c->wo[l], d, qw, kFewAdd, false)) {
        ProfScope prof(c, SV_PROF_GEMM);
        SV_HIP(c, few_rows_add((const bf16_t*)aa.out, (const bf16_t*)c->wo[l], h, T, d, qw, c->cold, st));
    } else {
        SV_TRY(gemm(c, aa.out, c->wo[l], part, T, d, qw, &s_o));
    }
    const bool lean_up = !few && s_o == 0 && lean_ok(c->wgu[l], 2 * m.d_ff, d, kFewGlu, true);
    if (!f32_up && !lean_up) SV_HIP(c, add_rmsnorm(h, part, s_o, c->ln2[l], a_norm, m.dtype, T, d, m.rms_eps, c->packed, st, last));
    if (m.n_experts > 0) {
        MoeArgs ma;
        ma.a = (const bf16_t*)a_norm; ma.w_router = (const bf16_t*)c->wrouter[l];
        ma.w_gate_up = (const bf16_t*)c->wgu[l]; ma.w_down = (const bf16_t*)c->wdown[l];
        ma.top_ids = c->at<int32_t>(L.moe_ids); ma.top_w = c->at<float>(L.moe_w); ma.router_logits = c->at<float>(L.moe_logits);
        ma.router_parts = (int)std::min<long long>(16, router_rows(L.P) / T);
        ma.live = c->at<int32_t>(L.moe_live); ma.tile_off = c->at<int32_t>(L.moe_off);
        ma.perm = c->at<int32_t>(L.moe_perm); ma.inv = c->at<int32_t>(L.moe_inv);
        ma.act = c->at<bf16_t>(L.moe_act); ma.y = c->at<float>(L.moe_y); ma.out = nullptr;   // combined by the next norm
        ma.T = T; ma.d = d; ma.E = m.n_experts; ma.top_k = m.top_k; ma.F = m.d_expert; ma.cold = c->cold;
        ProfScope prof(c, SV_PROF_MOE);
        SV_HIP(c, moe_ffn(ma, st));
        pending = -1;
        return SV_OK;
    }
    if (lean_up) {
        ProfScope prof(c, SV_PROF_GEMM);
        SV_HIP(c, few_rows_glu(h, (const bf16_t*)c->wgu[l], c->at<bf16_t>(L.act), T, m.d_ff, d, few_norm(c->ln2[l]), c->cold, st));
    } else if (c->packed && m.d_ff % 64 == 0) {
        // gate/up projection with SwiGLU in its epilogue: the [T, 2F] fp32 intermediate never exists
        ProfScope prof(c, SV_PROF_GEMM);
        const GateUp g = m.d_ff % 128 == 0 ? gate_up_launch(c, T, direct_loads(c->wgu[l])) : GateUp{};
        const bf16_t *ga = (const bf16_t*)a_norm, *gw = (const bf16_t*)c->wgu[l];
        if (g.strip.tiles > 0) SV_HIP(c, gemm_bf16_strip(ga, gw, c->at<float>(L.act), T, 2 * m.d_ff, d, 1, true, g.strip, c->cold, st));
        else if (g.tall.n > 0) SV_HIP(c, gemm_bf16_tall(ga, gw, c->at<float>(L.act), T, 2 * m.d_ff, d, 1, true, g.tall, st));
        else SV_HIP(c, gemm_bf16_ws_glu(ga, gw, c->at<bf16_t>(L.act), T, m.d_ff, d, st));
    } else if (f32) {
        ProfScope prof(c, SV_PROF_GEMM);
        SV_HIP(c, gemm_f32_glu(f32_up ? h : (const float*)a_norm, (const float*)c->wgu[l], c->at<float>(L.act), T, m.d_ff, d,
                               f32_up ? norm_by(c->ln2[l]) : F32Norm{}, st));
        if (!few) {
            SV_HIP(c, gemm_f32(c->at<float>(L.act), (const float*)c->wdown[l], h, T, d, m.d_ff, true, F32Norm{}, st));
            return SV_OK;
        }
    } else {
        int s_gu = 1;
        SV_TRY(gemm(c, a_norm, c->wgu[l], part, T, 2 * m.d_ff, d, &s_gu));
        SV_HIP(c, swiglu(part, s_gu, c->at<void>(L.act), T, m.d_ff, c->packed, st));
    }
    if (!few && lean_ok(c->wdown[l], d, m.d_ff, kFewAdd, false)) {
        ProfScope prof(c, SV_PROF_GEMM);
        SV_HIP(c, few_rows_add(c->at<bf16_t>(L.act), (const bf16_t*)c->wdown[l], h, T, d, m.d_ff, c->cold, st));
        return SV_OK;
    }
    SV_TRY(gemm(c, c->at<void>(L.act), c->wdown[l], part, T, d, m.d_ff, &pending));
    return SV_OK;
}

// The staged pass through all layers: rows prepared, residual stream complete but for the returned `pending`.
static int forward_layers(sv_ctx* c, const Pass& ps, const int32_t* last_tokens, const int32_t* drafts, const Prompts* pr, int& pending) {
    SV_TRY(prepare_rows(c, ps, last_tokens, drafts, pr, true));
    pending = 0;
    for (int l = 0; l < c->model.n_layers; ++l) SV_TRY(layer_rows(c, l, ps, pending));
    return SV_OK;
}

// Logits of M normalised rows.
static int head_rows(sv_ctx* c, const void* rows, int M, float* logits) {
    int one = 1;
    return gemm(c, rows, c->lm_head, logits, M, c->model.vocab, c->model.d_model, &one, false);
}

extern "C" int verify_prefill(sv_ctx* c, int32_t id, const int32_t* tokens, int32_t n, float* last_logits) {
    if (!c || !tokens) return SV_EINVAL;
    if (n <= 0) return c->fail(SV_EINVAL, "prefill of %d tokens", n);
    // a batch of one prompt
    return verify_prefill_batch(c, &id, 1, tokens, n, &n, last_logits);
}

// Prompts of several sequences at once, packed: a pass takes the next rows in prompt order, however many of each prompt
// fit, through the same kernels as a verification step (requests of different sizes, one causal chain each).  The passes
// are as few as hold all tokens, and of equal size.  Only the rows that end a prompt are wanted beyond their K and V: within a pass they
// belong to its first requests.  The last layer's attention, O and feed-forward take these rows only (7 layers of the 7B shape with the first
// step, 24 prompts of 100-500 tokens 21.6 -> 19.2 ms, one of 777 4.25 -> 4.00; their launch plans are those of few rows, so the sums are added up in
// another order), and where there is room their normalised rows are kept until all passes are done and the LM head's weights stream
// once, straight into the caller's logits.
extern "C" int verify_prefill_batch(sv_ctx* c, const int32_t* seq_ids, int32_t B, const int32_t* tokens, int32_t ld,
                                    const int32_t* n, float* last_logits) {
    if (!c || !seq_ids || !tokens || !n) return SV_EINVAL;
    if (B <= 0 || B > c->rt.max_batch || ld <= 0) return c->fail(SV_EINVAL, "prefill of %d prompts (limit %d), row pitch %d", B, c->rt.max_batch, ld);
    long long left = 0;
    for (int b = 0; b < B; ++b) {
        if (n[b] <= 0 || n[b] > ld) return c->fail(SV_EINVAL, "prompt %d has %d tokens (row pitch %d)", b, n[b], ld);
        if (b && n[b] > n[b - 1]) return c->fail(SV_EINVAL, "prompts must come longest first (prompt %d: %d after %d)", b, n[b], n[b - 1]);
        const int id = seq_ids[b];
        if (id < 0 || id >= c->rt.max_seqs || !c->seqs[id].live) return c->fail(SV_ENOSEQ, "sequence id %d not live", id);
        for (int b2 = 0; b2 < b; ++b2)
            if (seq_ids[b2] == id) return c->fail(SV_ENOSEQ, "sequence id %d appears twice in the batch", id);
        if (pages_for(c, c->seqs[id].len_ub + n[b]) > c->rt.max_pages_per_seq)
            return c->fail(SV_ENOPAGES, "sequence %d would exceed max_pages_per_seq", id);
        left += n[b];
    }
    const Prompts pr{tokens, ld};
    const sv_model& m = c->model;
    const Layout& L = c->lay;
    // the prompts' normalised last rows, in the place of a step's logits
    const size_t kept_bytes = (size_t)(B + 31) / 32 * 32 * m.d_model * (m.dtype == SV_BF16 ? 2 : 4);
    void* kept = kept_bytes <= sizeof(float) * (size_t)L.T * m.vocab ? c->at<void>(L.logits) : nullptr;
    std::vector<PassReq> rq;
    long long passes = (left + c->pass_rows - 1) / c->pass_rows;
    for (int b = 0, col = 0; b < B; --passes) {
        const long long room = std::min<long long>(c->pass_rows, ((left + passes - 1) / passes + 31) / 32 * 32);
        rq.clear();
        const int first = b;
        int T = 0, n_max = 0, ended = 0;
        while (b < B && T < room) {
            const int take = (int)std::min<long long>(n[b] - col, room - T);
            rq.push_back({seq_ids[b], take, b, col});
            T += take;
            n_max = std::max(n_max, take);
            col += take;
            if (col == n[b]) { ++ended; ++b; col = 0; }
        }
        left -= T;
        const Pass ps{rq.data(), (int)rq.size(), 0, n_max, T, kCausalK, last_logits ? ended : 0};
        if (const int rc = stage_pass(c, ps); rc != SV_OK) {      // no pages are left: the prompts that are done keep their logits
            if (kept && last_logits && first > 0) {
                const std::string why = c->err;
                SV_TRY(head_rows(c, kept, first, last_logits));
                c->err = why;
            }
            return rc;
        }
        int pending = 0;
        SV_TRY(forward_layers(c, ps, nullptr, nullptr, &pr, pending));
        if (ps.last > 0) {
            SV_TRY(add_norm(c, T, pending, c->final_norm, LastRows{c->at<int32_t>(L.stage) + L.st_req, ended, last_rows_only(c, ps), kept ? first : 0}, kept));
            if (!kept) SV_TRY(head_rows(c, c->at<void>(L.a_norm), ended, last_logits + (size_t)first * m.vocab));
            else if (b == B) SV_TRY(head_rows(c, kept, B, last_logits));
        }
        SV_HIP(c, add_rows(c->at<int32_t>(c->lay.seq_len), c->at<int32_t>(c->lay.stage) + c->lay.st_req, ps.B, c->stream));
        for (const PassReq& r : rq) c->seqs[r.seq].len_ub += r.n;
    }
    return SV_OK;
}

// Everything verify_step enqueues after the batch is staged: forward pass, accept/reject + draw, chain choice,
// rollback.
static int step_device_work(sv_ctx* c, const sv_batch* bt, const Pass& ps, const int32_t* drafts, const float* draft_probs,
                            const float* uniforms, const sv_out* out) {
    const int B = bt->B, k = bt->k, N = bt->N;
    int pending = 0;
    SV_TRY(forward_layers(c, ps, bt->last_tokens, drafts, nullptr, pending));
    const Layout& L = c->lay;
    const sv_model& m = c->model;
    float* logits = out->logits ? out->logits : c->at<float>(L.logits);   // a caller that wants them has them written in place
    if (m.dtype == SV_FP32 && gemm_f32_fuses(ps.T, m.vocab, m.d_model, kF32Plain)) {
        ProfScope prof(c, SV_PROF_GEMM);
        SV_HIP(c, gemm_f32(c->at<float>(L.h), (const float*)c->lm_head, logits, ps.T, m.vocab, m.d_model, false,
                           F32Norm{(const float*)c->final_norm, m.rms_eps}, c->stream));
    } else {
        SV_TRY(add_norm(c, ps.T, pending, c->final_norm));
        SV_TRY(head_rows(c, c->at<void>(L.a_norm), ps.T, logits));
    }

    SampleArgs sa;
    sa.logits = logits; sa.drafts = drafts; sa.draft_probs = draft_probs; sa.uniforms = uniforms;
    sa.draft_lens = bt->draft_lens; sa.stat_part = c->at<float>(L.stat_part); sa.draw_part = c->at<float>(L.draw_part);
    sa.seq_len = c->at<int32_t>(L.seq_len); sa.batch_seq = c->at<int32_t>(L.stage) + L.st_seq;
    sa.accepted_len = out->accepted_len; sa.out_tokens = out->out_tokens; sa.best_chain = out->best_chain;
    sa.B = B; sa.N = N; sa.k = k; sa.V = c->model.vocab; sa.verify_mode = c->rt.verify_mode; sa.sample_mode = c->rt.sample_mode;
    sa.temperature = c->rt.temperature;
    {
        ProfScope prof(c, SV_PROF_SAMPLER);
        SV_HIP(c, sample_verify(sa, c->stream));
    }

    RollbackArgs rb;
    rb.pool = c->rt.kv_pool; rb.geom = c->geom; rb.n_layers = c->model.n_layers; rb.dtype = c->model.dtype;
    rb.page_table = c->at<int32_t>(L.page_table); rb.max_pages_per_seq = c->rt.max_pages_per_seq;
    rb.batch_seq = c->at<int32_t>(L.stage) + L.st_seq; rb.seq_len = c->at<int32_t>(L.seq_len);
    rb.accepted_len = out->accepted_len; rb.best_chain = out->best_chain; rb.B = B; rb.N = N; rb.k = k;
    {
        ProfScope prof(c, SV_PROF_ROLLBACK);
        SV_HIP(c, compact_kept(rb, true, c->stream));
    }
    return SV_OK;
}

static void drop_graphs(sv_ctx* c) {
    bool launched = false;
    for (auto& g : c->graphs) launched |= g.exec != nullptr;
    if (launched) (void)hipStreamSynchronize(c->stream);  // an executable graph may still be replaying on the stream
    for (auto& g : c->graphs)
        if (g.exec) (void)hipGraphExecDestroy(g.exec);
    c->graphs.clear();
}

// Graph replay of the step's device work.  A step's launches depend on the batch shape and on the caller's
// buffers only (the lengths reach the kernels through device memory; the attention grid is sized for the most
// work items the shape can have), so one captured graph serves every step with the same shape and buffers.
// The first step of a kind runs as plain launches (the runtime loads each kernel at its first launch, which a capture is
// no place for), the second is captured, later ones replay.  Returns 1 if the work was enqueued through a graph, 0 if the caller should
// enqueue it itself, < 0 on error.
static int step_through_graph(sv_ctx* c, const sv_batch* bt, const Pass& ps, const int32_t* drafts, const float* draft_probs,
                              const float* uniforms, const sv_out* out) {
    if (!c->use_graph || c->stream == nullptr || c->prof_mask != 0) return 0;
    const void* ptr[9] = {bt->last_tokens, drafts, draft_probs, uniforms, bt->draft_lens,
                          out->accepted_len, out->out_tokens, out->best_chain, out->logits};
    sv_ctx::GraphEntry* e = nullptr;
    for (auto& g : c->graphs)
        if (g.B == bt->B && g.k == bt->k && g.N == bt->N && memcmp(g.ptr, ptr, sizeof(ptr)) == 0) e = &g;
    if (!e) {
        if (c->graphs.size() >= 8) {                       // forget the least recently used
            size_t old = 0;
            for (size_t i = 1; i < c->graphs.size(); ++i)
                if (c->graphs[i].used < c->graphs[old].used) old = i;
            if (c->graphs[old].exec) {
                (void)hipStreamSynchronize(c->stream);     // it may still be replaying
                (void)hipGraphExecDestroy(c->graphs[old].exec);
            }
            c->graphs.erase(c->graphs.begin() + old);
        }
        sv_ctx::GraphEntry g;
        g.B = bt->B; g.k = bt->k; g.N = bt->N;
        memcpy(g.ptr, ptr, sizeof(ptr));
        g.exec = nullptr;
        g.used = ++c->graph_clock;
        c->graphs.push_back(g);
        return 0;                                           // first step of this kind: plain launches
    }
    e->used = ++c->graph_clock;
    if (!e->exec) {
        hipGraph_t graph = nullptr;
        SV_HIP(c, hipStreamBeginCapture(c->stream, hipStreamCaptureModeThreadLocal));
        c->graph_launch_shape = true;
        const int rc = step_device_work(c, bt, ps, drafts, draft_probs, uniforms, out);
        c->graph_launch_shape = false;
        const hipError_t ec = hipStreamEndCapture(c->stream, &graph);
        if (rc != SV_OK || ec != hipSuccess || !graph) {
            if (graph) (void)hipGraphDestroy(graph);
            return rc != SV_OK ? rc : c->fail(SV_EHIP, "stream capture failed: %s", hipGetErrorString(ec));
        }
        const hipError_t ei = hipGraphInstantiate(&e->exec, graph, nullptr, nullptr, 0);
        (void)hipGraphDestroy(graph);
        if (ei != hipSuccess) { e->exec = nullptr; return c->fail(SV_EHIP, "graph instantiation failed: %s", hipGetErrorString(ei)); }
    }
    SV_HIP(c, hipGraphLaunch(e->exec, c->stream));
    return 1;
}

extern "C" int verify_step(sv_ctx* c, const sv_batch* bt, const int32_t* drafts, const float* draft_probs,
                           const float* uniforms, const sv_out* out) {
    if (!c || !bt || !out) return SV_EINVAL;
    const int B = bt->B, k = bt->k, N = bt->N;
    if (B <= 0 || B > c->rt.max_batch || k < 0 || k > c->rt.max_k || N <= 0 || N > c->rt.max_chains)
        return c->fail(SV_EINVAL, "batch %d / k %d / chains %d outside the limits given at init", B, k, N);
    if (!bt->seq_ids || !bt->last_tokens || (k > 0 && !drafts) || !out->accepted_len || !out->out_tokens || !out->best_chain)
        return c->fail(SV_EINVAL, "null argument");
    if (c->rt.verify_mode != SV_GREEDY && !uniforms) return c->fail(SV_EINVAL, "stochastic and match verification need uniforms");
    const int n = 1 + N * k;
    std::vector<PassReq> rq;
    Pass ps;
    SV_TRY(stage_batch(c, bt->seq_ids, B, n, k, rq, ps));
    const int via_graph = step_through_graph(c, bt, ps, drafts, draft_probs, uniforms, out);
    if (via_graph < 0) return via_graph;
    if (via_graph == 0) SV_TRY(step_device_work(c, bt, ps, drafts, draft_probs, uniforms, out));
    for (int b = 0; b < B; ++b) c->seqs[bt->seq_ids[b]].len_ub += k + 1;
    return SV_OK;
}

// -------------------------------------------------- single-operation entry points ---

static bool op_cold(size_t weights) { return weights * sizeof(bf16_t) > kCacheBytes; }      // one projection again and again finds smaller weights in the cache

extern "C" int sv_op_gemm_bf16(const void* A, const void* W, float* out, int M, int N, int K, int splits, int variant,
                               void* stream) {
    if (!A || !W || !out || M <= 0 || !gemm_bf16_shape_ok(N, K, splits) || !gemm_bf16_variant_ok(variant, N)) return SV_EINVAL;
    return gemm_bf16((const bf16_t*)A, (const bf16_t*)W, out, M, N, K, splits, variant, (hipStream_t)stream) ==
                   hipSuccess ? SV_OK : SV_EHIP;
}

extern "C" int sv_op_gemm_bf16_ws(const void* Ap, const void* Wp, float* out, int M, int N, int K, int splits, int wide,
                                  int row_tiles, void* stream) {
    if (!Ap || !Wp || !out || M <= 0 || N <= 0 || K <= 0 || splits <= 0 || N % (wide ? 256 : 128) != 0 ||
        K % (64 * splits) != 0 || row_tiles < 0 || (row_tiles > 5 && row_tiles != 8) || (row_tiles == 8 && N % 256 != 0))
        return SV_EINVAL;
    const bool tall = row_tiles == 8 && direct_loads(Ap) && direct_loads(Wp), cold = op_cold((size_t)N * K);     // (the other kernel's sums are the same)
    const hipError_t e = tall ? gemm_bf16_tall((const bf16_t*)Ap, (const bf16_t*)Wp, out, M, N, K, splits, false, gemm_bf16_tall_256(M), (hipStream_t)stream)
                                        : gemm_bf16_ws((const bf16_t*)Ap, (const bf16_t*)Wp, out, M, N, K, splits, wide != 0, cold, (hipStream_t)stream, row_tiles == 8 ? 0 : row_tiles);
    return e == hipSuccess ? SV_OK : SV_EHIP;
}

extern "C" int sv_op_gemm_plan(int M, int N, int K, int* splits, int* wide, int* row_tiles) {
    if (!splits || !wide || !row_tiles || M <= 0 || N <= 0 || K <= 0 || N % 128 != 0 || K % 64 != 0) return SV_EINVAL;
    // of the weight-streaming kernel, but where the 256-row tiles fill the chip four times over
    WsPlan p = plan_ws(M, N, K, true);
    if (N % 256 == 0 && M >= 1024 && (long long)((M + 255) / 256) * (N / 256) >= 4 * 256) p = WsPlan{1, true, 8, 0.0, 0.0, {}, {}};
    *splits = p.splits; *wide = p.wide ? 1 : 0; *row_tiles = p.row_tiles;
    return SV_OK;
}

extern "C" int sv_op_prefill_waves(const int* keys, int items, int n_kv_heads, int* waves) {
    if (!keys || !waves || items <= 0 || n_kv_heads <= 0) return SV_EINVAL;
    std::vector<int> lens(keys, keys + items);
    std::sort(lens.begin(), lens.end(), std::greater<int>());
    if (lens.back() <= 0) return SV_EINVAL;
    *waves = prefill_four_waves(lens.data(), items, n_kv_heads) ? 4 : 2;
    return SV_OK;
}

constexpr int kFormQkv = 4;                               // a step's launch only: where QKV may take another kernel than O and down

static bool step_form_ok(int M, int N, int K, int form) {
    return M > 0 && N > 0 && K > 0 && form >= 0 && form <= 2 && N % (form == 2 ? 256 : 128) == 0 && K % 64 == 0;
}

extern "C" int sv_op_gemm_step_plan(int M, int N, int K, int form, int* splits, int* wide, int* row_tiles, int* tall) {
    if (!splits || !wide || !row_tiles || !tall || !step_form_ok(M, N, K, form)) return SV_EINVAL;
    WsPlan p{1, false, 0, 0.0, 0.0, {}, {}};
    if (form == 2) p.tall = M > 160 ? gemm_bf16_tall_plan(M, N, K, 1).tiles : TallTiles{};
    else p = plan_wide(M, N, K, form == 0, -1, true);
    *splits = p.splits; *wide = p.wide ? 1 : 0; *row_tiles = p.row_tiles;
    tall[0] = p.tall.rw; tall[1] = p.tall.n; tall[2] = p.tall.rwt; tall[3] = p.tall.nt;
    return SV_OK;
}

extern "C" int sv_op_gemm_step_launch(int M, int N, int K, int form, int tile_mode, int experts, int aligned, sv_gemm_launch* out) {
    const bool qkv = form == kFormQkv;
    if (qkv) form = 0;
    if (!out || !step_form_ok(M, N, K, form) || tile_mode < -1 || tile_mode > 1) return SV_EINVAL;
    if (form != 1 && takes_few_rows(M, N, K, form == 2 ? kFewGlu : qkv ? kFewQkv : kFewAdd, form == 2, tile_mode, experts != 0, aligned != 0)) {
        *out = sv_gemm_launch{SV_GEMM_FEW, 1, 0, 0, 0, {0, 0, 0, 0}};
        return SV_OK;
    }
    WsPlan p{1, false, 0, 0.0, 0.0, {}, {}};
    if (form == 2) {
        const GateUp g = plan_gate_up(M, N, K, tile_mode, aligned != 0);
        p.tall = g.tall;
        p.strip = g.strip;
    } else {
        p = plan_packed(M, N, K, form == 0, tile_mode, experts != 0, aligned != 0);
    }
    const bool strip = p.strip.tiles > 0, tall = !strip && p.tall.n > 0;
    *out = sv_gemm_launch{strip ? SV_GEMM_STRIP : tall ? SV_GEMM_TALL : SV_GEMM_WS, p.splits, !strip && !tall && p.wide ? 1 : 0,
                          strip ? p.strip.tiles : tall ? 0 : p.row_tiles, 32 * p.strip.fs, {p.tall.rw, p.tall.n, p.tall.rwt, p.tall.nt}};
    return SV_OK;
}

extern "C" int sv_op_gemm_bf16_tall(const void* Ap, const void* Wp, void* out, int M, int N, int K, int splits, int gated,
                                    const int* tall, void* stream) {
    if (!Ap || !Wp || !out || M <= 0 || N <= 0 || K <= 0 || splits <= 0 || splits > kMaxSplitsWs || (gated && splits != 1) ||
        N % (gated ? 256 : 128) != 0 || K % 64 != 0 || K % (32 * splits) != 0)
        return SV_EINVAL;
    hipStream_t st = (hipStream_t)stream;
    auto weight_streaming = [&]() -> int {
        const hipError_t e = gated ? gemm_bf16_ws_glu((const bf16_t*)Ap, (const bf16_t*)Wp, (bf16_t*)out, M, N / 2, K, st)
                                   : gemm_bf16_ws((const bf16_t*)Ap, (const bf16_t*)Wp, (float*)out, M, N, K, splits, N % 256 == 0, op_cold((size_t)N * K), st);
        return e == hipSuccess ? SV_OK : SV_EHIP;
    };
    if (!tall) return gated ? weight_streaming() : SV_EINVAL;
    const TallTiles tl{tall[0], tall[1], tall[2], tall[3]};
    // heights that exist; all rows covered, no tile of padding alone (which also bounds the grid)
    if (tl.rw < 3 || tl.rw > 5 || tl.rwt < 0 || tl.rwt >= tl.rw || (tl.nt > 0) != (tl.rwt > 0) || tl.n < 1 || tl.nt < 0 || tl.n > M || tl.nt > M)
        return SV_EINVAL;
    const long long rows = 64LL * tl.rw * tl.n + 64LL * tl.rwt * tl.nt;
    if (rows < M || rows - 64 * (tl.nt > 0 ? tl.rwt : tl.rw) >= M) return SV_EINVAL;
    if (!direct_loads(Ap) || !direct_loads(Wp)) return K % (64 * splits) == 0 ? weight_streaming() : SV_EINVAL;     // the same sums
    return gemm_bf16_tall((const bf16_t*)Ap, (const bf16_t*)Wp, (float*)out, M, N, K, splits, gated != 0, tl, st) == hipSuccess ? SV_OK : SV_EHIP;
}

extern "C" int sv_op_gemm_bf16_strip(const void* Ap, const void* Wp, void* out, int M, int N, int K, int splits, int gated, int row_tiles,
                                     int features, void* stream) {
    if (!Ap || !Wp || !out || M <= 0 || N <= 0 || K <= 0 || splits <= 0 || splits > kMaxSplitsWs || (gated && splits != 1) ||
        N % (gated ? 256 : 128) != 0 || K % 64 != 0 || K % (32 * splits) != 0 || row_tiles < 1 || row_tiles > 10 || row_tiles == 7 ||
        row_tiles == 9 || M > 32 * row_tiles || (features != 128 && features != 160 && features != 224) || !direct_loads(Ap) || !direct_loads(Wp))
        return SV_EINVAL;
    return gemm_bf16_strip((const bf16_t*)Ap, (const bf16_t*)Wp, (float*)out, M, N, K, splits, gated != 0, StripTile{row_tiles, features / 32},
                           op_cold((size_t)N * K), (hipStream_t)stream) == hipSuccess ? SV_OK : SV_EHIP;
}

extern "C" int sv_op_pack_rows(const void* src, void* dst, int M, int K, void* stream) {
    if (!src || !dst || src == dst || M <= 0 || K <= 0 || K % 16 != 0) return SV_EINVAL;
    return pack_rows((const bf16_t*)src, (bf16_t*)dst, M, K, (hipStream_t)stream) == hipSuccess ? SV_OK : SV_EHIP;
}

extern "C" int sv_op_pack_weight(const void* src, void* dst, int N, int K, void* stream) {
    if (!src || !dst || src == dst || N <= 0 || K <= 0 || N % 128 != 0 || K % 32 != 0) return SV_EINVAL;
    return pack_weight((const bf16_t*)src, (bf16_t*)dst, N, K, (hipStream_t)stream) == hipSuccess ? SV_OK : SV_EHIP;
}

extern "C" int sv_op_sample(const float* logits, const int32_t* drafts, const float* draft_probs, const float* uniforms,
                            const int32_t* draft_lens, int B, int N, int k, int V, int verify_mode, int sample_mode,
                            float temperature, void* scratch, int32_t* accepted_len, int32_t* out_tokens,
                            int32_t* best_chain, void* stream) {
    if (!logits || (k > 0 && !drafts) || !scratch || !accepted_len || !out_tokens || !best_chain || B <= 0 || N <= 0 ||
        k < 0 || V <= 0 || !(temperature > 0.f) || verify_mode < 0 || verify_mode > 2 || (verify_mode != SV_GREEDY && !uniforms))
        return SV_EINVAL;
    const int T = B * (1 + N * k);
    SampleArgs sa;
    sa.logits = logits; sa.drafts = drafts; sa.draft_probs = draft_probs; sa.uniforms = uniforms; sa.draft_lens = draft_lens;
    sa.stat_part = reinterpret_cast<float*>(scratch);
    sa.draw_part = sa.stat_part + 4 * sample_part_entries(T);
    sa.seq_len = nullptr; sa.batch_seq = nullptr;
    sa.accepted_len = accepted_len; sa.out_tokens = out_tokens; sa.best_chain = best_chain;
    sa.B = B; sa.N = N; sa.k = k; sa.V = V; sa.verify_mode = verify_mode; sa.sample_mode = sample_mode; sa.temperature = temperature;
    return sample_verify(sa, (hipStream_t)stream) == hipSuccess ? SV_OK : SV_EHIP;
}

extern "C" size_t sv_op_sample_scratch_bytes(int B, int N, int k) {
    if (B <= 0 || N <= 0 || k < 0) return 0;
    return 2 * sizeof(float) * 4 * sample_part_entries(B * (1 + N * k));
}

struct MoeScratch { size_t ids, w, live, off, perm, inv, act, y, logits, total; };
static MoeScratch moe_scratch(int T, int d, int E, int top_k, int F) {
    MoeScratch m;
    size_t o = 0;
    auto take = [&](size_t bytes) { size_t at = o; o += align_up(bytes); return at; };
    const size_t tiles = (size_t)moe_max_tiles(T, E, top_k);
    m.ids = take(sizeof(int32_t) * (size_t)T * top_k);
    m.w = take(sizeof(float) * (size_t)T * top_k);
    m.live = take(sizeof(int32_t) * (2 + 2 * (size_t)E));
    m.off = take(sizeof(int32_t) * (E + 1));
    m.perm = take(sizeof(int32_t) * 32 * tiles);
    m.inv = take(sizeof(int32_t) * (size_t)T * top_k);
    m.act = take(sizeof(bf16_t) * 32 * tiles * F);
    m.y = take(sizeof(float) * 32 * tiles * d);
    m.logits = take(sizeof(float) * 4 * (size_t)T * E);
    m.total = o;
    return m;
}

extern "C" size_t sv_op_moe_scratch_bytes(int T, int d, int E, int top_k, int F) {
    if (!moe_shape_ok(T, d, E, top_k, F)) return 0;
    return moe_scratch(T, d, E, top_k, F).total;
}

extern "C" int sv_op_moe_ffn(const void* a_packed, const void* w_router, const void* w_gate_up_packed,
                             const void* w_down_packed, int T, int d, int E, int top_k, int F, void* scratch,
                             size_t scratch_bytes, float* out, int32_t* top_ids, float* top_w, void* stream) {
    if (!a_packed || !w_router || !w_gate_up_packed || !w_down_packed || !scratch || !out) return SV_EINVAL;
    if (!moe_shape_ok(T, d, E, top_k, F)) return SV_EUNSUPPORTED;
    const MoeScratch m = moe_scratch(T, d, E, top_k, F);
    if (scratch_bytes < m.total || ((uintptr_t)scratch & 255)) return SV_EINVAL;
    char* ws = reinterpret_cast<char*>(scratch);
    MoeArgs ma;
    ma.a = (const bf16_t*)a_packed; ma.w_router = (const bf16_t*)w_router;
    ma.w_gate_up = (const bf16_t*)w_gate_up_packed; ma.w_down = (const bf16_t*)w_down_packed;
    ma.top_ids = reinterpret_cast<int32_t*>(ws + m.ids); ma.top_w = reinterpret_cast<float*>(ws + m.w);
    ma.router_logits = reinterpret_cast<float*>(ws + m.logits);
    ma.live = reinterpret_cast<int32_t*>(ws + m.live); ma.tile_off = reinterpret_cast<int32_t*>(ws + m.off);
    ma.perm = reinterpret_cast<int32_t*>(ws + m.perm); ma.inv = reinterpret_cast<int32_t*>(ws + m.inv);
    ma.act = reinterpret_cast<bf16_t*>(ws + m.act); ma.y = reinterpret_cast<float*>(ws + m.y); ma.out = out;
    ma.T = T; ma.d = d; ma.E = E; ma.top_k = top_k; ma.F = F;
    ma.cold = op_cold((size_t)3 * F * d * std::min<long long>(E, (long long)T * top_k));
    hipStream_t st = (hipStream_t)stream;
    if (moe_ffn(ma, st) != hipSuccess) return SV_EHIP;
    if (top_ids && hipMemcpyAsync(top_ids, ma.top_ids, sizeof(int32_t) * (size_t)T * top_k, hipMemcpyDeviceToDevice, st) != hipSuccess)
        return SV_EHIP;
    if (top_w && hipMemcpyAsync(top_w, ma.top_w, sizeof(float) * (size_t)T * top_k, hipMemcpyDeviceToDevice, st) != hipSuccess)
        return SV_EHIP;
    return SV_OK;
}

extern "C" int sv_op_attention(sv_ctx* c, const int32_t* seq_ids, int B, int n, int k, int layer, const void* q, void* out) {
    if (!c || !seq_ids || !q || !out) return SV_EINVAL;
    if (B <= 0 || B > c->rt.max_batch || n <= 0 || B * n > c->lay.T || k < 0 || layer < 0 || layer >= c->model.n_layers ||
        (k > 0 && (n - 1) % k != 0) || (k == 0 && n != 1))
        return c->fail(SV_EINVAL, "attention of %d x %d rows (k=%d, layer %d) outside the limits given at init", B, n, k, layer);
    std::vector<PassReq> rq;
    Pass ps;
    SV_TRY(stage_batch(c, seq_ids, B, n, k, rq, ps));
    SV_TRY(prepare_rows(c, ps, nullptr, nullptr, nullptr, false));
    SV_HIP(c, attention(attn_args(c, ps, layer, q, out, false), c->stream));
    return SV_OK;
}

extern "C" int sv_op_layer(sv_ctx* c, const int32_t* seq_ids, int B, int n, int k, int layer, const float* h_in,
                           float* h_out, int32_t* top_ids, float* top_w) {
    if (!c || !seq_ids || !h_in || !h_out) return SV_EINVAL;
    if (B <= 0 || B > c->rt.max_batch || n <= 0 || B * n > c->lay.T || k < 0 || layer < 0 || layer >= c->model.n_layers ||
        (k > 0 && (n - 1) % k != 0) || (k == 0 && n != 1))
        return c->fail(SV_EINVAL, "layer %d over %d x %d rows (k=%d) outside the limits given at init", layer, B, n, k);
    std::vector<PassReq> rq;
    Pass ps;
    SV_TRY(stage_batch(c, seq_ids, B, n, k, rq, ps));
    const sv_model& m = c->model;
    const Layout& L = c->lay;
    const int T = B * n;
    const size_t bytes = sizeof(float) * (size_t)T * m.d_model;
    SV_TRY(prepare_rows(c, ps, nullptr, nullptr, nullptr, false));
    SV_HIP(c, hipMemcpyAsync(c->at<float>(L.h), h_in, bytes, hipMemcpyDeviceToDevice, c->stream));
    int pending = 0;
    SV_TRY(layer_rows(c, layer, ps, pending));
    // the feed-forward output is still pending: the residual add that the next layer's (or the final) norm would do
    SV_TRY(add_norm(c, T, pending, c->final_norm));
    SV_HIP(c, hipMemcpyAsync(h_out, c->at<float>(L.h), bytes, hipMemcpyDeviceToDevice, c->stream));
    if (m.n_experts > 0) {
        if (top_ids) SV_HIP(c, hipMemcpyAsync(top_ids, c->at<int32_t>(L.moe_ids), sizeof(int32_t) * (size_t)T * m.top_k, hipMemcpyDeviceToDevice, c->stream));
        if (top_w) SV_HIP(c, hipMemcpyAsync(top_w, c->at<float>(L.moe_w), sizeof(float) * (size_t)T * m.top_k, hipMemcpyDeviceToDevice, c->stream));
    }
    return SV_OK;
}

extern "C" int sv_op_rollback(sv_ctx* c, const int32_t* seq_ids, int B, int N, int k, const int32_t* accepted_len,
                              const int32_t* best_chain, int commit) {
    if (!c || !seq_ids || !accepted_len || !best_chain) return SV_EINVAL;
    if (B <= 0 || B > c->rt.max_batch || k < 0 || k > c->rt.max_k || N <= 0 || N > c->rt.max_chains)
        return c->fail(SV_EINVAL, "batch %d / k %d / chains %d outside the limits given at init", B, k, N);
    std::vector<PassReq> rq;
    Pass ps;
    SV_TRY(stage_batch(c, seq_ids, B, 1 + N * k, k, rq, ps));   // the slots of a pass: L .. L + N*k
    RollbackArgs rb;
    rb.pool = c->rt.kv_pool; rb.geom = c->geom; rb.n_layers = c->model.n_layers; rb.dtype = c->model.dtype;
    rb.page_table = c->at<int32_t>(c->lay.page_table); rb.max_pages_per_seq = c->rt.max_pages_per_seq;
    rb.batch_seq = c->at<int32_t>(c->lay.stage) + c->lay.st_seq; rb.seq_len = c->at<int32_t>(c->lay.seq_len);
    rb.accepted_len = accepted_len; rb.best_chain = best_chain; rb.B = B; rb.N = N; rb.k = k;
    {
        ProfScope prof(c, SV_PROF_ROLLBACK);
        SV_HIP(c, compact_kept(rb, false, c->stream));
        if (commit) SV_HIP(c, commit_lens(rb, c->stream));
    }
    if (commit)
        for (int b = 0; b < B; ++b) c->seqs[seq_ids[b]].len_ub += k + 1;
    return SV_OK;
}

extern "C" int sv_profile_enable(sv_ctx* c, unsigned kind_mask) {
    if (!c) return SV_EINVAL;
    c->prof_mask = kind_mask & ((1u << SV_PROF_KINDS) - 1u);
    return SV_OK;
}

extern "C" int sv_profile_read(sv_ctx* c, int kind, double* total_ms, int* launches) {
    if (!c || !total_ms || !launches || kind < 0 || kind >= SV_PROF_KINDS) return SV_EINVAL;
    SV_HIP(c, hipStreamSynchronize(c->stream));
    double tot = 0.0;
    int n = 0;
    std::vector<sv_ctx::ProfRec> keep;
    for (auto& r : c->prof_recs) {
        if (r.kind != kind) { keep.push_back(r); continue; }
        float ms = 0.f;
        if (hipEventElapsedTime(&ms, r.a, r.b) == hipSuccess) { tot += ms; ++n; }
        c->prof_free.push_back(r.a);
        c->prof_free.push_back(r.b);
    }
    c->prof_recs.swap(keep);
    *total_ms = tot;
    *launches = n;
    return SV_OK;
}

extern "C" int sv_seq_set_lens(sv_ctx* c, const int32_t* seq_ids, const int32_t* lens, int n) {
    if (!c || !seq_ids || !lens || n <= 0 || n > c->rt.max_batch) return SV_EINVAL;
    for (int i = 0; i < n; ++i) {
        const int id = seq_ids[i];
        if (id < 0 || id >= c->rt.max_seqs || !c->seqs[id].live) return c->fail(SV_ENOSEQ, "sequence id %d not live", id);
        if (lens[i] < 0 || lens[i] > (int)c->seqs[id].pages.size() * c->rt.page_size)
            return c->fail(SV_EINVAL, "length %d beyond the pages sequence %d holds", lens[i], id);
    }
    for (int i0 = 0; i0 < n; i0 += kLenPairs) {
        const int m = std::min(kLenPairs, n - i0);
        LenPairs pairs;
        for (int i = 0; i < m; ++i) { pairs.v[2 * i] = seq_ids[i0 + i]; pairs.v[2 * i + 1] = lens[i0 + i]; }
        hipLaunchKernelGGL(set_lens_kernel, dim3(1), dim3(256), 0, c->stream, c->at<int32_t>(c->lay.seq_len), pairs, m);
        SV_HIP(c, hipGetLastError());
    }
    for (int i = 0; i < n; ++i) c->seqs[seq_ids[i]].len_ub = lens[i];
    return SV_OK;
}

extern "C" int sv_set_option(sv_ctx* c, int option, int value) {
    if (!c) return SV_EINVAL;
    drop_graphs(c);                                       // captured launches carry the options they were made with
    switch (option) {
        case SV_OPT_GEMM_VARIANT:
            if (value < -1 || value > 2)
                return c->fail(SV_EINVAL, "gemm variant %d", value);
            c->gemm_variant = value;
            return SV_OK;
        case SV_OPT_GEMM_TILE:
            if (value < -1 || value > 1) return c->fail(SV_EINVAL, "gemm tile mode %d", value);
            c->gemm_tile = value;
            c->plans.clear();
            c->gate_up.clear();
            return SV_OK;
        case SV_OPT_ATTN_GENERIC:
            c->attn_generic = value != 0;
            return SV_OK;
        case SV_OPT_ATTN_CHUNK_KEYS:
            if (value != 0 && (value < kChunkKeys || value % 128 != 0)) return c->fail(SV_EINVAL, "chunk of %d keys", value);
            c->attn_chunk_opt = value;
            return SV_OK;
        case SV_OPT_GRAPH:
            if (value != 0 && c->stream == nullptr) return c->fail(SV_EINVAL, "graph replay needs a stream of its own, not the null stream");
            c->use_graph = value != 0;
            drop_graphs(c);
            return SV_OK;
        case SV_OPT_ATTN_MAX_ROW_TILES:
            if (value < 1 || value > 4) return c->fail(SV_EINVAL, "row tiles %d", value);
            c->attn_max_rt = value;
            return SV_OK;
        case SV_OPT_ATTN_MIN_ROW_TILES:
            if (value < 1 || value > 4) return c->fail(SV_EINVAL, "row tiles %d", value);
            c->attn_min_rt = value;
            return SV_OK;
        default:
            return c->fail(SV_EINVAL, "unknown option %d", option);
    }
}
