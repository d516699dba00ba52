// Accept / reject over the target logits, the choice of the chain to keep, the replacement or bonus draw, and the
// cache rollback.  Passes over vocabulary-wide data, bound by HBM or, in the race, by its hash:
//   row_stats   every logits row once, in parts: max, sum exp((x - max)/temp), argmax (lowest id on ties)
//   accept      per request: all (chain, slot) decisions side by side -- p_i(d_i) from the row statistics and one gathered
//               logit; u_i * q_i(d_i) < p_i(d_i) -- then the longest chain (lowest id on ties)
//   draw        one pass over the row that the kept chain's last token comes from (and the draft distribution's row when
//               a draft was rejected): weights w = max(p - q, 0) or p; inverse-CDF or exponential race.  Match
//               verification draws every row first and compares afterwards.
//   finish      the race's winner over the parts, output tokens, live length
// A launch costs more than the small stages do, so whoever needs a row's statistics folds its parts itself, the chain is
// chosen before the draw (one draw per request, not one per chain) and the length is advanced by whoever knows it last.
#include <math.h>
#include <algorithm>
#include "common.h"
#include "kernels.h"

namespace sv {

constexpr int NT = 1024;                                  // threads of an inverse-CDF draw
constexpr int NS = 256;                                   // threads of a statistics or race work-group

// Parts a vocabulary is cut into for `rows` rows: enough work-groups of 256 threads to fill the chip (few rows of a wide
// vocabulary), eight of them at many rows, no part shorter than one load of its threads.  Five rows of 152064: 8 parts of
// 1024 threads took 8.5 us, 32 of 256 take 7.2; 640 rows 94 us (4.1 TB/s) either way.
static int vocab_parts(int rows, int V) {
    const int want = std::min(32, std::max(kDrawParts, (4096 + rows - 1) / rows));
    return std::max(1, std::min(want, V / (4 * NS)));
}
size_t sample_part_entries(int rows) { return (size_t)kDrawParts * rows + 4096; }   // >= vocab_parts * rows

__device__ __forceinline__ int window_of(const SampleArgs& a, int b) { return a.draft_lens ? max(0, min(a.draft_lens[b], a.k)) : a.k; }

// Is row j of a request (0 = x0, then the drafts chain by chain) ever looked at?  Rows behind the draft window are not.
__device__ __forceinline__ bool row_counts(int j, int k, int klim) { return row_index_in_chain(j, k) <= klim; }

struct Stat { float m, s; int am; };

// A thread's ids are loaded four at a time, kAhead loads per batch and the next batch in flight while one is worked on
// (one new maximum and one rescale per batch, not per load); the exponentials are the hardware's base-2 ones on
// pre-scaled arguments.  2304 rows of 152064: 259 us (5.4 TB/s); with both ways of reading in one kernel, at 86 registers instead
// of 50, 299; with work-groups of 1024 threads and one batch each 340.
// VEC: rows end with a whole piece of four ids.  Otherwise they are read one by one, and a NaN among them counts as no id.
template <bool VEC>
__global__ __launch_bounds__(NS) void row_stats_kernel(SampleArgs a, float inv_temp) {
    const int t = blockIdx.x, V = a.V, n = 1 + a.N * a.k;
    if (a.draft_lens && !row_counts(t % n, a.k, window_of(a, t / n))) return;
    const float* row = a.logits + (int64_t)t * V;
    const int span = ((V + gridDim.y - 1) / gridDim.y + 3) & ~3;          // ids per part, a multiple of 4
    const int vbeg = blockIdx.y * span, vend = min(V, vbeg + span);
    float m = -INFINITY, s = 0.f;
    int am = 0x7fffffff;
    const float c2 = inv_temp * 1.4426950408889634f;
    constexpr int kAhead = 4, STEP = 4 * NS * kAhead;
    auto load = [&](int v0, floatx4 (&x)[kAhead]) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int v = v0 + u * 4 * NS;
            x[u] = floatx4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
            if (VEC) {
                if (v < vend) x[u] = *reinterpret_cast<const floatx4_any*>(row + v);
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (v + i < vend) x[u][i] = row[v + i];
            }
        }
    };
    auto take = [&](int v0, const floatx4 (&x)[kAhead]) __attribute__((always_inline)) {
        float mx = -INFINITY;
#pragma unroll
        for (int u = 0; u < kAhead; ++u) mx = fmaxf(mx, fmaxf(fmaxf(x[u][0], x[u][1]), fmaxf(x[u][2], x[u][3])));
        if (mx > m) {                                      // new maximum: its first holder in ascending id order
            s *= __builtin_amdgcn_exp2f((m - mx) * c2);    // (m = -inf: s is 0 and stays 0)
            m = mx;
#pragma unroll
            for (int u = kAhead - 1; u >= 0; --u)
#pragma unroll
                for (int i = 3; i >= 0; --i)
                    if (x[u][i] == mx) am = v0 + u * 4 * NS + i;
        }
        if (mx > -INFINITY) {
            float add = 0.f;
#pragma unroll
            for (int u = 0; u < kAhead; ++u)
                add += (__builtin_amdgcn_exp2f((x[u][0] - m) * c2) + __builtin_amdgcn_exp2f((x[u][1] - m) * c2)) +
                       (__builtin_amdgcn_exp2f((x[u][2] - m) * c2) + __builtin_amdgcn_exp2f((x[u][3] - m) * c2));
            if (!VEC && __builtin_expect(add != add, 0)) {
                add = 0.f;
#pragma unroll 1
                for (int u = 0; u < 4 * kAhead; ++u) {
                    const int v = v0 + (u >> 2) * 4 * NS + (u & 3);
                    const float y = v < vend ? row[v] : -INFINITY;
                    add += y > -INFINITY ? __builtin_amdgcn_exp2f((y - m) * c2) : 0.f;
                }
            }
            s += add;
        }
    };
    floatx4 xa[kAhead], xb[kAhead];
    int v = vbeg + 4 * threadIdx.x;
    load(v, xa);
    for (; v < vend; v += 2 * STEP) {
        load(v + STEP, xb);
        __builtin_amdgcn_sched_barrier(0);
        take(v, xa);
        load(v + 2 * STEP, xa);
        __builtin_amdgcn_sched_barrier(0);
        take(v + STEP, xb);
    }
    __shared__ float sm[NS / 64], ss[NS / 64];
    __shared__ int sa[NS / 64];
    // wave merge, then group merge: (m, s, am) with ties on m resolved to the lower id
    auto merge = [&](float& m1, float& s1, int& a1, float m2, float s2, int a2) {
        const float mm = fmaxf(m1, m2);
        const float f1 = m1 == -INFINITY ? 0.f : expf((m1 - mm) * inv_temp);
        const float f2 = m2 == -INFINITY ? 0.f : expf((m2 - mm) * inv_temp);
        s1 = s1 * f1 + s2 * f2;
        if (m2 > m1 || (m2 == m1 && a2 < a1)) a1 = a2;
        m1 = mm;
    };
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const float m2 = __shfl_xor(m, o), s2 = __shfl_xor(s, o);
        const int a2 = __shfl_xor(am, o);
        merge(m, s, am, m2, s2, a2);
    }
    if ((threadIdx.x & 63) == 0) {
        sm[threadIdx.x >> 6] = m;
        ss[threadIdx.x >> 6] = s;
        sa[threadIdx.x >> 6] = am;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < NS / 64; ++w) merge(m, s, am, sm[w], ss[w], sa[w]);
        reinterpret_cast<floatx4_any*>(a.stat_part)[(int64_t)t * gridDim.y + blockIdx.y] = floatx4{m, s, __int_as_float(am), 0.f};
    }
}

// A row's statistics from its parts (ascending ids: of equal maxima the first part's id stays).
__device__ __forceinline__ Stat row_stat(const SampleArgs& a, int row, float inv_temp) {
    const floatx4_any* in = reinterpret_cast<const floatx4_any*>(a.stat_part) + (int64_t)row * a.stat_parts;
    Stat r{-INFINITY, 0.f, 0x7fffffff};
#pragma unroll 8
    for (int i = 0; i < a.stat_parts; ++i) {
        const float m = in[i][0];
        const int am = __float_as_int(in[i][2]);
        r.am = m > r.m ? am : r.am;
        r.m = fmaxf(r.m, m);
    }
#pragma unroll 8
    for (int i = 0; i < a.stat_parts; ++i) {
        const float m = in[i][0];
        r.s += m == -INFINITY ? 0.f : in[i][1] * expf((m - r.m) * inv_temp);
    }
    return r;
}

// Logits row that holds the target distribution of draft slot i (1-based) of chain c of request b.
__device__ __forceinline__ int slot_row(int b, int c, int i, int n, int k) {
    return b * n + (i == 1 ? 0 : 1 + c * k + (i - 2));
}

// Winner of a race over its parts (larger score; lower id among equals); the residual's if it has one.
__device__ __forceinline__ int race_winner(const SampleArgs& a, int64_t idx, bool rejected) {
    const floatx4_any* in = reinterpret_cast<const floatx4_any*>(a.draw_part) + idx * a.draw_parts;
    float best_r = -INFINITY, best_p = -INFINITY;
    int arg_r = 0x7fffffff, arg_p = 0x7fffffff;
#pragma unroll 8
    for (int i = 0; i < a.draw_parts; ++i) {
        const float r = in[i][0], p = in[i][2];
        const int ar = __float_as_int(in[i][1]), ap = __float_as_int(in[i][3]);
        if (r > best_r || (r == best_r && ar < arg_r)) { best_r = r; arg_r = ar; }
        if (p > best_p || (p == best_p && ap < arg_p)) { best_p = p; arg_p = ap; }
    }
    return (rejected && best_r > -INFINITY) ? arg_r : arg_p;
}

// Output tokens and live length of request b (all lanes of its wave).
__device__ __forceinline__ void emit(const SampleArgs& a, int b, int best, int acc, int tok) {
    int32_t* out = a.out_tokens + (int64_t)b * (a.k + 1);
    for (int i = threadIdx.x; i <= a.k; i += 64)
        out[i] = i < acc ? a.drafts[((int64_t)b * a.N + best) * a.k + i] : i == acc ? tok : -1;
    if (threadIdx.x == 0) {
        a.accepted_len[b] = acc;
        a.best_chain[b] = best;
        if (a.seq_len) a.seq_len[a.batch_seq[b]] += acc + 1;
    }
}

constexpr int kChains = 1024;                             // chains of a request whose verdicts are in LDS at a time

// One wave per request.  Greedy verification ends here, match verification too (its rows were drawn before: each row's
// token is folded from the race's parts first); stochastic verification leaves the kept chain for the draw.
template <int MODE>
__global__ __launch_bounds__(64) void accept_kernel(SampleArgs a) {
    __shared__ int acc_sh[kChains];
    const int b = blockIdx.x, lane = threadIdx.x;
    const int n = 1 + a.N * a.k, klim = window_of(a, b);
    const float inv_temp = 1.0f / a.temperature;
    float* tok_of = a.stat_part + (int64_t)b * n * a.stat_parts * 4;      // match: a row's token, over its statistics
    if (MODE == 2) {
        for (int j = lane; j < n; j += 64)
            if (row_counts(j, a.k, klim)) tok_of[(int64_t)j * a.stat_parts * 4] = __int_as_float(race_winner(a, (int64_t)b * n + j, false));
    }
    auto slot_token = [&](int row) {
        return MODE == 2 ? __float_as_int(tok_of[(int64_t)(row - b * n) * a.stat_parts * 4]) : row_stat(a, row, inv_temp).am;
    };
    int best = 0, acc = -1;
    for (int c0 = 0; c0 < a.N; c0 += kChains) {
        const int chains = min(kChains, a.N - c0);
        for (int c = lane; c < chains; c += 64) acc_sh[c] = klim;
        __syncthreads();
        for (int i0 = lane; i0 < chains * a.k; i0 += 64) {
            const int c = c0 + i0 / a.k, i = i0 % a.k + 1;
            if (i > klim) continue;
            const int row = slot_row(b, c, i, n, a.k);
            const int64_t d = ((int64_t)b * a.N + c) * a.k + (i - 1);
            const int x = a.drafts[d];
            bool ok = false;                               // not a token of this vocabulary: rejected, nothing is read at it
            if ((unsigned)x < (unsigned)a.V) {
                if (MODE == 1) {
                    const Stat st = row_stat(a, row, inv_temp);
                    const float p = expf((a.logits[(int64_t)row * a.V + x] - st.m) * inv_temp) / st.s;
                    const float q = a.draft_probs ? a.draft_probs[d * a.V + x] : 1.0f;
                    ok = a.uniforms[((int64_t)b * a.N + c) * (a.k + 1) + (i - 1)] * q < p;
                } else {
                    ok = x == slot_token(row);
                }
            }
            if (!ok) atomicMin(&acc_sh[c - c0], i - 1);
        }
        __syncthreads();
        for (int c = 0; c < chains; ++c)
            if (acc_sh[c] > acc) { acc = acc_sh[c]; best = c0 + c; }
        __syncthreads();                                   // read before the next chains start over
    }
    if (MODE == 1) {
        if (lane == 0) { a.accepted_len[b] = acc; a.best_chain[b] = best; }
    } else {
        emit(a, b, best, acc, slot_token(slot_row(b, best, acc + 1, n, a.k)));
    }
}

// End of stochastic verification.
__global__ __launch_bounds__(64) void finish_kernel(SampleArgs a) {
    const int b = blockIdx.x;
    const int acc = a.accepted_len[b];
    emit(a, b, a.best_chain[b], acc, race_winner(a, b, acc < window_of(a, b)));
}

__device__ __forceinline__ uint64_t splitmix_finalise(uint64_t z) {
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// What a draw draws from.  ROWS == false (stochastic verification): the last token of a request's kept chain, from the
// residual after a rejection or from the bonus row.  ROWS == true (match verification): the target's own token of one
// logits row, i.e. of one draft slot, from that row's distribution; the randomness is keyed by the request's index in
// the batch and the slot alone (the uniform of chain 0), so every chain of a request is held to the same token at the
// same slot.
struct Draw { int row, xrej; bool rejected, dead; const float* qrow; float u; uint32_t key_hi; };
template <bool ROWS>
__device__ __forceinline__ Draw draw_of(const SampleArgs& a, int idx) {
    const int n = 1 + a.N * a.k;
    const int b = ROWS ? idx / n : idx;
    const int klim = window_of(a, b);
    const int j = ROWS ? idx % n : 0;
    const int acc = ROWS ? 0 : a.accepted_len[b], c = ROWS ? 0 : a.best_chain[b];
    const int64_t s = (int64_t)b * a.N + c;
    Draw d;
    d.dead = ROWS && !row_counts(j, a.k, klim);
    d.rejected = !ROWS && acc < klim;
    d.row = ROWS ? idx : slot_row(b, c, acc + 1, n, a.k);
    // a rejected id outside the vocabulary was rejected unread: the replacement comes from p_r itself (q taken as zero)
    const int xraw = d.rejected ? a.drafts[s * a.k + acc] : -1;
    d.xrej = (unsigned)xraw < (unsigned)a.V ? xraw : -1;
    d.qrow = (d.rejected && a.draft_probs && d.xrej >= 0) ? a.draft_probs + (s * a.k + acc) * a.V : nullptr;
    // slot served by row j of a request: row 0 -> slot 1, the row of draft i of any chain -> slot i + 1
    d.u = ROWS ? a.uniforms[(int64_t)b * a.N * (a.k + 1) + row_index_in_chain(j, max(a.k, 1))] : a.uniforms[s * (a.k + 1) + a.k];
    d.key_hi = (uint32_t)(ROWS ? b : s);
    return d;
}

// Exponential race: argmax_v ln w_v - ln e_v, e_v = -log1p(-U_v); the residual's winner and, for the case that the
// residual is identically zero, the winner under p as well.  Per id the race needs a hash, and two logarithms that
// almost no id needs: e_v >= U_v, so an id can only beat the best score s so far if w_v > U_v e^s, and that is tested
// with the hardware's base-2 exponential and a margin of a thousandth (where the exponential is about to flush to zero the
// rounding of its argument, near 120, is the larger error: 1e-5).  A wave shares its best score; it runs
// the logarithms for a few of its ids only.  One draw per request over 152064 ids, with both logarithms for every id
// before: 256 requests 186 -> 112 us, 128 requests 86 -> 66, one request 29 -> 19 (start-up chain: verdict, row, parts).
// The test starts from a lower bound of the score of the row's most likely id, which the statistics name: every wave began with none, and
// worked its way up through half a dozen rounds of logarithms.  Where that id holds 0.9 of the probability 256 requests take 95 -> 68 us, 128
// requests 71 -> 55, five 17.2 -> 12.6, match draws of 147 rows 67 -> 52 and of 96 rows 51 -> 41; in flat rows (logits of standard deviation 0.3), which the
// bound does not help, 94.0 -> 93.7, 70.3 -> 70.5, 16.9 -> 18.1, 66 -> 66, 51 -> 51.  (Its exact score, by the library's logarithms, and branches over the parts for
// the id cost flat rows 3 to 4 us: code that runs once is mostly waited for.)
template <bool ROWS>
__global__ __launch_bounds__(NS) void race_kernel(SampleArgs a) {
    const Draw d = draw_of<ROWS>(a, blockIdx.x);
    if (d.dead) return;
    const int V = a.V;
    const float* lrow = a.logits + (int64_t)d.row * V;
    const int span = ((V + gridDim.y - 1) / gridDim.y + 3) & ~3;
    const int vbeg = blockIdx.y * span, vend = min(V, vbeg + span);
    const bool vec = (V & 3) == 0;
    constexpr int STEP = 4 * NS;
    struct Ids { floatx4 x, q; };                          // four ids' logits and draft probabilities
    auto load4 = [&](const float* src, int v, float fill) __attribute__((always_inline)) {
        floatx4 x = {fill, fill, fill, fill};
        if (vec) {
            if (v < vend) x = *reinterpret_cast<const floatx4_any*>(src + v);
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (v + i < vend) x[i] = src[v + i];
        }
        return x;
    };
    auto load = [&](int v, Ids& t) __attribute__((always_inline)) {
        t.x = load4(lrow, v, -INFINITY);
        t.q = d.qrow ? load4(d.qrow, v, 0.f) : floatx4{0.f, 0.f, 0.f, 0.f};
    };
    const int v0 = vbeg + 4 * threadIdx.x;
    Ids ta, tb;
    load(v0, ta);
    const float inv_temp = 1.0f / a.temperature;
    const Stat st = row_stat(a, d.row, inv_temp);
    const float m = st.m, log_sum = logf(st.s);
    const float c2 = inv_temp * 1.4426950408889634f, l2 = log_sum * 1.4426950408889634f;
    const uint64_t key = ((uint64_t)d.key_hi << 32) | (uint64_t)__float_as_uint(d.u);
    float best_r = -INFINITY, best_p = -INFINITY;
    int arg_r = 0x7fffffff, arg_p = 0x7fffffff;
    constexpr float kMargin = 1.001f;
    constexpr uint64_t kStride = 0x9E3779B97F4A7C15ull;
    auto uniform_of = [](uint64_t seed) __attribute__((always_inline)) {
        return ((float)(uint32_t)(splitmix_finalise(seed) >> 32) + 0.5f) * 2.3283064365386963e-10f;
    };
    // e^(a score that the row's winner has at least): the wave's best, and from the start a lower bound of that of the most likely id, whichever
    // part holds it: p a thousandth too small, and at least as much as -log1p(-U) in the place of it (U + U^2 / 2 + ... below 2^-8).
    float floor_p = 0.f, floor_r = 0.f;
    if ((unsigned)st.am < (unsigned)V) {
        const float U = uniform_of(key + (uint64_t)(st.am + 1) * kStride);
        const float over_e = __builtin_amdgcn_rcpf(U < 0.00390625f ? U * 1.005f : __builtin_amdgcn_logf(1.0f - U) * -0.694f);
        const float p = __builtin_amdgcn_rcpf(st.s) * 0.999f;
        floor_p = p * over_e;
        if (d.rejected) floor_r = fmaxf(0.f, (p - (d.qrow ? d.qrow[st.am] : st.am == d.xrej ? 1.0f : 0.0f)) * over_e);
    }
    float thr_p = floor_p, thr_r = floor_r;
    auto four = [&](int v, const Ids& t) __attribute__((always_inline)) {
        const uint64_t seed = key + (uint64_t)(v + 1) * kStride;
        float U[4], p_ub[4], q[4];
        unsigned todo = 0;
        auto can_win = [&](int i) __attribute__((always_inline)) {
            return !(U[i] * thr_p > p_ub[i]) | (d.rejected & !(U[i] * thr_r > (p_ub[i] - q[i]) * kMargin));
        };
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            U[i] = uniform_of(seed + i * kStride);
            // (no smaller than what the hardware's exponential flushes to zero: still an upper bound of p)
            p_ub[i] = fmaxf(__builtin_amdgcn_exp2f(fmaf(t.x[i] - m, c2, -l2)) * kMargin, 1e-37f);
            q[i] = d.qrow ? t.q[i] : (v + i == d.xrej ? 1.0f : 0.0f);
            todo |= ((v + i < vend) & can_win(i)) ? 1u << i : 0u;
        }
        // ids that may win, each lane's next one at a time; what the new best rules out is dropped.  (One copy of the
        // logarithms per four ids: unrolled over eight of them the kernel ran out of the instruction cache, 115 -> 165 us.)
        while (__any(todo != 0)) {
            const int i = __ffs(todo) - 1;
            if (i >= 0) {
                const float x = i == 0 ? t.x[0] : i == 1 ? t.x[1] : i == 2 ? t.x[2] : t.x[3];
                const float qi = i == 0 ? q[0] : i == 1 ? q[1] : i == 2 ? q[2] : q[3];
                const float Ui = i == 0 ? U[0] : i == 1 ? U[1] : i == 2 ? U[2] : U[3];
                const float ln_e = logf(-log1pf(-Ui));
                const float lp = (x - m) * inv_temp - log_sum;
                const float sp = lp - ln_e;
                if (sp > best_p) { best_p = sp; arg_p = v + i; }
                if (d.rejected) {
                    const float w = fmaxf(expf(lp) - qi, 0.0f);
                    if (w > 0.f) {
                        const float sr = logf(w) - ln_e;
                        if (sr > best_r) { best_r = sr; arg_r = v + i; }
                    }
                }
                todo &= todo - 1;
            }
            thr_p = fmaxf(floor_p, expf(wave_max(best_p)));
            if (d.rejected) thr_r = fmaxf(floor_r, expf(wave_max(best_r)));
#pragma unroll
            for (int k = 0; k < 4; ++k) todo &= can_win(k) ? ~0u : ~(1u << k);
        }
    };
    // the bounds are uniform, so that all lanes of a wave meet in the votes and shuffles; the next ids are on their way
    for (int o = 0; vbeg + o < vend; o += 2 * STEP) {
        load(v0 + o + STEP, tb);
        four(v0 + o, ta);
        load(v0 + o + 2 * STEP, ta);
        four(v0 + o + STEP, tb);
    }
    __shared__ float sh_r[NS / 64], sh_p[NS / 64];
    __shared__ int sh_ar[NS / 64], sh_ap[NS / 64];
    auto take = [](float& bv, int& ba, float ov, int oa) {
        if (ov > bv || (ov == bv && oa < ba)) { bv = ov; ba = oa; }
    };
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        take(best_r, arg_r, __shfl_xor(best_r, o), __shfl_xor(arg_r, o));
        take(best_p, arg_p, __shfl_xor(best_p, o), __shfl_xor(arg_p, o));
    }
    if ((threadIdx.x & 63) == 0) {
        sh_r[threadIdx.x >> 6] = best_r; sh_ar[threadIdx.x >> 6] = arg_r;
        sh_p[threadIdx.x >> 6] = best_p; sh_ap[threadIdx.x >> 6] = arg_p;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < NS / 64; ++w) {
            take(best_r, arg_r, sh_r[w], sh_ar[w]);
            take(best_p, arg_p, sh_p[w], sh_ap[w]);
        }
        reinterpret_cast<floatx4_any*>(a.draw_part)[(int64_t)blockIdx.x * gridDim.y + blockIdx.y] =
            floatx4{best_r, __int_as_float(arg_r), best_p, __int_as_float(arg_p)};
    }
}

// Inverse-CDF draw: one work-group per draw.
template <bool ROWS>
__global__ __launch_bounds__(NT) void cdf_kernel(SampleArgs a) {
    const Draw d = draw_of<ROWS>(a, blockIdx.x);
    if (d.dead) return;
    const int V = a.V;
    const float* lrow = a.logits + (int64_t)d.row * V;
    const float inv_temp = 1.0f / a.temperature;
    const Stat st = row_stat(a, d.row, inv_temp);
    const float m = st.m, sum = st.s, u = d.u;

    auto prob = [&](int v) { return expf((lrow[v] - m) * inv_temp) / sum; };
    auto resid = [&](int v, float p) {          // weight of id v in the residual distribution
        if (!d.rejected) return p;
        const float q = d.qrow ? d.qrow[v] : (v == d.xrej ? 1.0f : 0.0f);
        return fmaxf(p - q, 0.0f);
    };
    // inverse CDF over ascending id.  Thread i owns the contiguous ids [i*seg, (i+1)*seg); sums in double.
    const int seg = (V + NT - 1) / NT;
    const int v0 = threadIdx.x * seg, v1 = min(V, v0 + seg);
    __shared__ double seg_r[NT], seg_p[NT];
    __shared__ int pick_seg, use_p;
    __shared__ double target, before;
    double sr = 0.0, spp = 0.0;
    for (int v = v0; v < v1; ++v) {
        const float p = prob(v);
        spp += (double)p;
        sr += (double)resid(v, p);
    }
    seg_r[threadIdx.x] = sr;
    seg_p[threadIdx.x] = spp;
    __syncthreads();
    if (threadIdx.x == 0) {
        double tot_r = 0.0, tot_p = 0.0;
        for (int i = 0; i < NT; ++i) { tot_r += seg_r[i]; tot_p += seg_p[i]; }
        const int up = !(tot_r > 0.0);
        const double* segs = up ? seg_p : seg_r;
        const double tgt = (double)u * (up ? tot_p : tot_r);
        double run = 0.0;
        int pick = -1;
        for (int i = 0; i < NT; ++i) {
            if (run + segs[i] > tgt) { pick = i; break; }
            run += segs[i];
        }
        if (pick < 0) {          // u * total reached the total through rounding: last segment with weight
            run = 0.0;
            for (int i = 0; i < NT; ++i) if (segs[i] > 0.0) pick = i;
            for (int i = 0; i < pick; ++i) run += segs[i];
        }
        pick_seg = pick; use_p = up; target = tgt; before = run;
        // no segment has a weight (NaN logits): id 0, rather than what an earlier draw left there
        if (pick < 0) reinterpret_cast<floatx4_any*>(a.draw_part)[blockIdx.x] = floatx4{-INFINITY, 0.f, 0.f, __int_as_float(0)};
    }
    __syncthreads();
    if ((int)threadIdx.x == pick_seg) {
        double run = before;
        int tok = -1, last_pos = -1;
        for (int v = v0; v < v1; ++v) {
            const float p = prob(v);
            const float w = use_p ? p : resid(v, p);
            if (w > 0.f) last_pos = v;
            run += (double)w;
            if (run > target) { tok = v; break; }
        }
        const int drawn = tok >= 0 ? tok : last_pos;
        reinterpret_cast<floatx4_any*>(a.draw_part)[blockIdx.x] = floatx4{-INFINITY, 0.f, 0.f, __int_as_float(drawn)};   // a race of one
    }
}

// Move the kept chain's accepted entries to slots L+1 .. L+a (chain 0 already sits there).  One work-group per
// (request, layer).  In the tile layout of the cache a key's K entries of one head are head_dim/8 whole 16-byte
// pieces (one per 8-wide slice of the head), moved as such with one index computation each; its V entries lie
// one element apart per dimension (V is stored transposed, keys innermost) and move one by one.  Source slots
// (>= L+1+k for a chain other than 0) and destination slots (<= L+k) never overlap.  committed: the live length has
// been advanced by acc + 1 already.
template <typename T>
__global__ __launch_bounds__(256) void compact_kernel(RollbackArgs r, bool committed) {
    const int b = blockIdx.x, layer = blockIdx.y;
    const int best = r.best_chain[b], acc = r.accepted_len[b];
    if (best <= 0 || best >= r.N || acc <= 0 || acc > r.k) return;
    const int seq = r.batch_seq[b];
    const int L = r.seq_len[seq] - (committed ? acc + 1 : 0);
    const int32_t* pages = r.page_table + (int64_t)seq * r.max_pages_per_seq;
    T* pool = reinterpret_cast<T*>(r.pool);
    const int hd = r.geom.head_dim, H = r.geom.n_kv_heads;
    constexpr int EPP = 16 / (int)sizeof(T);              // elements per 16-byte piece
    const int ppk = hd / 8;                               // pieces of 8 consecutive dimensions per (key, head)
    // K: 8 consecutive dimensions of one key are contiguous (16 bytes in bf16, two 16-byte pieces in fp32)
    for (int e = threadIdx.x; e < acc * H * ppk; e += 256) {
        const int i = e / (H * ppk) + 1, rem = e % (H * ppk), h = rem / ppk, d = (rem % ppk) * 8;
        const int src = L + 1 + best * r.k + (i - 1), dst = L + i;
        const int64_t si = kv_k_index(r.geom, layer, pages[src / r.geom.page_size], h, src % r.geom.page_size, d);
        const int64_t di = kv_k_index(r.geom, layer, pages[dst / r.geom.page_size], h, dst % r.geom.page_size, d);
#pragma unroll
        for (int q = 0; q < 8 / EPP; ++q)
            *reinterpret_cast<u32x4*>(pool + di + q * EPP) = *reinterpret_cast<const u32x4*>(pool + si + q * EPP);
    }
    // V: one element per (key, head, dimension)
    for (int e = threadIdx.x; e < acc * H * hd; e += 256) {
        const int i = e / (H * hd) + 1, rem = e % (H * hd), h = rem / hd, d = rem % hd;
        const int src = L + 1 + best * r.k + (i - 1), dst = L + i;
        pool[kv_v_index(r.geom, layer, pages[dst / r.geom.page_size], h, dst % r.geom.page_size, d)] =
            pool[kv_v_index(r.geom, layer, pages[src / r.geom.page_size], h, src % r.geom.page_size, d)];
    }
}

__global__ void commit_len_kernel(RollbackArgs r) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b < r.B) r.seq_len[r.batch_seq[b]] += r.accepted_len[b] + 1;
}

hipError_t sample_verify(const SampleArgs& args, hipStream_t st) {
    SampleArgs a = args;
    const int T = a.B * (1 + a.N * a.k);
    a.stat_parts = vocab_parts(T, a.V);
    a.draw_parts = a.sample_mode == 1 ? vocab_parts(a.verify_mode == 2 ? T : a.B, a.V) : 1;
    if (a.V % 4 == 0) hipLaunchKernelGGL(row_stats_kernel<true>, dim3(T, a.stat_parts), dim3(NS), 0, st, a, 1.0f / a.temperature);
    else hipLaunchKernelGGL(row_stats_kernel<false>, dim3(T, a.stat_parts), dim3(NS), 0, st, a, 1.0f / a.temperature);
    if (a.verify_mode == 0) {
        hipLaunchKernelGGL(accept_kernel<0>, dim3(a.B), dim3(64), 0, st, a);
    } else if (a.verify_mode == 2) {
        if (a.sample_mode == 1) hipLaunchKernelGGL(race_kernel<true>, dim3(T, a.draw_parts), dim3(NS), 0, st, a);
        else hipLaunchKernelGGL(cdf_kernel<true>, dim3(T), dim3(NT), 0, st, a);
        hipLaunchKernelGGL(accept_kernel<2>, dim3(a.B), dim3(64), 0, st, a);
    } else {
        hipLaunchKernelGGL(accept_kernel<1>, dim3(a.B), dim3(64), 0, st, a);
        if (a.sample_mode == 1) hipLaunchKernelGGL(race_kernel<false>, dim3(a.B, a.draw_parts), dim3(NS), 0, st, a);
        else hipLaunchKernelGGL(cdf_kernel<false>, dim3(a.B), dim3(NT), 0, st, a);
        hipLaunchKernelGGL(finish_kernel, dim3(a.B), dim3(64), 0, st, a);
    }
    return hipGetLastError();
}

hipError_t compact_kept(const RollbackArgs& r, bool committed, hipStream_t st) {
    if (r.N <= 1) return hipSuccess;
    if (r.dtype == 1) hipLaunchKernelGGL(compact_kernel<bf16_t>, dim3(r.B, r.n_layers), dim3(256), 0, st, r, committed);
    else hipLaunchKernelGGL(compact_kernel<float>, dim3(r.B, r.n_layers), dim3(256), 0, st, r, committed);
    return hipGetLastError();
}

hipError_t commit_lens(const RollbackArgs& r, hipStream_t st) {
    hipLaunchKernelGGL(commit_len_kernel, dim3((r.B + 63) / 64), dim3(64), 0, st, r);
    return hipGetLastError();
}

}  // namespace sv
