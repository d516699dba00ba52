// Mixture-of-experts feed-forward of the verification pass on gfx950 (bf16 weights, fp32 accumulation):
// softmax router -> top-k -> renormalised weights; rows bucketed by expert; per expert
// (silu(x Wg^T) * (x Wu^T)) Wd^T; weighted combine.  The paper evaluates such a model (Section 5.3, the
// Qwen3-235B MoE run); the FFN definition itself is the usual one of that model family.
//
// With a few dozen rows per expert the two expert products are bound by streaming the expert weights once
// (1.2 GB a layer at 128 experts of 3 x 2048 x 768), so the kernels are built around that stream: one
// work-group per (expert, strip of output features) pulls its strip of packed weight fragments straight
// from HBM into registers through a ring of loads in flight, while the expert's rows (at most 128 at a time)
// sit in LDS as MFMA operands.  Experts that received no row cost nothing.
#include <hip/hip_runtime.h>

#include "common.h"
#include "kernels.h"

namespace sv {

typedef __attribute__((ext_vector_type(16))) float floatx16;

// ------------------------------------------------------------------ router
// Logits by MFMA (v_mfma_f32_32x32x16_bf16).  A work-group takes 32 rows and one of KQ parts of the reduction;
// each of its four waves covers a quarter of that part for all ET = E/32 expert tiles -- expert rows as the
// first operand straight from the row-major router matrix, the activation fragment straight from the packed
// activations (1 KB contiguous), four slices of loads in flight ahead of the products.  The waves' partial
// logits meet in LDS and leave as one plane [part][row][expert] in global memory.
// A single tile of rows makes KQ work-groups, which is few for a cold router matrix: there every wave is a work-group
// of its own and leaves its own plane, which the choice adds up in the order in which LDS would have (20 rows: 11.9 -> 5.4 us).
constexpr int kRouterRows = 32;

template <int ET>
__global__ __launch_bounds__(256) void moe_logits_kernel(MoeArgs a, int KQ, int wave_planes) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    float* logit = reinterpret_cast<float*>(smem);           // [4 waves][32][E + 1]
    constexpr int E = 32 * ET, pitch = E + 1, plane = kRouterRows * pitch;
    // 32-row tile of the packed activations, part of the reduction; wave_planes: work-groups of one wave, a quarter part each
    const int tile = blockIdx.x, kq = wave_planes ? blockIdx.y >> 2 : blockIdx.y;
    const int lane = threadIdx.x & 63, wave = wave_planes ? blockIdx.y & 3 : threadIdx.x >> 6;
    const int l32 = lane & 31, lg = lane >> 5;
    const int kslices = a.d / 16, nks = kslices / (4 * KQ), ks0 = (kq * 4 + wave) * nks;
    const bf16_t* a_src = a.a + ((int64_t)tile * kslices + ks0) * 512 + lane * 8;
    const bf16_t* w_src = a.w_router + (int64_t)l32 * a.d + ks0 * 16 + 8 * lg;
    constexpr int GS = 4;
    floatx16 acc[ET];
#pragma unroll
    for (int et = 0; et < ET; ++et)
#pragma unroll
        for (int q = 0; q < 16; ++q) acc[et][q] = 0.f;
    u32x4 xa[2][GS], wa[2][GS][ET];
    auto load_group = [&](int g, u32x4 (&x)[GS], u32x4 (&w)[GS][ET]) {
#pragma unroll
        for (int s_ = 0; s_ < GS; ++s_) {
            const int ks = g * GS + s_;
            const bool ok = ks < nks;
            const int kc = ok ? ks : nks - 1;
            const u32x4 xv = *reinterpret_cast<const u32x4*>(a_src + (int64_t)kc * 512);
            x[s_] = ok ? xv : u32x4{0, 0, 0, 0};                // a slice past the end contributes nothing
#pragma unroll
            for (int et = 0; et < ET; ++et) w[s_][et] = *reinterpret_cast<const u32x4*>(w_src + (int64_t)et * 32 * a.d + kc * 16);
        }
    };
    auto mma_group = [&](const u32x4 (&x)[GS], const u32x4 (&w)[GS][ET]) {
#pragma unroll
        for (int s_ = 0; s_ < GS; ++s_)
#pragma unroll
            for (int et = 0; et < ET; ++et)
                acc[et] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, w[s_][et]),
                                                                 __builtin_bit_cast(bf16x8, x[s_]), acc[et], 0, 0, 0);
    };
    const int ngroups = (nks + GS - 1) / GS;
    load_group(0, xa[0], wa[0]);
    for (int g = 0; g < ngroups; g += 2) {
        load_group(g + 1, xa[1], wa[1]);                       // past the end: zero activations
        __builtin_amdgcn_sched_barrier(0);
        mma_group(xa[0], wa[0]);
        __builtin_amdgcn_sched_barrier(0);
        load_group(g + 2, xa[0], wa[0]);
        __builtin_amdgcn_sched_barrier(0);
        mma_group(xa[1], wa[1]);
        __builtin_amdgcn_sched_barrier(0);
    }
    // acc[et][4 q + i] <-> expert et*32 + 8 q + 4 lg + i, row l32
    if (wave_planes) {
        if (tile * 32 + l32 < a.T) {
            float* dst = a.router_logits + ((int64_t)blockIdx.y * a.T + tile * 32 + l32) * a.E + 4 * lg;
#pragma unroll
            for (int et = 0; et < ET; ++et)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *reinterpret_cast<floatx4*>(dst + et * 32 + 8 * q) = floatx4{acc[et][4 * q], acc[et][4 * q + 1], acc[et][4 * q + 2], acc[et][4 * q + 3]};
        }
        return;
    }
#pragma unroll
    for (int et = 0; et < ET; ++et)
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int i = 0; i < 4; ++i) logit[wave * plane + l32 * pitch + et * 32 + 8 * q + 4 * lg + i] = acc[et][4 * q + i];
    __syncthreads();
    float* dst = a.router_logits + ((int64_t)kq * a.T + (int64_t)tile * 32) * E;
#pragma unroll 8
    for (int i = threadIdx.x; i < kRouterRows * E; i += 256) {
        const int r = i / E, e = i % E;
        if (tile * 32 + r < a.T)
            dst[(int64_t)r * E + e] = (logit[r * pitch + e] + logit[plane + r * pitch + e]) + (logit[2 * plane + r * pitch + e] + logit[3 * plane + r * pitch + e]);
    }
}

// Router choice of one row by one wave.  router_sum: the row's logits, lane l those of experts l, l + 64, ..., its planes added in
// order, all of up to sixteen in flight together (one plane per part, or with QUADS four, of the part's waves).  route_row:
// softmax over the experts, top_k by repeated arg-max (lowest id among equals), renormalisation.  Lane j < top_k returns choice j.  The
// arg-max runs on the probabilities' bit patterns (ordered like the numbers; 0 = taken, or NaN: never chosen) by DPP: through shuffles
// its sixteen reductions were near half of the time (640 rows: 9.7 -> 5.8 us).
constexpr int kPerLane = 4;                                  // experts per lane: E <= 256
template <bool QUADS>
__device__ __forceinline__ void router_sum(const MoeArgs& a, int planes, int t, int lane, float (&x)[kPerLane]) {
    constexpr int BATCH = QUADS ? 16 : 4;
#pragma unroll
    for (int i = 0; i < kPerLane; ++i) x[i] = 0.f;
    for (int kq0 = 0; kq0 < planes; kq0 += BATCH) {
        float part[BATCH][kPerLane];
#pragma unroll
        for (int u = 0; u < BATCH; ++u)
#pragma unroll
            for (int i = 0; i < kPerLane; ++i)
                part[u][i] = kq0 + u < planes && lane + 64 * i < a.E ? a.router_logits[((int64_t)(kq0 + u) * a.T + t) * a.E + lane + 64 * i] : 0.f;
#pragma unroll
        for (int i = 0; i < kPerLane; ++i)
#pragma unroll
            for (int u = 0; u < BATCH; u += 4)
                if (QUADS) x[i] += (part[u][i] + part[u + 1][i]) + (part[u + 2][i] + part[u + 3][i]);
                else for (int v = 0; v < 4; ++v) x[i] += part[u + v][i];
    }
}

__device__ __forceinline__ void route_row(const MoeArgs& a, const float (&x)[kPerLane], int lane, int& id, float& weight) {
    constexpr int PER = kPerLane;
    float mx = -INFINITY;
#pragma unroll
    for (int i = 0; i < PER; ++i) mx = lane + 64 * i < a.E ? fmaxf(mx, x[i]) : mx;
    mx = wave_max(mx);
    float sum = 0.f;
    uint32_t key[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const float p = lane + 64 * i < a.E ? expf(x[i] - mx) : 0.f;
        sum += p > 0.f ? p : 0.f;
        key[i] = (lane + 64 * i < a.E && p >= 0.f) ? __float_as_uint(p) + 1 : 0;
    }
    sum = wave_sum(sum);
    float kept_sum = 0.f, mine = 0.f;
    int mine_id = 0;
    for (int j = 0; j < a.top_k; ++j) {
        uint32_t best = key[0];
        int best_e = lane;
#pragma unroll
        for (int i = 1; i < PER; ++i)
            if (key[i] > best) { best = key[i]; best_e = lane + 64 * i; }    // ascending ids: the first maximum is kept
        const uint32_t top = wave_max_u32(best);
        // lowest id among the equal maxima; with nothing left but NaN still a valid expert id
        const int win = top == 0 ? j : 255 - (int)wave_max_u32(best == top ? 255 - best_e : 0);
#pragma unroll
        for (int i = 0; i < PER; ++i)
            if (lane + 64 * i == win) key[i] = 0;
        const float p = (top == 0 ? -1.f : __uint_as_float(top - 1)) / sum;
        kept_sum += p;
        if (lane == j) { mine = p; mine_id = win; }
    }
    id = mine_id;
    weight = mine / kept_sum;
}

__global__ __launch_bounds__(256) void moe_select_kernel(MoeArgs a, int KQ) {
    const int lane = threadIdx.x & 63;
    const int t = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (t >= a.T) return;
    int id;
    float w, x[kPerLane];
    router_sum<false>(a, KQ, t, lane, x);
    route_row(a, x, lane, id, w);
    if (lane < a.top_k) {
        a.top_ids[(size_t)t * a.top_k + lane] = id;
        a.top_w[(size_t)t * a.top_k + lane] = w;
    }
}

// ------------------------------------------------------------------ grouping
// First tile of every bucket: exclusive prefix sum of the buckets' tile counts, `mine` that of expert threadIdx.x (E <= 256:
// four waves scan their 64 experts with lane shifts, then add the totals of the waves before them); and the list of the experts
// that have a tile, for the products.  All threads call it.
__device__ __forceinline__ void bucket_offsets(int mine, int32_t* offs, const MoeArgs& a) {
    __shared__ int wave_tot[4], wave_live[4];
    const int e = threadIdx.x, lane = e & 63, E = a.E;
    int incl = mine;
    const uint64_t live = __ballot(mine > 0);
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int up = __shfl_up(incl, d);
        if (lane >= d) incl += up;
    }
    if (e < 256 && lane == 63) { wave_tot[e >> 6] = incl; wave_live[e >> 6] = __popcll(live); }
    __syncthreads();
    if (e < E) {
        int base = 0, rank = __popcll(live & ((1ull << lane) - 1));
        for (int w = 0; w < (e >> 6); ++w) { base += wave_tot[w]; rank += wave_live[w]; }
        offs[e] = base + incl - mine;
        if (mine > 0) reinterpret_cast<u32x2*>(a.live)[1 + rank] = u32x2{(uint32_t)e | (uint32_t)mine << 16, (uint32_t)offs[e]};
        if (e == E - 1) { offs[E] = base + incl; a.live[0] = rank + (mine > 0); }
    }
    __syncthreads();
}

// Up to 32 rows (one operand tile): choice and grouping in one work-group, two rows per wave.  Every expert that is
// chosen at all gets one tile, in which a row stands where it stands in the activations: the products then read the
// activations' own tile, and there is nothing to gather.  20 rows: choice, grouping and gather 8.9 + 4.7 + 6.1 us in three
// launches, 11.6 in this one.
template <bool QUADS>
__global__ __launch_bounds__(1024) void moe_route_tile_kernel(MoeArgs a, int planes) {
    __shared__ int32_t chosen[256], offs[257];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (threadIdx.x < 256) chosen[threadIdx.x] = 0;
    __syncthreads();
    int id[2] = {0, 0};
    float x[2][kPerLane];
#pragma unroll
    for (int r = 0; r < 2; ++r)
        if (wave + 16 * r < a.T) router_sum<QUADS>(a, planes, wave + 16 * r, lane, x[r]);
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        const int t = wave + 16 * r;
        if (t < a.T) {
            float w;
            route_row(a, x[r], lane, id[r], w);
            if (lane < a.top_k) {
                chosen[id[r]] = 1;
                a.top_ids[t * a.top_k + lane] = id[r];
                a.top_w[t * a.top_k + lane] = w;
            }
        }
    }
    __syncthreads();
    bucket_offsets(threadIdx.x < a.E ? chosen[threadIdx.x] : 0, offs, a);
    if (threadIdx.x <= a.E) a.tile_off[threadIdx.x] = offs[threadIdx.x];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        const int t = wave + 16 * r;
        if (t < a.T && lane < a.top_k) a.inv[t * a.top_k + lane] = offs[id[r]] * 32 + t;
    }
}

// One work-group.  Every (row, expert) assignment sets bit `row` in its expert's bitmap (an OR: the result
// does not depend on the order of the atomics); the rank of a row inside its expert's bucket is the number of
// set bits below it.  Buckets are padded to whole 32-row tiles: bucket e owns padded rows
// 32 * tile_off[e] .. 32 * tile_off[e+1] - 1; perm[padded row] = source row (padding rows name row 0, their
// results are never read), inv[assignment] = padded row.
__global__ __launch_bounds__(1024) void moe_group_kernel(MoeArgs a) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int W = (a.T + 31) / 32;
    uint32_t* bm = reinterpret_cast<uint32_t*>(smem);                               // [E][W]
    uint16_t* below = reinterpret_cast<uint16_t*>(smem + (size_t)a.E * W * 4);      // [E][W] set bits in earlier words
    int32_t* offs = reinterpret_cast<int32_t*>(smem + (size_t)a.E * W * 6);          // [E + 1] first tile of a bucket
    int32_t* cnts = offs + a.E + 1;                                                  // [E]
    const int n_asg = a.T * a.top_k;
    for (int i = threadIdx.x; i < a.E * W; i += 1024) bm[i] = 0;
    __syncthreads();
    // the ids of eight assignments of a thread in flight together; those of the first eight stay for the second pass
    constexpr int AHEAD = 8;
    int kept[AHEAD];
    for (int i0 = threadIdx.x; i0 < n_asg; i0 += 1024 * AHEAD) {
        int id[AHEAD];
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) id[u] = i0 + 1024 * u < n_asg ? a.top_ids[i0 + 1024 * u] : -1;
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) {
            const int t = (i0 + 1024 * u) / a.top_k;
            if (id[u] >= 0) atomicOr(&bm[id[u] * W + (t >> 5)], 1u << (t & 31));
            if (i0 == (int)threadIdx.x) kept[u] = id[u];
        }
    }
    __syncthreads();
    for (int e = threadIdx.x; e < a.E; e += 1024) {
        int run = 0;
        for (int w = 0; w < W; ++w) {
            below[e * W + w] = (uint16_t)run;
            run += __popc(bm[e * W + w]);
        }
        cnts[e] = run;
    }
    __syncthreads();
    bucket_offsets(threadIdx.x < a.E ? (cnts[threadIdx.x] + 31) / 32 : 0, offs, a);
    for (int e = threadIdx.x; e <= a.E; e += 1024) {
        a.tile_off[e] = offs[e];
        if (e < a.E) {
            for (int r = cnts[e]; r < (offs[e + 1] - offs[e]) * 32; ++r) a.perm[offs[e] * 32 + r] = 0;
        }
    }
    for (int i0 = threadIdx.x; i0 < n_asg; i0 += 1024 * AHEAD) {
        if (i0 != (int)threadIdx.x) {
#pragma unroll
            for (int u = 0; u < AHEAD; ++u) kept[u] = i0 + 1024 * u < n_asg ? a.top_ids[i0 + 1024 * u] : -1;
        }
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) {
            const int i = i0 + 1024 * u, t = i / a.top_k, e = kept[u];
            if (e < 0) continue;
            const int r = below[e * W + (t >> 5)] + __popc(bm[e * W + (t >> 5)] & ((1u << (t & 31)) - 1u));
            const int prow = offs[e] * 32 + r;
            a.inv[i] = prow;
            a.perm[prow] = t;
        }
    }
}

// ------------------------------------------------------------------ rows of a bucket as operand tiles
// The packed activations keep 16 bytes of a row per 1 KB fragment, so a strip that gathered its expert's rows
// itself would pull a whole cache line for every 16 bytes, and every one of the F/64 strips of the expert again
// (measured: 2.7 GB of L2 requests per layer for 0.8 GB of weights).  The gather is done once instead: two
// work-groups copy the 32 rows of one padded tile (half of the slices each) into operand order [tile][d/16][64][8].  The tiles live in
// the buffer of the expert outputs y, which is not written before the first product has read them.
__global__ __launch_bounds__(256) void moe_gather_kernel(MoeArgs a) {
    const int tile = blockIdx.x;
    if (tile >= a.tile_off[a.E]) return;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int kslices = a.d / 16;
    const int t = a.perm[tile * 32 + (lane & 31)];
    const bf16_t* src = a.a + ((int64_t)(t >> 5) * kslices) * 512 + ((t & 31) + 32 * (lane >> 5)) * 8;
    bf16_t* dst = reinterpret_cast<bf16_t*>(a.y) + ((int64_t)tile * kslices) * 512 + lane * 8;
    const int half = kslices / 2;                               // blockIdx.y: which half of the slices
    for (int s0 = blockIdx.y * half + wave * 4; s0 < (blockIdx.y + 1) * half; s0 += 16) {   // four slices in flight per wave
        u32x4 v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = *reinterpret_cast<const u32x4*>(src + (int64_t)(s0 + i) * 512);
#pragma unroll
        for (int i = 0; i < 4; ++i) store_stream(reinterpret_cast<u32x4*>(dst + (int64_t)(s0 + i) * 512), v[i]);
    }
}

// ------------------------------------------------------------------ expert products
// MODE 0: rows = the gathered tiles (up to 32 rows: the activations' only tile); waves 0,1 produce 64 gate features,
//         waves 2,3 the 64 up features of the same indices; the epilogue forms silu(gate) * up and writes it, rounded to
//         bf16, as packed MFMA operand tiles for MODE 1.
// MODE 1: rows = those tiles; four waves produce 128 output features; fp32 results go to y[padded row][d].
// A work-group handles the expert's row tiles MTMAX at a time (re-streaming its weight strip for experts with more).  Most
// experts hold one or two tiles, and what a group of MT tiles costs beside the weights grows with MT: a fill copies
// MT x 8 KB through L2, LDS and registers, as much as the weights themselves at MT = 4.  So the loop exists for one, two
// and four tiles, and the launch takes the smallest MTMAX that holds an ordinary expert, with as many work-groups per CU as
// its registers and LDS leave room for.  128 experts of 3 x 2048 x 768, against four tiles throughout: 640 rows (two tiles an
// expert) 171.9 + 88.8 -> 160.5 + 85.6 us, 20 rows (one) 129.7 + 65.7 -> 118.1 + 63.9 (4.9 TB/s of weights; a plain
// stream reaches 6.0).  Sixteen weight fragments in flight instead of eight, where one tile leaves registers for them, 2 %;
// with two tiles they cost the fourth work-group and gain nothing.
// The gathered tiles, silu(gate) * up and the outputs leave as streams (store_stream; of 640 rows 31, 12 and 62 MB).  640 rows: gather 11.6 -> 10.7
// us, products 167 + 88.5 -> 157 + 87, the next layer's attention 235 -> 231, the norm that combines the outputs 8.8 -> 9.3; 20 rows 114 + 58.6 ->
// 112 + 58.7; one to ten rows level.  The weights are read as a stream as well: 640 rows 157 + 88.5 -> 146 + 86.5, 20 rows 111 + 57.7 -> 104 + 58.4.
constexpr int kMoeSlices = 8;                               // 16-wide slices per fill

template <int MODE, int MT, bool STREAM>
__device__ __forceinline__ void moe_tiles(const MoeArgs& a, unsigned char* abuf, const char* w_base, int p, int tile, int nt_here, bool one_tile) {
    constexpr int KA = kMoeSlices, PD = (MT == 1 ? 2 : 1) * kMoeSlices, APW = MT * KA / 4;
    const int K = MODE == 0 ? a.d : a.F;                    // reduction width
    const int kslices = K / 16, nfill = kslices / KA;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l32 = lane & 31, lg = lane >> 5;

    // this wave's share of a fill: APW slices of row tile wave * MT / 4; tiles past the bucket repeat its last
    const int my = wave * MT / 4, ks_mine = (wave * APW) % KA;
    const bf16_t* rows = MODE == 1 ? a.act : one_tile ? a.a : reinterpret_cast<const bf16_t*>(a.y);
    // Both streams are read through buffer descriptors: a slice is a scalar offset, so that the ring needs no lane addresses
    // (sixteen of them spilled).  The scalar offset is no part of a descriptor's range check, so what is requested past the end
    // is the last slice or fill again, never the memory behind the matrix.
    const char* a_base = reinterpret_cast<const char*>(rows + ((int64_t)(MODE == 0 && one_tile ? 0 : tile + (my < nt_here ? my : nt_here - 1)) * kslices + ks_mine) * 512);
    const auto a_desc = buffer_of(a_base, (kslices - ks_mine) * 1024), w_desc = buffer_of(w_base, (kslices - 1) * 4096 + 1024);
    auto load_a = [&](int slice) __attribute__((always_inline)) { return buffer_load16(a_desc, lane * 16, slice * 1024); };
    auto load_w = [&](int slice) __attribute__((always_inline)) { return buffer_load16<STREAM ? kStreamLoad : 0>(w_desc, lane * 16, slice * 4096); };
    unsigned char* a_dst = abuf + (wave * APW) * 1024 + lane * 16;
    constexpr int BUF = MT * KA * 1024;

    floatx16 acc[MT];
#pragma unroll
    for (int j = 0; j < MT; ++j)
#pragma unroll
        for (int q = 0; q < 16; ++q) acc[j][q] = 0.f;

    u32x4 wring[PD];
    // The rows of a fill are requested two fills ahead: loads return in order, so what is waited for at the end of a fill
    // must be older than the weights that are to stay in flight.
    u32x4 areg[2][APW];
#pragma unroll
    for (int f = 0; f < 2; ++f)
#pragma unroll
        for (int i = 0; i < APW; ++i) areg[f][i] = load_a(min(f, nfill - 1) * KA + i);
#pragma unroll
    for (int s = 0; s < PD; ++s) wring[s] = load_w(min(s, kslices - 1));
#pragma unroll
    for (int i = 0; i < APW; ++i) *reinterpret_cast<u32x4*>(a_dst + i * 1024) = areg[0][i];

    // a fill from LDS buffer (MT = 1: and ring half) H = fill % 2
    auto do_fill = [&](int fill, auto half) __attribute__((always_inline)) {
        constexpr int H = decltype(half)::value;
        __builtin_amdgcn_s_waitcnt(0xC07F);                 // own LDS writes done
        __builtin_amdgcn_s_barrier();
#pragma unroll
        for (int i = 0; i < APW; ++i) areg[H][i] = load_a(min(fill + 2, nfill - 1) * KA + i);
        const unsigned char* ab = abuf + H * BUF + lane * 16;
        bf16x8 af[2][MT];
#pragma unroll
        for (int j = 0; j < MT; ++j) af[0][j] = *reinterpret_cast<const bf16x8*>(ab + (j * KA) * 1024);
#pragma unroll
        for (int s = 0; s < KA; ++s) {
            const int slice = fill * KA + s;
            if (s + 1 < KA) {
#pragma unroll
                for (int j = 0; j < MT; ++j)
                    af[(s + 1) & 1][j] = *reinterpret_cast<const bf16x8*>(ab + (j * KA + s + 1) * 1024);
            }
            __builtin_amdgcn_sched_barrier(0);
            const bf16x8 wf = __builtin_bit_cast(bf16x8, wring[(H * KA + s) % PD]);
#pragma unroll
            for (int j = 0; j < MT; ++j)
                if (MT < 4 || j < nt_here)    // MODE 1: rows first, so that a half wave stores 128 contiguous bytes of an output row
                    acc[j] = MODE == 0 ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf, af[s & 1][j], acc[j], 0, 0, 0)
                                       : __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[s & 1][j], wf, acc[j], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            // refill the slot just consumed (after its readers, so the load lands in place)
            wring[(H * KA + s) % PD] = load_w(min(slice + PD, kslices - 1));
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int i = 0; i < APW; ++i) *reinterpret_cast<u32x4*>(a_dst + (1 - H) * BUF + i * 1024) = areg[1 - H][i];
    };
    for (int fill = 0; fill + 1 < nfill; fill += 2) {
        do_fill(fill, std::integral_constant<int, 0>{});
        do_fill(fill + 1, std::integral_constant<int, 1>{});
    }
    if (nfill & 1) do_fill(nfill - 1, std::integral_constant<int, 0>{});

    if (MODE == 1) {
#pragma unroll
        for (int j = 0; j < MT; ++j) {
            if (j < nt_here) {
                // acc[j][4 q + r] <-> padded row 32 (tile + j) + 8 q + 4 lg + r, feature 128 p + 32 wave + l32
                float* dst = a.y + ((int64_t)(tile + j) * 32 + 4 * lg) * a.d + p * 128 + wave * 32 + l32;
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int r = 0; r < 4; ++r) store_stream(dst + (int64_t)(8 * q + r) * a.d, (float)acc[j][4 * q + r]);
            }
        }
        __builtin_amdgcn_s_waitcnt(0xC07F);
        __builtin_amdgcn_s_barrier();                       // every wave is done with abuf before the next group refills it
    } else {
        // up halves travel through LDS to the waves that hold the gate halves of the same features
        __builtin_amdgcn_s_waitcnt(0xC07F);
        __builtin_amdgcn_s_barrier();                       // all reads of abuf are over
        float* xbuf = reinterpret_cast<float*>(abuf);       // [2 waves][MT][16][64] floats
        if (wave >= 2) {
#pragma unroll
            for (int j = 0; j < MT; ++j)
#pragma unroll
                for (int q = 0; q < 16; ++q) xbuf[(((wave - 2) * MT + j) * 16 + q) * 64 + lane] = acc[j][q];
        }
        __builtin_amdgcn_s_waitcnt(0xC07F);
        __builtin_amdgcn_s_barrier();
        if (wave < 2) {
            const int fs = (p * 64 + wave * 32) / 16;       // first 16-wide feature slice of this wave
#pragma unroll
            for (int j = 0; j < MT; ++j) {
                if (j < nt_here) {
                    bf16_t* dst = a.act + ((int64_t)(tile + j) * (a.F / 16) + fs) * 512;
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        float r[4];
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const float g = acc[j][4 * q + i];
                            const float u = xbuf[((wave * MT + j) * 16 + 4 * q + i) * 64 + lane];
                            r[i] = silu_mul(g, u);
                        }
                        // features 8q + 4 lg .. +3 of this wave's 32: slice q/2, half q%2, elements 4 lg ..
                        u32x2 pk = {pack2bf(r[0], r[1]), pack2bf(r[2], r[3])};
                        store_stream(reinterpret_cast<u32x2*>(dst + ((q >> 1) * 64 + l32 + 32 * (q & 1)) * 8 + 4 * lg), pk);
                    }
                }
            }
        }
        __builtin_amdgcn_s_waitcnt(0xC07F);
        __builtin_amdgcn_s_barrier();                       // xbuf is read before the next group overwrites it
    }
}

template <int MODE, int MTMAX>
__global__ __launch_bounds__(256, MTMAX == 4 ? 2 : 4) void moe_gemm_kernel(MoeArgs a, int one_tile) {
    __shared__ __attribute__((aligned(16))) unsigned char abuf[2 * MTMAX * kMoeSlices * 1024];
    const int Ntot = MODE == 0 ? 2 * a.F : a.d;             // weight rows per expert
    const int strips = MODE == 0 ? a.F / 64 : a.d / 128;
    // consecutive work-group ids go round the eight XCDs: the strips of an expert are given ids eight apart, so
    // that they share one L2 and the expert's tiles are fetched once (E is a multiple of 8).  The experts are those that have
    // rows, dealt to the XCDs in turn: by their own numbers one XCD may get fourteen of them and another ten (20 rows, 93 of 128
    // experts: the two products of a layer 184 -> 173 us).
    const int grp = blockIdx.x / (8 * strips), in_grp = blockIdx.x % (8 * strips);
    const int at = grp * 8 + (in_grp & 7), p = in_grp >> 3;
    if (at >= a.live[0]) return;
    const u32x2 entry = reinterpret_cast<const u32x2*>(a.live)[1 + at];
    const int e = entry[0] & 0xffff, ntile = entry[0] >> 16, tile0 = entry[1];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int nt_local;                                           // this wave's 32-feature tile among the expert's rows
    if (MODE == 0) nt_local = wave < 2 ? 2 * p + wave : a.F / 32 + 2 * p + (wave - 2);
    else nt_local = 4 * p + wave;
    const int nt = e * (Ntot / 32) + nt_local, kslices = (MODE == 0 ? a.d : a.F) / 16;
    const char* w_base = reinterpret_cast<const char*>((MODE == 0 ? a.w_gate_up : a.w_down) + (((int64_t)(nt >> 2) * kslices) * 4 + (nt & 3)) * 512);
    auto groups = [&](auto stream) __attribute__((always_inline)) {
        constexpr bool STREAM = decltype(stream)::value;
        for (int g0 = 0; g0 < ntile; g0 += MTMAX) {
            const int left = ntile - g0, nt_here = left < MTMAX ? left : MTMAX;
            if (MTMAX == 1 || nt_here == 1) moe_tiles<MODE, 1, STREAM>(a, abuf, w_base, p, tile0 + g0, 1, one_tile);
            else if (MTMAX == 2 || nt_here == 2) moe_tiles<MODE, 2, STREAM>(a, abuf, w_base, p, tile0 + g0, 2, one_tile);
            else if constexpr (MTMAX == 4) moe_tiles<MODE, 4, STREAM>(a, abuf, w_base, p, tile0 + g0, nt_here, one_tile);
        }
    };
    // As a stream where the strip is read once: the second group of an expert with more tiles finds it in L2 (three layers of 128 experts, us a
    // pass, streamed throughout against this: 2304 rows 4085 -> 3923, prompts of 100 to 500 tokens, 24 and 8, 5987 -> 5657 and 2636 -> 2525)
    if (a.cold && ntile <= MTMAX) groups(std::true_type{});
    else groups(std::false_type{});
}

// ------------------------------------------------------------------ combine
// out[t][:] = sum over the row's top_k experts, in slot order, of weight * y[padded row of that assignment][:]
__global__ __launch_bounds__(256) void moe_combine_kernel(MoeArgs a) {
    const int t = blockIdx.x;
    for (int c = threadIdx.x * 4; c < a.d; c += 1024) {
        floatx4 s = {0.f, 0.f, 0.f, 0.f};
        for (int j = 0; j < a.top_k; ++j) {
            const float w = a.top_w[(size_t)t * a.top_k + j];
            const floatx4 v = *reinterpret_cast<const floatx4*>(a.y + (int64_t)a.inv[(size_t)t * a.top_k + j] * a.d + c);
            s[0] = fmaf(w, v[0], s[0]); s[1] = fmaf(w, v[1], s[1]); s[2] = fmaf(w, v[2], s[2]); s[3] = fmaf(w, v[3], s[3]);
        }
        *reinterpret_cast<floatx4*>(a.out + (int64_t)t * a.d + c) = s;
    }
}

int moe_shape_ok(int T, int d, int E, int top_k, int F) {
    if (T <= 0 || d <= 0 || E <= 0 || top_k <= 0 || F <= 0) return 0;
    if (E % 64 != 0 || E > 256 || top_k > E || top_k > 64) return 0;       // router: 32-expert MFMA tiles, four experts per lane, top_k <= lanes
    if (d % 128 != 0 || F % 128 != 0) return 0;                            // eight 16-wide slices per fill; 128-feature strips
    if (moe_group_lds_bytes(T, E) > 150 * 1024 || (size_t)4 * kRouterRows * (E + 1) * 4 > 150 * 1024) return 0;
    return 1;
}

size_t moe_group_lds_bytes(int T, int E) {
    const size_t W = (T + 31) / 32;
    return (size_t)E * W * 6 + (size_t)(2 * E + 1) * 4 + 16;
}

int moe_max_tiles(int T, int E, int top_k) { return (T * top_k) / 32 + E; }

hipError_t moe_ffn(const MoeArgs& a, hipStream_t st) {
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e1 = hipFuncSetAttribute(reinterpret_cast<const void*>(moe_group_kernel),
                                            hipFuncAttributeMaxDynamicSharedMemorySize, 150 * 1024);
        if (e1 != hipSuccess) return e1;
        for (const void* k : {reinterpret_cast<const void*>(moe_logits_kernel<2>), reinterpret_cast<const void*>(moe_logits_kernel<4>),
                              reinterpret_cast<const void*>(moe_logits_kernel<6>), reinterpret_cast<const void*>(moe_logits_kernel<8>)}) {
            hipError_t e2 = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, 150 * 1024);
            if (e2 != hipSuccess) return e2;
        }
        attr_set = true;
    }
    // parts of the router's reduction: as many as leave every wave at least two 16-wide slices, at most four
    const int kslices = a.d / 16;
    int KQ = 4;
    while (KQ > 1 && (kslices % (4 * KQ) != 0 || kslices / (4 * KQ) < 2)) KQ >>= 1;
    const bool one_tile = a.T <= 32, wave_planes = one_tile && a.router_parts >= 4 * KQ;
    const size_t router_lds = (size_t)4 * kRouterRows * (a.E + 1) * 4;
    const dim3 rgrid((a.T + kRouterRows - 1) / kRouterRows, wave_planes ? 4 * KQ : KQ), rblock(wave_planes ? 64 : 256);
    switch (a.E / 32) {
        case 2: hipLaunchKernelGGL(moe_logits_kernel<2>, rgrid, rblock, wave_planes ? 0 : router_lds, st, a, KQ, (int)wave_planes); break;
        case 4: hipLaunchKernelGGL(moe_logits_kernel<4>, rgrid, rblock, wave_planes ? 0 : router_lds, st, a, KQ, (int)wave_planes); break;
        case 6: hipLaunchKernelGGL(moe_logits_kernel<6>, rgrid, rblock, wave_planes ? 0 : router_lds, st, a, KQ, (int)wave_planes); break;
        case 8: hipLaunchKernelGGL(moe_logits_kernel<8>, rgrid, rblock, wave_planes ? 0 : router_lds, st, a, KQ, (int)wave_planes); break;
        default: return hipErrorInvalidValue;
    }
    if (one_tile) {
        if (wave_planes) hipLaunchKernelGGL(moe_route_tile_kernel<true>, dim3(1), dim3(1024), 0, st, a, 4 * KQ);
        else hipLaunchKernelGGL(moe_route_tile_kernel<false>, dim3(1), dim3(1024), 0, st, a, KQ);
    } else {
        hipLaunchKernelGGL(moe_select_kernel, dim3((a.T + 3) / 4), dim3(256), 0, st, a, KQ);
        hipLaunchKernelGGL(moe_group_kernel, dim3(1), dim3(1024), moe_group_lds_bytes(a.T, a.E), st, a);
        hipLaunchKernelGGL(moe_gather_kernel, dim3(moe_max_tiles(a.T, a.E, a.top_k), 2), dim3(256), 0, st, a);
    }
    // tiles an ordinary expert holds: one if the rows are, two up to 48 rows an expert, else four
    auto products = [&](auto up, auto down) {
        hipLaunchKernelGGL(up, dim3(a.E * (a.F / 64)), dim3(256), 0, st, a, (int)one_tile);
        hipLaunchKernelGGL(down, dim3(a.E * (a.d / 128)), dim3(256), 0, st, a, (int)one_tile);
    };
    if (one_tile) products(moe_gemm_kernel<0, 1>, moe_gemm_kernel<1, 1>);
    else if ((long long)a.T * a.top_k <= 48LL * a.E) products(moe_gemm_kernel<0, 2>, moe_gemm_kernel<1, 2>);
    else products(moe_gemm_kernel<0, 4>, moe_gemm_kernel<1, 4>);
    if (a.out) hipLaunchKernelGGL(moe_combine_kernel, dim3(a.T), dim3(256), 0, st, a);
    return hipGetLastError();
}

}  // namespace sv
