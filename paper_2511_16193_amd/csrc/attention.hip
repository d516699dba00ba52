// Verify attention: the n new rows of every request attend that request's paged KV cache plus the
// new rows they are allowed to see.  Every cached byte is read once per step however many rows
// verify against it -- that reuse across the k+1 rows is the saving of parallel verification -- so
// the kernel is bound by HBM bandwidth and is organised around streaming K/V.
//
// bf16 path (head_dim 128).  A work-group owns one (request, kv head, chunk of keys) and R tiles of 16 of the
// G*n query rows that share the kv head (G = q heads per kv head), stacked.  Each of its waves walks its own
// 32-key tiles of the chunk: K (32 x 128) and V^T (128 x 32) of a tile are stored in the page in MFMA operand
// order, S^T = K Q^T is formed with v_mfma_f32_16x16x32_bf16, the online softmax runs in fp32 on the four keys
// per row each lane holds, and P^T (as two or three bf16 terms) goes back as the B operand of O^T += V^T P^T.  The score
// tile's register layout (a lane holds 4 consecutive keys of one row, for two 16-key blocks) is used unchanged as
// the PV operand; the reduction index of that MFMA is only a label, so V^T is simply stored with the same key
// order.  Waves are merged through LDS, chunks by a second small kernel (split-KV).
// Two kernels: up to 48 stacked rows in one work-group, tiles are prefetched into registers and handled one after
// the other; with more rows, tiles travel through an LDS ring and the three stages of consecutive tiles are woven
// into one instruction stream.
//
// More stacked rows than one work-group takes are split over row groups.  A prefill has hundreds of them per request and
// mostly one piece of keys: its work items are (request, 64 stacked rows, piece), their keys end at the last one the rows
// see, and a request of one piece is finished in the kernel (no partials, no merge).
//
// Generic path (fp32 models, other head sizes, page sizes that are no power of two, steps of more than 256 stacked rows per kv
// head): one work-group per (row, head).
#include <math.h>
#include <algorithm>
#include <type_traits>
#include "common.h"
#include "kernels.h"

namespace sv {

constexpr int HD = 128;
constexpr int TILE_KEYS = 32;

struct KTile { u32x4 k[2][4]; u32x4 v[8]; };
constexpr int kTileBytes = 2 * TILE_KEYS * HD * 2;     // K and V of one 32-key tile: 16 KB
// Largest of the eight scores a lane holds of one row tile, for the kernel whose time is its instruction count (the
// skewed one below).  Written as the instructions themselves: through fmaxf the compiler first passes every score
// through a v_max_f32 x, x, x of its own (it must assume signalling NaNs in what an MFMA returns), eleven
// instructions where four do.
__device__ __forceinline__ float max8(const floatx4& a, const floatx4& b) {
    float r, t;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a[0]), "v"(a[1]), "v"(a[2]));
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(t) : "v"(a[3]), "v"(b[0]), "v"(b[1]));
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(r), "v"(b[2]), "v"(b[3]));
    asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(r), "v"(t));
    return r;
}

// ---- Up to three row tiles in one work-group (at most 48 stacked rows) ----
// Four waves per work-group, one work-group per CU (two with a single row tile); each wave has the next tile's
// loads in flight in a second register set while it works on the current one.  Tile after tile per wave: scores,
// online softmax, PV, not skewed.  At these sizes the kernel runs at the rate the cache can be streamed at, and
// inside a verification step it measured 3-14 % faster than the skewed kernel below (which is ahead once the
// products dominate: four row tiles, or several row groups streaming the same keys).
// ONCE: a tile is read by this work-group only, and from HBM: as a stream (load_stream): 320 rows of 64 requests 131 -> 119 us a layer, 96 requests' single rows
// 164 -> 151, 640 rows beside 8 q heads a kv head 230 -> 210, five rows of one request 13.6 -> 13.0.
template <int R, bool ONCE>
__global__ __launch_bounds__(256, R == 1 ? 2 : 1) void attn_bf16_regs_kernel(AttnArgs a, float scale_log2e) {
    // work item = one piece of one request's keys, cut by the host from its upper bounds of the lengths.
    // Launch order: the kv heads of an item are neighbours, so the list's longest-first order holds chip-wide.
    // With more than 64 stacked rows the row tiles are split over row_groups work-groups that stream the same
    // keys; work-group ids 8 apart run on the same XCD, so the groups of one (item, head) are placed 8 apart
    // and started together: the second reader of a tile finds it in that XCD's L2.
    const int slot = blockIdx.x / (8 * a.row_groups), rem = blockIdx.x % (8 * a.row_groups);
    const int rg = rem >> 3, pair = slot * 8 + (rem & 7);
    const int n_items = a.n_work_dev ? *a.n_work_dev : a.n_work;
    if (pair >= n_items * a.Hkv) return;
    const int hkv = pair % a.Hkv;
    const int4* item = reinterpret_cast<const int4*>(a.work) + 2 * (pair / a.Hkv);
    const int4 keys = item[0], where = item[1];
    const int seq = keys.x, n = keys.w, t0 = where.x;
    const int L = a.seq_len[seq];
    const int total = L + n;
    const int kbeg = keys.y;
    if (kbeg >= total) return;                            // the live length fell short of the host's bound
    const int G = a.Hq / a.Hkv, rows = G * n;
    const int row0 = where.y + rg * R * 16;               // first stacked row of this work-group
    // a prefill item's rows see no further than their last one; a piece beyond that still takes one (masked) tile
    const int kend = a.row_items ? max(kbeg + 1, min(min(keys.z, total), L + (min(row0 + R * 16, rows) - 1) / G + 1)) : min(keys.z, total);

    const int tid = threadIdx.x, lane = tid & 63;
    // wave index as a scalar: tile numbers, page-table reads and page addresses stay on the scalar unit
    // (a vector page-table load would have to be waited for with vmcnt(0), draining the K/V prefetch)
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, lg = lane >> 4;
    const bf16_t* pool = reinterpret_cast<const bf16_t*>(a.pool);
    const int page_shift = 31 - __builtin_clz(a.geom.page_size), page_mask = a.geom.page_size - 1;
    const int32_t* pages = a.page_table + (int64_t)seq * a.max_pages_per_seq;

    // Q^T operand: lane holds row rt*16 + l16, head_dim slice kk*32 + lg*8 .. +8
    u32x4 qf[R][4];
#pragma unroll
    for (int rt = 0; rt < R; ++rt) {
        const int r = row0 + rt * 16 + l16;
        const bool ok = r < rows;
        const int j = ok ? r / G : 0, hl = ok ? r % G : 0;
        const bf16_t* qp = reinterpret_cast<const bf16_t*>(a.q) + ((int64_t)(t0 + j) * a.Hq + hkv * G + hl) * HD;
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
            qf[rt][kk] = ok ? *reinterpret_cast<const u32x4*>(qp + kk * 32 + lg * 8) : u32x4{0, 0, 0, 0};
    }

    // A row sees every cached key, x0 (key L) and the drafts of its own chain up to itself: the keys
    // [vis_lo, vis_hi).  Rows of x0 and padding rows get an empty interval.
    int vis_lo[R], vis_hi[R];
#pragma unroll
    for (int rt = 0; rt < R; ++rt) {
        const int r = row0 + rt * 16 + l16;
        const int j = r < rows ? r / G : 0;
        vis_lo[rt] = j > 0 ? L + 1 + row_chain(j, a.k) * a.k : 0;
        vis_hi[rt] = j > 0 ? vis_lo[rt] + row_index_in_chain(j, a.k) : 0;
    }

    floatx4 o[8][R];
    float m_run[R], mc[R], l_run[R];      // reference maximum (raw score), the same times scale*log2(e), partial sum
#pragma unroll
    for (int rt = 0; rt < R; ++rt) {
        m_run[rt] = -INFINITY;
        mc[rt] = 0.f;
        l_run[rt] = 0.f;
#pragma unroll
        for (int ht = 0; ht < 8; ++ht) o[ht][rt] = floatx4{0.f, 0.f, 0.f, 0.f};
    }

    // The tile's base address is wave-uniform (scalar page number, head, offset): it is kept in scalar registers
    // and every load is "scalar base + lane offset + immediate".  With per-lane 64-bit addresses in vector
    // registers the compiler, short of registers, computed the next tile's address into registers that an
    // in-flight load was still to fill, and had to wait for that load -- and, loads returning in order, for the
    // whole previous tile -- before it could issue the rest: the prefetch never overlapped anything.
    auto uniform = [](int64_t v) {
        const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)v >> 32));
        return (int64_t)(((uint64_t)hi << 32) | lo);
    };
    const int lane_off = lane * 8;
    auto load_tile = [&](int key0, KTile& t) {
        const int page = pages[key0 >> page_shift];
        const int off = key0 & page_mask;
        const int64_t ki = kv_k_index(a.geom, a.layer, page, hkv, off, 0), vi = kv_v_index(a.geom, a.layer, page, hkv, off, 0);
        // one scalar base per 4 KB (the immediate offset of a load reaches 4095 bytes)
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
            const bf16_t* kp = pool + uniform(ki + kb * 2048);
            const bf16_t* vp = pool + uniform(vi + kb * 2048);
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {
                const u32x4 *ks = reinterpret_cast<const u32x4*>(kp + kk * 512 + lane_off), *vs = reinterpret_cast<const u32x4*>(vp + kk * 512 + lane_off);
                t.k[kb][kk] = ONCE ? load_stream(ks) : *ks;
                t.v[kb * 4 + kk] = ONCE ? load_stream(vs) : *vs;
            }
        }
    };

    // One 32-key tile: scores, online softmax, PV.  key0 >= kInvalidKey marks a tile past the end of the
    // chunk (its registers hold a re-load of the last tile): every key is masked and nothing changes.
    constexpr int kInvalidKey = 0x3fffffff;
    auto process = [&](const KTile& t, int key0) {
        // S^T = K Q^T (raw dot products): s[kb][rt][i] <-> key key0 + kb*16 + 4*lg + i, row rt*16 + l16
        floatx4 s[2][R];
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int rt = 0; rt < R; ++rt) {
                floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kk = 0; kk < 4; ++kk)
                    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                        __builtin_bit_cast(bf16x8, t.k[kb][kk]), __builtin_bit_cast(bf16x8, qf[rt][kk]), acc, 0, 0, 0);
                s[kb][rt] = acc;
            }
        if (key0 + TILE_KEYS > L) {   // tile touches the new rows or the end: apply visibility
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int rt = 0; rt < R; ++rt)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int key = key0 + kb * 16 + 4 * lg + i;
                        // bitwise, not short-circuit: this must stay a compare + select chain.  (With
                        // && / || the compiler built branches here and dropped the value of the first
                        // element on the path "beyond L, yet visible".)
                        const bool vis = (key <= L) | ((key >= vis_lo[rt]) & (key < vis_hi[rt]));
                        s[kb][rt][i] = vis ? s[kb][rt][i] : -INFINITY;
                    }
        }
        // Lazy reference maximum.  The softmax reference m_ref of a row is common to the 4 lane groups
        // that share the row (they feed one MFMA accumulator) and is only moved when some score would
        // make 2^(c(s - m_ref)) exceed 2^16 (or on the row's first visible key): fp32 has the range to
        // spare, and the cross-lane reduction + accumulator rescale leave the per-tile path.
        bool trig = false;
        float lmax[R];
#pragma unroll
        for (int rt = 0; rt < R; ++rt) {
            lmax[rt] = fmaxf(fmaxf(fmaxf(s[0][rt][0], s[0][rt][1]), fmaxf(s[0][rt][2], s[0][rt][3])),
                             fmaxf(fmaxf(s[1][rt][0], s[1][rt][1]), fmaxf(s[1][rt][2], s[1][rt][3])));
            trig |= ((m_run[rt] == -INFINITY) & (lmax[rt] > -INFINITY)) | (fmaf(lmax[rt], scale_log2e, -mc[rt]) > 16.0f);
        }
        if (__any(trig)) {
#pragma unroll
            for (int rt = 0; rt < R; ++rt) {
                float mx = lmax[rt];
                mx = fmaxf(mx, __shfl_xor(mx, 16));
                mx = fmaxf(mx, __shfl_xor(mx, 32));
                const float m_new = fmaxf(m_run[rt], mx);
                const float mc_new = m_new == -INFINITY ? 0.f : m_new * scale_log2e;
                const float alpha = m_run[rt] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mc[rt] - mc_new);
                l_run[rt] *= alpha;
#pragma unroll
                for (int ht = 0; ht < 8; ++ht) o[ht][rt] = o[ht][rt] * alpha;
                m_run[rt] = m_new;
                mc[rt] = mc_new;
            }
        }
#pragma unroll
        for (int rt = 0; rt < R; ++rt) {
            floatx2 p[4];
            float psum = 0.f;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                p[i] = floatx2{__builtin_amdgcn_exp2f(fmaf(s[0][rt][2 * i], scale_log2e, -mc[rt])),
                               __builtin_amdgcn_exp2f(fmaf(s[0][rt][2 * i + 1], scale_log2e, -mc[rt]))};
                p[2 + i] = floatx2{__builtin_amdgcn_exp2f(fmaf(s[1][rt][2 * i], scale_log2e, -mc[rt])),
                                   __builtin_amdgcn_exp2f(fmaf(s[1][rt][2 * i + 1], scale_log2e, -mc[rt]))};
                psum += (p[i].x + p[i].y) + (p[2 + i].x + p[2 + i].y);
            }
            l_run[rt] += psum;
            // P goes to the MFMA as three bf16 terms (24 significant bits in all).  One bf16 term would
            // leave a 2^-9 relative error in the output however many keys there are (V has zero mean, so
            // the output is as small as the error's random walk); two terms leave 2^-17, still enough to
            // move every few-hundredth output across a bf16 rounding boundary.
            u32x4 pf[3];
#pragma unroll
            for (int tm = 0; tm < 3; ++tm)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const bf16x2 hb = __builtin_convertvector(p[i], bf16x2);
                    pf[tm][i] = __builtin_bit_cast(uint32_t, hb);
                    if (tm < 2) p[i] = p[i] - __builtin_convertvector(hb, floatx2);
                }
#pragma unroll
            for (int ht = 0; ht < 8; ++ht) {
                const u32x4 vf = t.v[ht];
#pragma unroll
                for (int tm = 2; tm >= 0; --tm)
                    o[ht][rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vf),
                                                                        __builtin_bit_cast(bf16x8, pf[tm]), o[ht][rt], 0, 0, 0);
            }
        }
    };

    // Two tiles per trip, ping-pong between two register sets: while one tile is processed the loads of the next
    // are in flight.  (A third set in flight was measured and does not pay: per tile the wave is bound by its own
    // instruction issue -- 96 MFMAs plus the softmax arithmetic at three row tiles -- not by the load latency.)
    // Loads are unconditional (past the end they re-load the last tile) so that the wait before a tile's math
    // only has to cover that tile's loads and the other set stays in flight.
    const int ntiles = (kend - kbeg + TILE_KEYS - 1) / TILE_KEYS;
    const int last = ntiles - 1;
    auto key_of = [&](int it) { return it < ntiles ? kbeg + it * TILE_KEYS : kInvalidKey; };
    {
        KTile ta, tb;
        load_tile(kbeg + min(wave, last) * TILE_KEYS, ta);
        for (int it = wave; it < ntiles; it += 8) {
            // the fences keep a tile's math (and the waits it starts with) behind the issue of the next tile's loads
            load_tile(kbeg + min(it + 4, last) * TILE_KEYS, tb);
            __builtin_amdgcn_sched_barrier(0);
            process(ta, kbeg + it * TILE_KEYS);
            __builtin_amdgcn_sched_barrier(0);
            load_tile(kbeg + min(it + 8, last) * TILE_KEYS, ta);
            __builtin_amdgcn_sched_barrier(0);
            process(tb, key_of(it + 4));
            __builtin_amdgcn_sched_barrier(0);
        }
    }

    // ---- merge the four waves of the group through LDS (maxima in log2 units from here on) ----
#pragma unroll
    for (int rt = 0; rt < R; ++rt) m_run[rt] = m_run[rt] == -INFINITY ? -INFINITY : mc[rt];
    constexpr int RP = 16 * R;
    __shared__ float m_sh[4][RP], l_sh[4][RP], l_fin[RP];
    extern __shared__ __attribute__((aligned(16))) float o_dyn[];          // [4 waves][HD][RP + 1]
    float (*o_sh)[HD][RP + 1] = reinterpret_cast<float (*)[HD][RP + 1]>(o_dyn);
#pragma unroll
    for (int rt = 0; rt < R; ++rt) {
        float l = l_run[rt];
        l += __shfl_xor(l, 16);
        l += __shfl_xor(l, 32);
        if (lg == 0) {
            m_sh[wave][rt * 16 + l16] = m_run[rt];
            l_sh[wave][rt * 16 + l16] = l;
        }
    }
    __syncthreads();
    float fac[R], m_all[R], l_all[R];
#pragma unroll
    for (int rt = 0; rt < R; ++rt) {
        const int r = rt * 16 + l16;
        float mm = fmaxf(fmaxf(m_sh[0][r], m_sh[1][r]), fmaxf(m_sh[2][r], m_sh[3][r]));
        const float ms = mm == -INFINITY ? 0.f : mm;
        float ll = 0.f;
#pragma unroll
        for (int w = 0; w < 4; ++w) ll += l_sh[w][r] * exp2f(m_sh[w][r] - ms);
        fac[rt] = exp2f(m_run[rt] - ms);
        m_all[rt] = mm;
        l_all[rt] = ll;
        if (wave == 0 && lg == 0) l_fin[r] = ll;
    }
    // every wave lays its rescaled accumulators down in its own LDS plane, all four at once; after one barrier
    // the work-group adds the planes up on the way out (taking turns on a single plane cost four serialised
    // read-modify-write passes, some 10 us per work-group)
#pragma unroll
    for (int rt = 0; rt < R; ++rt)
#pragma unroll
        for (int ht = 0; ht < 8; ++ht)
#pragma unroll
            for (int i = 0; i < 4; ++i) o_sh[wave][ht * 16 + 4 * lg + i][rt * 16 + l16] = o[ht][rt][i] * fac[rt];
    __syncthreads();
    const int rows_here = min(rows - row0, RP);
    if (where.z < 0) {                                    // the request's only piece: the finished rows leave here
        for (int e = tid; e < rows_here * (HD / 4); e += 256) {
            const int r = e / (HD / 4), d = (e % (HD / 4)) * 4;
            float v[4];
#pragma unroll
            for (int i = 0; i < 4; ++i)
                v[i] = ((o_sh[0][d + i][r] + o_sh[1][d + i][r]) + (o_sh[2][d + i][r] + o_sh[3][d + i][r])) / l_fin[r];
            const int g = row0 + r, h = hkv * G + g % G;
            *reinterpret_cast<u32x2*>(reinterpret_cast<bf16_t*>(a.out) + act_index(t0 + g / G, h * HD + d, a.Hq * HD, a.out_packed)) =
                u32x2{pack2bf(v[0], v[1]), pack2bf(v[2], v[3])};
        }
        return;
    }
    const int64_t pbase = (int64_t)where.z + (int64_t)hkv * where.w + row0;
    for (int e = tid; e < rows_here * HD; e += 256) {
        const int r = e / HD, d = e % HD;
        a.part_o[(pbase + r) * HD + d] = (o_sh[0][d][r] + o_sh[1][d][r]) + (o_sh[2][d][r] + o_sh[3][d][r]);
    }
    if (wave == 0 && lg == 0) {
#pragma unroll
        for (int rt = 0; rt < R; ++rt) {
            const int r = rt * 16 + l16;
            if (r < rows_here) {
                a.part_ml[(pbase + r) * 2] = m_all[rt];
                a.part_ml[(pbase + r) * 2 + 1] = l_all[rt];
            }
        }
    }
}

// R row tiles per work-group, W waves, two slots per wave for K and for V in the LDS ring (W * 32 KB of LDS).
// Run as W = 2, two work-groups to a CU, and in a small prefill as W = 4.
// ONCE: no other row group or item reads these keys, and they come from HBM: as a stream (load_stream; 63 rows of 256 requests 497 -> 445 us; with a second
// row group to find them in L2 685 -> 703).
// PT: bf16 terms the softmax weights are split into for the PV products.  With four row tiles (or several row
// groups) this kernel is bound by its matrix products and the power they draw, and three quarters of them are PV
// products: it runs with PT = 2 (16 significant bits; the 2^-17 relative it leaves is the size of the fp32
// accumulation error of a few thousand keys, i.e. nothing the result did not carry already), a quarter fewer
// products than with three terms.  The register kernel above is bound by the stream and keeps three.  So does a prefill, whose
// rows become the cache that every later step reads: with two terms 1.3 in a thousand outputs are rounded to another bf16
// value than the exact sums', with three 0.03 to 0.4; 24 prompts of 100-500 tokens 24.56 -> 24.54 ms, one of 777 4.37 -> 4.39.
template <int R, int W, int PT, bool ONCE = false>
__global__ __launch_bounds__(64 * W, 1) void attn_bf16_kernel(AttnArgs a, float scale_log2e) {
    // Work item = one piece of one request's keys, cut by the host from its upper bounds of the lengths.
    // Launch order: the kv heads of an item are neighbours, so the list's longest-first order holds chip-wide.
    // With more stacked rows than one work-group takes, the row tiles are split over row_groups work-groups that
    // stream the same keys; work-group ids 8 apart run on the same XCD, so the groups of one (item, head) are
    // placed 8 apart and started together: the second reader of a tile finds it in that XCD's L2.
    // A work-group is W waves, each alone on its SIMD (the accumulators leave no room for a second), and takes
    // half of the CU's LDS: two work-groups share a CU, so that while one starts an item (three dependent reads:
    // item, page table, first tile) or merges its waves, the other keeps streaming.
    constexpr int RP = 16 * R;
    __shared__ float m_sh[W][RP], l_sh[W][RP], l_fin[RP];
    const int slot_id = blockIdx.x / (8 * a.row_groups), rem = blockIdx.x % (8 * a.row_groups);
    const int rg = rem >> 3, pair = slot_id * 8 + (rem & 7);
    const int n_items = a.n_work_dev ? *a.n_work_dev : a.n_work;
    if (pair >= n_items * a.Hkv) return;
    const int hkv = pair % a.Hkv;
    const int4* item = reinterpret_cast<const int4*>(a.work) + 2 * (pair / a.Hkv);
    const int4 keys = item[0], where = item[1];
    const int seq = keys.x, n = keys.w, t0 = where.x;
    const int L = a.seq_len[seq];
    const int total = L + n;
    const int kbeg = keys.y;
    if (kbeg >= total) return;                            // the live length fell short of the host's bound
    const int G = a.Hq / a.Hkv, rows = G * n;
    const int row0 = where.y + rg * R * 16;               // first stacked row of this work-group
    // a prefill item's rows see no further than their last one; a piece beyond that still takes one (masked) tile
    const int kend = a.row_items ? max(kbeg + 1, min(min(keys.z, total), L + (min(row0 + R * 16, rows) - 1) / G + 1)) : min(keys.z, total);

    const int tid = threadIdx.x, lane = tid & 63;
    // wave index as a scalar: tile numbers, page-table reads and page addresses stay on the scalar unit
    // (a vector page-table load would have to be waited for with vmcnt(0), draining the K/V prefetch)
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, lg = lane >> 4;
    const bf16_t* pool = reinterpret_cast<const bf16_t*>(a.pool);
    const int page_shift = 31 - __builtin_clz(a.geom.page_size), page_mask = a.geom.page_size - 1;
    // The page table is read through the constant address space: nothing writes it while the kernel runs, and
    // only so do the lookups stay scalar loads once the loop holds direct-to-LDS loads (which the compiler must
    // otherwise assume may alias any global read; a vector lookup would be waited for with vmcnt(0), draining
    // the K/V prefetch).
    typedef const __attribute__((address_space(4))) int32_t* const_i32_ptr;
    const_i32_ptr pages = (const_i32_ptr)(a.page_table + (int64_t)seq * a.max_pages_per_seq);

    // Q^T operand: lane holds row rt*16 + l16, head_dim slice kk*32 + lg*8 .. +8
    u32x4 qf[R][4];
#pragma unroll
    for (int rt = 0; rt < R; ++rt) {
        const int r = row0 + rt * 16 + l16;
        const bool ok = r < rows;
        const int j = ok ? r / G : 0, hl = ok ? r % G : 0;
        const bf16_t* qp = reinterpret_cast<const bf16_t*>(a.q) + ((int64_t)(t0 + j) * a.Hq + hkv * G + hl) * HD;
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
            qf[rt][kk] = ok ? *reinterpret_cast<const u32x4*>(qp + kk * 32 + lg * 8) : u32x4{0, 0, 0, 0};
    }

    // A row sees every cached key, x0 (key L) and the drafts of its own chain up to itself: the keys
    // [vis_lo, vis_hi).  Rows of x0 and padding rows get an empty interval.
    int vis_lo[R], vis_hi[R];
#pragma unroll
    for (int rt = 0; rt < R; ++rt) {
        const int r = row0 + rt * 16 + l16;
        const int j = r < rows ? r / G : 0;
        vis_lo[rt] = j > 0 ? L + 1 + row_chain(j, a.k) * a.k : 0;
        vis_hi[rt] = j > 0 ? vis_lo[rt] + row_index_in_chain(j, a.k) : 0;
    }

    floatx4 o[8][R];
    // reference (log2 units), partial sum, and the raw score above which the reference moves: -inf until the row has seen a key
    float mc[R], l_run[R], limit[R];
    const float unscale = 1.0f / scale_log2e;
#pragma unroll
    for (int rt = 0; rt < R; ++rt) {
        mc[rt] = 0.f;
        l_run[rt] = 0.f;
        limit[rt] = -INFINITY;
#pragma unroll
        for (int ht = 0; ht < 8; ++ht) o[ht][rt] = floatx4{0.f, 0.f, 0.f, 0.f};
    }

    // K/V tiles travel HBM -> LDS -> registers.  Each wave owns a ring of two slots for K and two for V (8 KB each)
    // in LDS that it fills with direct-to-LDS loads (16 bytes per lane, 1 KB per instruction, no registers held
    // while in flight) and reads back into one register set.  A wave reads only what it loaded itself: no barriers.
    // The tile's base address is wave-uniform (scalar page number, head, offset) and kept in scalar registers.
    auto uniform = [](int64_t v) {
        const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)v >> 32));
        return (int64_t)(((uint64_t)hi << 32) | lo);
    };
    extern __shared__ __attribute__((aligned(16))) unsigned char attn_lds[];
    // Tiles start on multiples of 32 keys, where the cache's index functions reduce to
    //   K: layer * layer_elems + page * page_elems + (head * page_size + key_in_page) * 128,   V: the same + v_off
    // (kv_k_index / kv_v_index with tok % 32 == 0, dim == 0); K and V of a tile are 8 KB each, contiguous, and are
    // copied verbatim.
    const char* head_base = reinterpret_cast<const char*>(pool + ((int64_t)a.layer * a.geom.layer_elems + (int64_t)hkv * a.geom.page_size * HD));
    const int64_t v_off = (int64_t)a.geom.n_kv_heads * a.geom.page_size * HD * 2;
    const uint32_t lane_bytes = lane * 16;
    // Ring layout per wave: K slots 0, 1, then V slots 0, 1 (8 KB each).
    const uint32_t ring = (uint32_t)(uintptr_t)SV_LDS_PTR(attn_lds) + wave * (2 * kTileBytes), ring_lane = ring + lane_bytes;
    // KB `piece` of the eight of a tile's K (or V) into the ring slot at `dst`, in order: 0 and 4 set what the next three go by
    auto request = [&](const char* src, uint32_t dst, auto piece) __attribute__((always_inline)) {
        constexpr int F = decltype(piece)::value;
        dma_piece<F % 4, ONCE>(src + F / 4 * 4096, lane_bytes, dst + F / 4 * 4096);
    };

    // Wave w takes tiles w, w + W, ... of the piece: its tile t starts at key tile_key(t).
    const int ntiles = (kend - kbeg + TILE_KEYS - 1) / TILE_KEYS;
    const int last = ntiles - 1;
    const int n_my = wave < ntiles ? (ntiles - wave + W - 1) / W : 0;
    auto tile_key = [&](int t) { return kbeg + min(wave + W * t, last) * TILE_KEYS; };   // past the end: a valid tile
    auto page_of = [&](int t) { return pages[tile_key(t) >> page_shift]; };
    auto k_of = [&](int t, int page) { return head_base + uniform(((int64_t)page * a.geom.page_elems + (tile_key(t) & page_mask) * HD) * 2); };

    // The three stages of a tile -- scores S^T = K Q^T (MFMA), softmax (vector ALU), O^T += V^T P^T (MFMA) -- depend
    // on each other, and a wave alone on its SIMD issues one instruction at a time: done tile after tile, the
    // matrix unit idles through the softmax and the vector ALU through the products.  So the loop is skewed: trip j adds the PV
    // products of tile j - 1 and forms the scores of tile j + 1, with the softmax of tile j woven in, a few vector instructions behind
    // each product.  The softmax follows one row tile behind the products that read the terms of P it writes, and is ahead of
    // the products that write the scores it reads, so one set of registers holds each of them and nothing is copied.
    // K and V of a tile are read from the ring while the other one is multiplied (K of tile j + 1 beside the PV products, V of
    // tile j beside the scores); a slot is requested again as soon as it has been read (K of tile j + 3, V of tile j + 2), a KB at a time
    // between the products.  Each half starts with everything landed but the newest 24 requests.
    // The last trip forms no scores and requests nothing more (with 63 to 125 rows of 256 requests behind 60 to 200 keys, two to four tiles a wave, that is
    // 1 to 3 % of the launch).
    // The page of a tile is looked up a trip before its K is requested; V lies a fixed distance behind K.
    // Two products in a row add to the same accumulators (the terms of P, the slices of the head dimension): the chip's power is what a long run of
    // this kernel is bound by, and such pairs draw less of it (a loop of products alone sustains 2.13 PFLOP/s, 2.01 with other accumulators every
    // time); with the terms outermost the loop takes 3 % fewer cycles and a step 3 % longer.
    // 32 requests of 16k-32k keys, 125 stacked rows, us a layer: woven by the compiler from three parts with two sets of scores, all requests at the
    // head of a trip 693, so 658; million cycles summed over the dies 10.2 and 9.8; the step of eight layers 1.5 to 2 % shorter.
    floatx4 s[2][R];                                      // [key block][row tile]
    u32x4 pf[R][PT];                                      // P^T as bf16 terms
    u32x4 kreg[2][4], vreg[8];
    float lmax[R];
    const char *k2 = k_of(1, page_of(1)), *k3 = k_of(2, page_of(2));     // K of tiles j + 2, j + 3 (j = -1)
    int page4 = page_of(3);                               // page of tile j + 4
    uint32_t odd = 0;                                     // 8192 x parity of tile j + 1: where its K lies, and V of tile j - 1
    auto fence = []() __attribute__((always_inline)) { __builtin_amdgcn_sched_barrier(0); };
    auto read_k = [&](uint32_t addr, auto piece) __attribute__((always_inline)) {
        constexpr int F = decltype(piece)::value;
        lds_read16<F * 1024>(kreg[F >> 2][F & 3], addr);
    };
    auto read_v = [&](uint32_t addr, auto piece) __attribute__((always_inline)) {
        constexpr int F = decltype(piece)::value;
        lds_read16<2 * 8192 + F * 1024>(vreg[F], addr);
    };
    auto wait_k = [&]() __attribute__((always_inline)) {
        lds_landed(kreg[0][0]);
#pragma unroll
        for (int f = 1; f < 8; ++f) lds_landed_too(kreg[f >> 2][f & 3]);
    };
    auto wait_v = [&]() __attribute__((always_inline)) {
        lds_landed(vreg[0]);
#pragma unroll
        for (int f = 1; f < 8; ++f) lds_landed_too(vreg[f]);
    };
    // Step `step` of the softmax of row tile rt: two keys of each of its rows take 2 PT steps.
    // P goes to the MFMA as PT bf16 terms (8 significant bits each).  One term would leave a 2^-9
    // relative error in the output however many keys there are (V has zero mean, so the output is
    // as small as the error's random walk): as much as the rounding of the output itself.
    float e0, e1, sum_a, sum_b;
    uint32_t high;
    auto soft = [&](auto row, auto which) __attribute__((always_inline)) {
        constexpr int rt = decltype(row)::value, step = decltype(which)::value % (2 * PT), q = decltype(which)::value / (2 * PT);
        constexpr int i = (q & 1) * 2 + (q >> 1), t = step / 2 - 1;      // pairs of keys 0, 2, 1, 3; steps 2, 3: term 0; 4, 5: term 1
        if constexpr (step == 0) {
            e0 = fmaf(s[i >> 1][rt][2 * (i & 1)], scale_log2e, -mc[rt]);
            e1 = fmaf(s[i >> 1][rt][2 * (i & 1) + 1], scale_log2e, -mc[rt]);
        } else if constexpr (step == 1) {
            e0 = __builtin_amdgcn_exp2f(e0);
            e1 = __builtin_amdgcn_exp2f(e1);
        } else if constexpr (step % 2 == 0) {
            if constexpr (step == 2) {
                if constexpr (q == 0) sum_a = e0 + e1;
                else if constexpr (q == 1) sum_a += e0 + e1;
                else if constexpr (q == 2) sum_b = e0 + e1;
                else l_run[rt] += sum_a + (sum_b + (e0 + e1));
            }
            high = pack2bf(e0, e1);
            pf[rt][t][i] = high;
        } else {
            e0 -= __uint_as_float(high << 16);
            e1 -= __uint_as_float(high & 0xffff0000u);
            if constexpr (t == PT - 2) pf[rt][PT - 1][i] = pack2bf(e0, e1);
        }
    };
    constexpr int kSteps = 8 * PT;                        // steps of a row tile's softmax, and its PV products
    constexpr int GS = R == 2 ? 1 : 2;                    // row tiles whose scores are formed together
    // of tile j + 1; softmax of the last row tile of tile j.  LAST: there is no tile j + 1
    auto scores = [&](auto soft_c, auto read_c, auto last_c) __attribute__((always_inline)) {
        constexpr bool LAST = decltype(last_c)::value;
        constexpr int NM = 8 * R, AHEAD = 8 * GS * ((R - 1) / GS), EACH = (kSteps + AHEAD - 1) / AHEAD;      // products before the last row tile's scores are written
        static_for<NM>([&](auto mi) __attribute__((always_inline)) {
            constexpr int m = decltype(mi)::value, grp = m / (8 * GS), x = m - grp * 8 * GS;
            constexpr int kk = x % 4, kb = x / 4 % 2, rt = grp * GS + x / 8;
            const floatx4 zero = {0.f, 0.f, 0.f, 0.f};
            if constexpr (!LAST)
                s[kb][rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kreg[kb][kk]), __builtin_bit_cast(bf16x8, qf[rt][kk]),
                                                                    kk == 0 ? zero : s[kb][rt], 0, 0, 0);
            fence();
            if constexpr (decltype(soft_c)::value)
                static_for<EACH>([&](auto u) __attribute__((always_inline)) {
                    constexpr int st = m * EACH + decltype(u)::value;
                    if constexpr (st < kSteps) { soft(std::integral_constant<int, R - 1>{}, std::integral_constant<int, st>{}); fence(); }
                });
            if constexpr (decltype(read_c)::value && m < 8) { read_v(ring_lane + (odd ^ 8192), mi); fence(); }
            if constexpr (decltype(read_c)::value && m == NM / 2 - 1) wait_v();
            if constexpr (!LAST && m >= NM / 2 && m % (NM / 16) == 0 && (m - NM / 2) / (NM / 16) < 8) {
                request(k2 + v_off, ring + 2 * 8192 + (odd ^ 8192), std::integral_constant<int, (m - NM / 2) / (NM / 16)>{});
                fence();
            }
        });
        if constexpr (!LAST)
#pragma unroll
            for (int rt = 0; rt < R; ++rt)                // into ordinary registers: arithmetic cannot read the accumulation ones
                asm volatile("" : "+v"(s[0][rt]), "+v"(s[1][rt]));
    };
    auto products = [&](auto row, auto with) __attribute__((always_inline)) {          // PV products of a row tile, with(product) behind each
        constexpr int rt = decltype(row)::value;
        static_for<kSteps>([&](auto mi) __attribute__((always_inline)) {
            constexpr int m = decltype(mi)::value, tm = PT - 1 - m % PT, ht = m / PT;
            o[ht][rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vreg[ht]), __builtin_bit_cast(bf16x8, pf[rt][tm]),
                                                                o[ht][rt], 0, 0, 0);
            fence();
            with(mi);
        });
    };
    auto nothing = [](auto) __attribute__((always_inline)) {};
    const std::integral_constant<int, 0> i0;

    auto trip = [&](auto pv_c, auto last_c, int j) __attribute__((always_inline)) {
        constexpr bool PV = decltype(pv_c)::value, LAST = decltype(last_c)::value;
        if constexpr (!LAST) wait_vmcnt<24>();
        const int key0 = kbeg + (wave + W * j) * TILE_KEYS;
        if (key0 + TILE_KEYS > L) {   // tile touches the new rows or the end: apply visibility
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int rt = 0; rt < R; ++rt)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int key = key0 + kb * 16 + 4 * lg + i;
                        // bitwise, not short-circuit: this must stay a compare + select chain.  (With
                        // && / || the compiler built branches here and dropped the value of the first
                        // element on the path "beyond L, yet visible".)
                        const bool vis = (key <= L) | ((key >= vis_lo[rt]) & (key < vis_hi[rt]));
                        s[kb][rt][i] = vis ? s[kb][rt][i] : -INFINITY;
                    }
        }
        // Lazy reference maximum.  The softmax reference m_ref of a row is common to the 4 lane groups
        // that share the row (they feed one MFMA accumulator) and is only moved when some score would
        // make 2^(c(s - m_ref)) exceed 2^16 (or on the row's first visible key): fp32 has the range to
        // spare, and the cross-lane reduction + accumulator rescale leave the per-tile path.
        // One comparison with that score a row (it took four vector instructions; 280 -> 260 a tile besides the products): 125 stacked rows
        // of 16k-32k keys 692 -> 682 and 689 -> 671 us a layer, 63 rows 515 -> 512.  (In the register kernel, bound by the stream: no change.)
        bool trig = false;
        fence();
        auto first = [&](auto mi) __attribute__((always_inline)) {
            constexpr int m = decltype(mi)::value;
            if constexpr (m < 8) {
                if constexpr (!LAST) { read_k(ring_lane + odd, mi); fence(); }
            } else if constexpr (m < 8 + R) {
                lmax[m - 8] = max8(s[0][m - 8], s[1][m - 8]);
                trig |= lmax[m - 8] > limit[m - 8];
                fence();
            }
        };
        if constexpr (PV) products(i0, first);
        else static_for<kSteps>(first);
        if constexpr (!LAST) wait_k();
        if (__builtin_expect(__any(trig), 0)) {
            // Move the reference.  It is kept at a whole number of log2 units, so the factor between the old and
            // the new one is a power of two: what was accumulated against the old reference (the sums, the
            // accumulators, and the bf16 terms of P^T whose PV products are still pending) is rescaled exactly.
#pragma unroll
            for (int rt = 0; rt < R; ++rt) {
                float mx = lmax[rt];
                mx = fmaxf(mx, __shfl_xor(mx, 16));
                mx = fmaxf(mx, __shfl_xor(mx, 32));
                const bool seen = limit[rt] > -INFINITY, some = mx > -INFINITY;
                const float to = ceilf(mx * scale_log2e), mc_new = !some ? mc[rt] : seen ? fmaxf(mc[rt], to) : to;
                const int shift = (int)fmaxf(mc[rt] - mc_new, -200.f);
                const float alpha = seen ? ldexpf(1.0f, shift) : 0.f;
                l_run[rt] *= alpha;
#pragma unroll
                for (int ht = 0; ht < 8; ++ht) {
                    // The accumulators live in the accumulation registers, which arithmetic cannot read.  The empty
                    // statement pins their copy to ordinary registers here, on the rare path (the compiler otherwise
                    // makes those 32 R copies at the head of every trip of the loop, needed or not).
                    floatx4 t = o[ht][rt];
                    asm volatile("" : "+v"(t));
                    o[ht][rt] = t * alpha;
                }
                if (PV && rt > 0) {
#pragma unroll
                    for (int tm = 0; tm < PT; ++tm)
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const uint32_t w = pf[rt][tm][i];
                            const float lo = __builtin_bit_cast(float, w << 16) * alpha;
                            const float hi = __builtin_bit_cast(float, w & 0xffff0000u) * alpha;
                            pf[rt][tm][i] = (__builtin_bit_cast(uint32_t, lo) >> 16) | (__builtin_bit_cast(uint32_t, hi) & 0xffff0000u);
                        }
                }
                mc[rt] = mc_new;
                limit[rt] = (seen | some) ? (mc_new + 16.0f) * unscale : -INFINITY;
            }
        }
        fence();
        static_for<R - 1>([&](auto prev) __attribute__((always_inline)) {
            constexpr int rt = decltype(prev)::value + 1, N = kSteps * (R - 1);
            auto behind = [&](auto mi) __attribute__((always_inline)) {
                constexpr int m = decltype(mi)::value, at = kSteps * (rt - 1) + m;
                soft(prev, mi);
                fence();
                if constexpr (!LAST && at % (N / 8) == N / 8 - 1 && at / (N / 8) < 8) {
                    request(k3, ring + odd, std::integral_constant<int, at / (N / 8)>{});
                    fence();
                }
            };
            if constexpr (PV) products(std::integral_constant<int, rt>{}, behind);
            else static_for<kSteps>(behind);
        });
        wait_vmcnt<LAST ? 16 : 24>();
        fence();
        scores(std::true_type{}, std::true_type{}, last_c);
        if constexpr (LAST) return;
        odd ^= 8192;
        k2 = k3;
        k3 = k_of(j + 4, page4);
        page4 = page_of(j + 5);
        fence();
    };
    if (n_my > 0) {
        const char* k1 = k_of(0, page_of(0));
        static_for<8>([&](auto f) __attribute__((always_inline)) { request(k1, ring, f); });
        static_for<8>([&](auto f) __attribute__((always_inline)) { request(k2, ring + 8192, f); });
        static_for<8>([&](auto f) __attribute__((always_inline)) { request(k1 + v_off, ring + 2 * 8192, f); });
        wait_vmcnt<16>();
        fence();
        static_for<8>([&](auto f) __attribute__((always_inline)) { read_k(ring_lane, f); });
        wait_k();
        fence();
        static_for<8>([&](auto f) __attribute__((always_inline)) { request(k3, ring, f); });
        scores(std::false_type{}, std::false_type{}, std::false_type{});
        odd = 8192;
        k2 = k3;
        k3 = k_of(3, page4);
        page4 = page_of(4);
        fence();
        if (n_my == 1) {
            trip(std::false_type{}, std::true_type{}, 0);
        } else {
            trip(std::false_type{}, std::false_type{}, 0);
            for (int j = 1; j < n_my - 1; ++j) trip(std::true_type{}, std::false_type{}, j);
            trip(std::true_type{}, std::true_type{}, n_my - 1);
        }
        static_for<R>([&](auto rt) __attribute__((always_inline)) { products(rt, nothing); });
    }
    wait_vmcnt<0>();                                      // the ring is about to be reused for the merge

    // ---- merge the waves of the group through LDS (maxima in log2 units from here on) ----
    float m_run[R];
#pragma unroll
    for (int rt = 0; rt < R; ++rt) m_run[rt] = limit[rt] > -INFINITY ? mc[rt] : -INFINITY;
    float (*o_sh)[HD][RP + 1] = reinterpret_cast<float (*)[HD][RP + 1]>(attn_lds);   // [W waves][HD][RP + 1], over the rings
#pragma unroll
    for (int rt = 0; rt < R; ++rt) {
        float l = l_run[rt];
        l += __shfl_xor(l, 16);
        l += __shfl_xor(l, 32);
        if (lg == 0) {
            m_sh[wave][rt * 16 + l16] = m_run[rt];
            l_sh[wave][rt * 16 + l16] = l;
        }
    }
    __syncthreads();
    float fac[R], m_all[R], l_all[R];
#pragma unroll
    for (int rt = 0; rt < R; ++rt) {
        const int r = rt * 16 + l16;
        float mm = m_sh[0][r];
#pragma unroll
        for (int w = 1; w < W; ++w) mm = fmaxf(mm, m_sh[w][r]);
        const float ms = mm == -INFINITY ? 0.f : mm;
        float ll = 0.f;
#pragma unroll
        for (int w = 0; w < W; ++w) ll += l_sh[w][r] * exp2f(m_sh[w][r] - ms);
        fac[rt] = exp2f(m_run[rt] - ms);
        m_all[rt] = mm;
        l_all[rt] = ll;
        if (wave == 0 && lg == 0) l_fin[r] = ll;
    }
    // every wave lays its rescaled accumulators down in its own LDS plane, all four at once; after one barrier
    // the work-group adds the planes up on the way out (taking turns on a single plane cost four serialised
    // read-modify-write passes, some 10 us per work-group)
#pragma unroll
    for (int rt = 0; rt < R; ++rt)
#pragma unroll
        for (int ht = 0; ht < 8; ++ht)
#pragma unroll
            for (int i = 0; i < 4; ++i) o_sh[wave][ht * 16 + 4 * lg + i][rt * 16 + l16] = o[ht][rt][i] * fac[rt];
    __syncthreads();
    const int rows_here = min(rows - row0, RP);
    if (where.z < 0) {                                    // the request's only piece: the finished rows leave here
        for (int e = tid; e < rows_here * (HD / 4); e += 64 * W) {
            const int r = e / (HD / 4), d = (e % (HD / 4)) * 4;
            float v[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                v[i] = o_sh[0][d + i][r];
#pragma unroll
                for (int w = 1; w < W; ++w) v[i] += o_sh[w][d + i][r];
                v[i] /= l_fin[r];
            }
            const int g = row0 + r, h = hkv * G + g % G;
            *reinterpret_cast<u32x2*>(reinterpret_cast<bf16_t*>(a.out) + act_index(t0 + g / G, h * HD + d, a.Hq * HD, a.out_packed)) =
                u32x2{pack2bf(v[0], v[1]), pack2bf(v[2], v[3])};
        }
        return;
    }
    const int64_t pbase = (int64_t)where.z + (int64_t)hkv * where.w + row0;
    for (int e = tid; e < rows_here * HD; e += 64 * W) {
        const int r = e / HD, d = e % HD;
        float acc = o_sh[0][d][r];
#pragma unroll
        for (int w = 1; w < W; ++w) acc += o_sh[w][d][r];
        a.part_o[(pbase + r) * HD + d] = acc;
    }
    if (wave == 0 && lg == 0) {
#pragma unroll
        for (int rt = 0; rt < R; ++rt) {
            const int r = rt * 16 + l16;
            if (r < rows_here) {
                a.part_ml[(pbase + r) * 2] = m_all[rt];
                a.part_ml[(pbase + r) * 2 + 1] = l_all[rt];
            }
        }
    }
}

// Combine the chunk partials of one row: out = sum_c 2^(m_c - M) O_c / sum_c 2^(m_c - M) l_c.  A thread
// owns four consecutive dimensions of one q head; a work-group covers 256 / 32 = 8 heads of the row.  The 32 threads of a
// head take one piece's (m, l) each, all at once, and share the factors; eight pieces' O are in flight at a time.  Rows that
// follow each other go to one XCD (their packed output shares cache lines): 320 / 800 rows 6.9 / 19.3 -> 5.8 / 16.0 us.
__global__ __launch_bounds__(256) void attn_merge_kernel(AttnArgs a) {
    const int t_out = xcd_remap(blockIdx.x, gridDim.x), h = blockIdx.y * 8 + (threadIdx.x >> 5), lane = threadIdx.x & 31, d = lane * 4;
    if (h >= a.Hq) return;                                // (whole groups of 32)
    const int t = a.last_of ? a.last_of[t_out * kReqInts] + a.last_of[t_out * kReqInts + 1] - 1 : t_out;
    bf16_t* dst = reinterpret_cast<bf16_t*>(a.last_of ? a.last_out : a.out) + act_index(t_out, h * HD + d, a.Hq * HD, a.out_packed);
    const int4 pt = reinterpret_cast<const int4*>(a.row_part)[t];
    const int nch = pt.w;                                 // 0: a request of one piece, already written
    if (nch == 0) {
        if (a.last_of) *reinterpret_cast<u32x2*>(dst) = *reinterpret_cast<const u32x2*>(reinterpret_cast<const bf16_t*>(a.out) + act_index(t, h * HD + d, a.Hq * HD, a.out_packed));
        return;
    }
    const int G = a.Hq / a.Hkv, hkv = h / G;
    const int64_t base = (int64_t)pt.x + (int64_t)hkv * pt.y + h % G;
    const floatx2* ml = reinterpret_cast<const floatx2*>(a.part_ml) + base;
    float M = -INFINITY;
    for (int c = lane; c < nch; c += 32) M = fmaxf(M, ml[(int64_t)c * pt.z].x);
#pragma unroll
    for (int o = 16; o > 0; o >>= 1) M = fmaxf(M, __shfl_xor(M, o, 32));
    floatx4 num = {0.f, 0.f, 0.f, 0.f};
    float den = 0.f;
    for (int c0 = 0; c0 < nch; c0 += 32) {
        const floatx2 x = c0 + lane < nch ? ml[(int64_t)(c0 + lane) * pt.z] : floatx2{-INFINITY, 0.f};
        const float f = exp2f(x.x - M);
        den += f * x.y;
        for (int c = c0; c < min(nch, c0 + 32); c += 8) {
            floatx4 o[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) o[u] = *reinterpret_cast<const floatx4*>(a.part_o + (base + (int64_t)min(c + u, nch - 1) * pt.z) * HD + d);
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const float fu = __shfl(f, (c + u) & 31, 32);             // pieces past the end: factor 0
                num[0] += fu * o[u][0]; num[1] += fu * o[u][1]; num[2] += fu * o[u][2]; num[3] += fu * o[u][3];
            }
        }
    }
#pragma unroll
    for (int o = 16; o > 0; o >>= 1) den += __shfl_xor(den, o, 32);
    // four consecutive dimensions stay inside one 8-element piece of either output order
    u32x2 pk = {pack2bf(num[0] / den, num[1] / den), pack2bf(num[2] / den, num[3] / den)};
    *reinterpret_cast<u32x2*>(dst) = pk;
}

// Generic path: one work-group of four waves per (new row, q head), keys in chunks of 256.  Scores with a thread per
// key (eight consecutive dimensions of a key are one contiguous piece), softmax weights in LDS, then a thread per
// (dimension, share of the chunk's tiles): the cache keeps eight keys of a dimension side by side, so V comes in whole
// pieces too.  fp32 throughout, online softmax from chunk to chunk.  A key that the row does not see takes no part at all:
// its weight is marked below zero and its V, which may hold anything, is not multiplied; only tiles that hold such keys are
// looked at for it (in all of them it cost 4 to 8 %; so, the fp32 prefill 1 % and the steps nothing).  (With a lane per key
// holding all D accumulators, V element by element and D wave reductions at the end, the step of 20 rows with 132 keys took 43 us
// a layer; 6.2 us now.)  A row's cached length comes with its other descriptions, one read less in the chain that a small step's launch
// consists of.  (The chunk's first tile of V requested before the softmax saves another, 1 to 3 % of a step of few rows with 64 fp32 dimensions, but
// costs many rows 3 to 4 % -- two layers of 12 heads, 99 / 288 rows of 4200 / 1500 keys 574 / 964 -> 599 / 993 us a step --, 128 dimensions up to 20 % and bf16 5 %.)
template <typename T, int D>
__global__ __launch_bounds__(256) void attn_generic_kernel(AttnArgs a, float scale) {
    constexpr int CK = 256, GROUPS = 256 / D, EP = 16 / (int)sizeof(T);
    const int t_out = blockIdx.x, t = a.last_of ? a.last_of[t_out * kReqInts] + a.last_of[t_out * kReqInts + 1] - 1 : t_out, h = blockIdx.y, tid = threadIdx.x;
    const int4 info = reinterpret_cast<const int4*>(a.row_info)[t];
    const int seq = info.x, j = info.y;
    const int L = info.w, total = L + info.z;
    const int end = a.row_items ? L + j + 1 : total;      // a prefill row sees nothing beyond itself
    const int all_seen = a.row_items ? end : L;           // up to here it sees every key
    const int hkv = h / (a.Hq / a.Hkv);
    const int32_t* pages = a.page_table + (int64_t)seq * a.max_pages_per_seq;
    const T* pool = reinterpret_cast<const T*>(a.pool);
    __shared__ __attribute__((aligned(16))) float q[D];
    __shared__ __attribute__((aligned(16))) float p[CK];
    __shared__ float red[4], acc_sh[GROUPS][D];
    for (int d = tid; d < D; d += 256) q[d] = Store<T>::load(reinterpret_cast<const T*>(a.q) + ((int64_t)t * a.Hq + h) * D + d);
    __syncthreads();
    auto load8 = [](const T* src, float* dst) {            // eight elements, 16-byte aligned
#pragma unroll
        for (int u = 0; u < 8 / EP; ++u) {
            const u32x4 w = *reinterpret_cast<const u32x4*>(src + u * EP);
#pragma unroll
            for (int e = 0; e < EP; ++e)
                dst[u * EP + e] = EP == 4 ? __uint_as_float(w[e]) : __uint_as_float((e & 1) ? (w[e >> 1] & 0xffff0000u) : (w[e >> 1] << 16));
        }
    };
    const int dim = tid % D, grp = tid / D;
    float m = -INFINITY, l = 0.f, acc = 0.f;
    for (int c0 = 0; c0 < end; c0 += CK) {
        const int key = c0 + tid;
        float s = -INFINITY;
        const bool seen = key < end && (key < L || row_sees(j, key - L, a.k));
        if (seen) {
            const T* kp = pool + kv_k_index(a.geom, a.layer, pages[key / a.geom.page_size], hkv, key % a.geom.page_size, 0);
            s = 0.f;
#pragma unroll
            for (int c = 0; c < D / 8; ++c) {               // dims 8 c ..: slice c / 4 of 32 dims, lane group c % 4 (16 keys of 8 each)
                float kv[8];
                load8(kp + ((c >> 2) * 64 + (c & 3) * 16) * 8, kv);
#pragma unroll
                for (int e = 0; e < 8; ++e) s = fmaf(q[8 * c + e], kv[e], s);
            }
            s *= scale;
        }
        const float mw = wave_max(s);
        if ((tid & 63) == 0) red[tid >> 6] = mw;
        __syncthreads();
        const float m_new = fmaxf(m, fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3])));
        const float ms = m_new == -INFINITY ? 0.f : m_new;
        const float pv = seen ? expf(s - ms) : 0.f, alpha = expf(m - ms);
        p[tid] = seen ? pv : -1.f;
        l = l * alpha + pv;
        acc *= alpha;
        m = m_new;
        __syncthreads();
        auto weigh = [&](int tile, auto masked) __attribute__((always_inline)) {
            const int k0 = c0 + tile * TILE_KEYS;           // a tile lies inside a page
            const T* vp = pool + kv_v_index(a.geom, a.layer, pages[k0 / a.geom.page_size], hkv, k0 % a.geom.page_size, dim);
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                float v[8];
                load8(vp + g * 128, v);                     // keys 4 g .. 4 g + 3 and 16 + 4 g .. of the tile
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float w0 = p[tile * TILE_KEYS + 4 * g + e], w1 = p[tile * TILE_KEYS + 16 + 4 * g + e];
                    acc = decltype(masked)::value && w0 < 0.f ? acc : fmaf(w0, v[e], acc);
                    acc = decltype(masked)::value && w1 < 0.f ? acc : fmaf(w1, v[4 + e], acc);
                }
            }
        };
        int tile = grp;                                     // first the tiles in which nothing is masked
        for (; tile < CK / TILE_KEYS && c0 + (tile + 1) * TILE_KEYS <= all_seen; tile += GROUPS) weigh(tile, std::false_type{});
        for (; tile < CK / TILE_KEYS && c0 + tile * TILE_KEYS < end; tile += GROUPS) weigh(tile, std::true_type{});
        __syncthreads();
    }
    acc_sh[grp][dim] = acc;
    l = wave_sum(l);
    if ((tid & 63) == 0) red[tid >> 6] = l;
    __syncthreads();
    if (tid < D) {
        float v = acc_sh[0][tid];
#pragma unroll
        for (int g = 1; g < GROUPS; ++g) v += acc_sh[g][tid];
        const float den = (red[0] + red[1]) + (red[2] + red[3]);
        Store<T>::store(reinterpret_cast<T*>(a.last_of ? a.last_out : a.out) + act_index(t_out, h * D + tid, a.Hq * D, a.out_packed), v / den);
    }
}

// A step's request of more than kStepRows stacked rows stays with the generic kernel: fp32 softmax weights, and a chain that
// has run into NaN does not touch the others (the MFMA kernels multiply a masked key's V by zero).  No drafter in use
// stacks so many (8 q heads per kv head and 32 drafts), so the line is drawn for that and not for speed.
bool attn_mfma_ok(int dtype, int hd, int page_size, bool force_generic, int step_rows) {
    return !force_generic && dtype == 1 && hd == HD && page_size % TILE_KEYS == 0 && (page_size & (page_size - 1)) == 0 && step_rows <= kStepRows;
}

// Four waves take most of a CU's LDS: one work-group a CU, where two waves leave room for another.  So up to 256 work-groups, each as long as its keys,
// they run in half the time (one prompt's last rows, 8 work-groups, 48 -> 33 us), but for the few keys of whose time the merge of the waves is the
// larger part.  Of 257 to 512 some wait for a place, shortest last: still ahead where the pairs that share one are no longer than the longest alone
// (one prompt of 777 tokens, 340 work-groups, 44.0 -> 38.4 us; of 1100, 484, 7 us a layer less), behind where all are alike (pieces of 832 to 1100 keys in 300 to 512
// work-groups 5 to 12 us more, of 260 to 400 keys, four prompts, 2 to 6) -- until the keys are so many that a lone work-group's pace decides (4200 to
// 5440 keys 3 less to 1 more, 8160 and up 7 to 43 less).  us a layer in a prefill, over 2 to 16 kv heads.
constexpr int kPrefillLong = 256, kPrefillPairs = 512, kPrefillEndless = 4096;

bool prefill_four_waves(const int* keys, int items, int Hkv) {
    constexpr int CUS = 256;
    const long long wgs = (long long)items * Hkv;
    if (items == 0 || wgs > 2 * CUS || keys[0] < kPrefillLong) return false;
    if (wgs <= CUS || keys[0] >= kPrefillEndless) return true;
    int pair = 0;                                         // most keys of two that share a place
    for (int i = CUS; i < wgs; ++i) pair = std::max(pair, keys[i / Hkv] + keys[(2 * CUS - 1 - i) / Hkv]);
    return keys[0] >= kPrefillPairs && 10 * pair <= 11 * keys[0];
}

hipError_t attention(const AttnArgs& a, hipStream_t st) {
    const float scale = 1.0f / sqrtf((float)a.hd);
    const int G = a.Hq / a.Hkv;
    if (attn_mfma_ok(a.dtype, a.hd, a.geom.page_size, a.force_generic, a.row_items ? 0 : G * a.n_max)) {
        const float sl2 = scale * 1.44269504088896340736f;
        // up to four 16-row tiles per work-group; more stacked rows are split over row groups
        AttnArgs b = a;
        const int tiles = a.row_items ? kItemRows / 16 : (G * a.n_max + 15) / 16;
        const int cap = a.row_items ? 4 : std::min(4, std::max(1, a.max_row_tiles));
        b.row_groups = (tiles + cap - 1) / cap;
        const int R = b.row_groups == 1 ? std::max(tiles, a.min_row_tiles) : (tiles + b.row_groups - 1) / b.row_groups;
        const int items = a.grid_items > 0 ? a.grid_items : a.n_work;
        dim3 grid((items * a.Hkv + 7) / 8 * 8 * b.row_groups);
        auto launch = [&](auto kern, int r, int waves) -> hipError_t {
            const size_t lds = std::max((size_t)waves * HD * (16 * r + 1) * sizeof(float), (size_t)waves * 2 * kTileBytes);
            hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            if (e != hipSuccess) return e;
            hipLaunchKernelGGL(kern, grid, dim3(64 * waves), lds, st, b, sl2);
            return hipGetLastError();
        };
        auto launch_regs = [&](auto kern, int r) -> hipError_t {
            const size_t lds = (size_t)4 * HD * (16 * r + 1) * sizeof(float);
            hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            if (e != hipSuccess) return e;
            hipLaunchKernelGGL(kern, grid, dim3(256), lds, st, b, sl2);
            return hipGetLastError();
        };
        hipError_t e;
        const bool once = a.cold && b.row_groups == 1 && !a.row_items;
        if (b.row_groups > 1 || R >= 4) {
            switch (R) {
                case 1: e = launch_regs(attn_bf16_regs_kernel<1, false>, 1); break;
                case 2: e = launch(attn_bf16_kernel<2, 2, 2>, 2, 2); break;
                case 3: e = launch(attn_bf16_kernel<3, 2, 2>, 3, 2); break;
                default: e = a.row_items ? (a.four_waves ? launch(attn_bf16_kernel<4, 4, 3>, 4, 4) : launch(attn_bf16_kernel<4, 2, 3>, 4, 2))
                           : once ? launch(attn_bf16_kernel<4, 2, 2, true>, 4, 2) : launch(attn_bf16_kernel<4, 2, 2>, 4, 2); break;
            }
        } else {
            switch (R) {
                case 1: e = once ? launch_regs(attn_bf16_regs_kernel<1, true>, 1) : launch_regs(attn_bf16_regs_kernel<1, false>, 1); break;
                case 2: e = once ? launch_regs(attn_bf16_regs_kernel<2, true>, 2) : launch_regs(attn_bf16_regs_kernel<2, false>, 2); break;
                default: e = once ? launch_regs(attn_bf16_regs_kernel<3, true>, 3) : launch_regs(attn_bf16_regs_kernel<3, false>, 3); break;
            }
        }
        if (e != hipSuccess) return e;
        if (a.merge || a.last_of) hipLaunchKernelGGL(attn_merge_kernel, dim3(a.last_of ? a.n_last : a.T, (a.Hq + 7) / 8), dim3(256), 0, st, b);
        return hipGetLastError();
    }
    dim3 grid(a.last_of ? a.n_last : a.T, a.Hq);
    if (a.dtype == 1 && a.hd == 128)
        hipLaunchKernelGGL((attn_generic_kernel<bf16_t, 128>), grid, dim3(256), 0, st, a, scale);
    else if (a.dtype == 1 && a.hd == 64)
        hipLaunchKernelGGL((attn_generic_kernel<bf16_t, 64>), grid, dim3(256), 0, st, a, scale);
    else if (a.dtype == 0 && a.hd == 128)
        hipLaunchKernelGGL((attn_generic_kernel<float, 128>), grid, dim3(256), 0, st, a, scale);
    else if (a.dtype == 0 && a.hd == 64)
        hipLaunchKernelGGL((attn_generic_kernel<float, 64>), grid, dim3(256), 0, st, a, scale);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace sv
