// Dense projections of the target's forward pass: out[s][M][N] = A[M, Ks] * W[N, Ks]^T, where the
// reduction dimension may be cut into `splits` contiguous ranges whose partial products are written
// side by side and summed by the consuming kernel (deterministic split-K).
//
// bf16 path: v_mfma_f32_16x16x32_bf16, fp32 accumulate.  A work-group of WM x WN waves computes a
// (16*MT*WM) x (16*NT*WN) tile; the weight tile is the MFMA "A" operand (rows = output features) and the
// activation tile the "B" operand, so a lane ends up with four consecutive output features of one
// token and stores them as one 16-byte word.  Operand tiles are staged through LDS (row pitch 72
// elements: the 16 lanes of a quarter-wave hit 64 distinct banks), double buffered, with the next
// tile's global loads in flight during the MFMAs of the current one.  Work-group ids are remapped so
// that the groups that share one weight panel run on the same XCD (one L2) at about the same time.
#include <algorithm>
#include <cmath>
#include <type_traits>
#include "common.h"
#include "kernels.h"

namespace sv {

constexpr int BK = 64;
constexpr int LDS_PITCH = BK + 8;

template <int MT, int NT, int WM, int WN>
__global__ __launch_bounds__(64 * WM * WN) void gemm_bf16_kernel(
    const bf16_t* __restrict__ A, const bf16_t* __restrict__ W, float* __restrict__ out,
    int M, int N, int K, int k_per_split, int splits, int tiles_m, int tiles_n) {
    constexpr int BM = 16 * MT * WM;       // tokens per group tile
    constexpr int BN = 16 * NT * WN;       // output features per group tile
    constexpr int NTHR = 64 * WM * WN;
    constexpr int A_CH = BM * (BK / 8) / NTHR;   // 16-byte chunks per thread
    constexpr int W_CH = BN * (BK / 8) / NTHR;
    static_assert(BM * (BK / 8) % NTHR == 0 && BN * (BK / 8) % NTHR == 0, "tile/threads mismatch");

    extern __shared__ __attribute__((aligned(16))) bf16_t lds[];
    bf16_t* As = lds;                                  // [2][BM][LDS_PITCH]
    bf16_t* Ws = lds + 2 * BM * LDS_PITCH;             // [2][BN][LDS_PITCH]

    const int nblk = tiles_m * tiles_n * splits;
    int logical = xcd_remap(blockIdx.x, nblk);
    const int tm = logical % tiles_m;
    logical /= tiles_m;
    const int sp = logical % splits;
    const int tn = logical / splits;
    const int m0 = tm * BM, n0 = tn * BN;
    const int kbeg = sp * k_per_split;
    const int nk = k_per_split / BK;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave % WM, wn = wave / WM;
    const int l16 = lane & 15, lg = lane >> 4;

    u32x4 a_reg[A_CH], w_reg[W_CH];
    auto load_global = [&](int kt) {
        const int k0 = kbeg + kt * BK;
#pragma unroll
        for (int i = 0; i < A_CH; ++i) {
            const int cid = tid + i * NTHR, row = cid >> 3, ch = cid & 7;
            int gm = m0 + row;
            gm = gm < M ? gm : M - 1;
            a_reg[i] = *reinterpret_cast<const u32x4*>(A + (int64_t)gm * K + k0 + ch * 8);
        }
#pragma unroll
        for (int i = 0; i < W_CH; ++i) {
            const int cid = tid + i * NTHR, row = cid >> 3, ch = cid & 7;
            w_reg[i] = *reinterpret_cast<const u32x4*>(W + (int64_t)(n0 + row) * K + k0 + ch * 8);
        }
    };
    auto store_lds = [&](int buf) {
#pragma unroll
        for (int i = 0; i < A_CH; ++i) {
            const int cid = tid + i * NTHR, row = cid >> 3, ch = cid & 7;
            *reinterpret_cast<u32x4*>(As + (buf * BM + row) * LDS_PITCH + ch * 8) = a_reg[i];
        }
#pragma unroll
        for (int i = 0; i < W_CH; ++i) {
            const int cid = tid + i * NTHR, row = cid >> 3, ch = cid & 7;
            *reinterpret_cast<u32x4*>(Ws + (buf * BN + row) * LDS_PITCH + ch * 8) = w_reg[i];
        }
    };

    floatx4 acc[NT][MT];
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int j = 0; j < MT; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};

    load_global(0);
    store_lds(0);
    __syncthreads();
    for (int kt = 0; kt < nk; ++kt) {
        const int buf = kt & 1;
        if (kt + 1 < nk) load_global(kt + 1);
#pragma unroll
        for (int kk = 0; kk < BK / 32; ++kk) {
            bf16x8 wf[NT], af[MT];
#pragma unroll
            for (int i = 0; i < NT; ++i)
                wf[i] = *reinterpret_cast<const bf16x8*>(
                    Ws + (buf * BN + (wn * NT + i) * 16 + l16) * LDS_PITCH + kk * 32 + lg * 8);
#pragma unroll
            for (int j = 0; j < MT; ++j)
                af[j] = *reinterpret_cast<const bf16x8*>(
                    As + (buf * BM + (wm * MT + j) * 16 + l16) * LDS_PITCH + kk * 32 + lg * 8);
#pragma unroll
            for (int i = 0; i < NT; ++i)
#pragma unroll
                for (int j = 0; j < MT; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[i], af[j], acc[i][j], 0, 0, 0);
        }
        if (kt + 1 < nk) store_lds(buf ^ 1);
        __syncthreads();
    }

    // lane holds, per (i, j): features n = n0 + (wn*NT+i)*16 + 4*lg + {0..3}, token m = m0 + (wm*MT+j)*16 + l16
    float* dst = out + (int64_t)sp * M * N;
#pragma unroll
    for (int j = 0; j < MT; ++j) {
        const int m = m0 + (wm * MT + j) * 16 + l16;
        if (m < M) {
#pragma unroll
            for (int i = 0; i < NT; ++i) {
                const int n = n0 + (wn * NT + i) * 16 + 4 * lg;
                *reinterpret_cast<floatx4_any*>(dst + (int64_t)m * N + n) = acc[i][j];
            }
        }
    }
}

typedef __attribute__((ext_vector_type(16))) float floatx16;

// ---- second bf16 kernel: weight streaming (v_mfma_f32_32x32x16_bf16; one wave per SIMD issuing independent
// 16x16x32 MFMAs reaches 1.34 PFLOP/s over the chip, the 32x32x16 form 2.41: a kernel whose accumulators leave room
// for one wave per SIMD only must use the larger form).  For the few hundred rows of a verification step the
// projections sit on the ridge between HBM and MFMA, and what matters is that the weights stream at
// memory speed.  A wave owns a strip of NT 32-feature tiles and loads ITS weight fragments (packed
// order: one contiguous 1 KB per fragment) straight from global memory into the registers the MFMA
// reads, PD k-slices ahead, with no LDS and no barrier on that path.  Only the activations, which every
// wave needs, go through LDS: KA 16-wide slices of all MT 32-token tiles per fill (packed order too, so
// a fill is a handful of contiguous 1 KB copies), double buffered, one barrier per fill.
template <int MT, int NT, int KA, int PD, bool GLU, bool STREAM, bool LEAVE>
__device__ __forceinline__ void gemm_bf16_ws_body(
    const bf16_t* __restrict__ Ap, const bf16_t* __restrict__ Wp, float* __restrict__ out,
    int M, int N, int K, int k_per_split, int splits, int tiles_m, int tiles_n, int tn0, int block_id) {
    constexpr int BM = 32 * MT, BN = 128 * NT;
    constexpr int AFR = MT * KA;                          // activation fragments per fill
    static_assert(AFR % 4 == 0, "fill must split over 4 waves");
    constexpr int APW = AFR / 4;                          // 1 KB pieces per wave per fill
    __shared__ __attribute__((aligned(16))) unsigned char abuf[2][AFR * 1024];

    const int nblk = tiles_m * tiles_n * splits;
    int logical = xcd_remap(block_id, nblk);
    const int tm = logical % tiles_m;
    logical /= tiles_m;
    const int sp = logical % splits;
    const int tn = tn0 + logical / splits;
    const int m0 = tm * BM, n0 = tn * BN;
    const int ks0 = sp * (k_per_split / 16);              // first 16-wide slice of this split
    const int nfill = k_per_split / (16 * KA);
    const int kslices = K / 16;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l32 = lane & 31, lg = lane >> 5;

    // activations, packed [M/32][K/16][64][8]: piece i of this wave's share of a fill
    const int m_tiles_total = (M + 31) / 32;
    const bf16_t* a_src[APW];
#pragma unroll
    for (int i = 0; i < APW; ++i) {
        const int f = wave * APW + i;                     // fragment of the fill: tile f / KA, slice f % KA
        int mt = m0 / 32 + f / KA;
        mt = mt < m_tiles_total ? mt : m_tiles_total - 1;
        a_src[i] = Ap + ((int64_t)mt * kslices + ks0 + f % KA) * 512 + lane * 8;
    }
    // weights, packed [N/128][K/16][4][64][8]: fragment (tile nt, slice ks)
    const bf16_t* w_src[NT];
#pragma unroll
    for (int i = 0; i < NT; ++i) {
        // gated form (N = 2F weight rows, gate rows first).  NT == 1: work-group tn covers features
        // 64 tn .. 64 tn + 63; waves 0,1 stream their gate rows, waves 2,3 the up rows of the same features.
        // NT == 2: work-group tn covers features 128 tn .. 128 tn + 127; every wave streams the gate rows (i = 0)
        // and the up rows (i = 1) of its own 32 features.
        const int nt = !GLU ? n0 / 32 + wave * NT + i
                     : NT == 1 ? (wave < 2 ? 2 * tn + wave : N / 64 + 2 * tn + (wave - 2))
                               : (i == 0 ? 4 * tn + wave : N / 64 + 4 * tn + wave);
        w_src[i] = Wp + (((int64_t)(nt >> 2) * kslices + ks0) * 4 + (nt & 3)) * 512 + lane * 8;
    }
    constexpr int W_STEP = 4 * 512;                       // elements between consecutive slices of a tile
    // STREAM: no other row tile reads these weights
    auto load_w = [&](int i, int slice) __attribute__((always_inline)) {
        const u32x4* p = reinterpret_cast<const u32x4*>(w_src[i] + (int64_t)slice * W_STEP);
        return STREAM ? load_stream(p) : *p;
    };

    floatx16 acc[NT][MT];
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int j = 0; j < MT; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

    const int total_slices = nfill * KA;
    u32x4 wring[PD][NT];                                  // weight fragments in flight
#pragma unroll
    for (int p = 0; p < PD; ++p)
#pragma unroll
        for (int i = 0; i < NT; ++i)
            wring[p][i] = load_w(i, p < total_slices ? p : total_slices - 1);

    // first fill
    u32x4 areg[APW];
#pragma unroll
    for (int i = 0; i < APW; ++i) areg[i] = *reinterpret_cast<const u32x4*>(a_src[i]);
#pragma unroll
    for (int i = 0; i < APW; ++i) *reinterpret_cast<u32x4*>(&abuf[0][(wave * APW + i) * 1024 + lane * 16]) = areg[i];

    for (int fill = 0; fill < nfill; ++fill) {
        // everyone's share of this fill is in LDS; the other buffer has no reader left
        __builtin_amdgcn_s_waitcnt(0xC07F);               // lgkmcnt(0): own LDS writes done
        __builtin_amdgcn_s_barrier();
        // next fill's activations: loaded unconditionally (the last fill is loaded twice) so that the loop body
        // has no branch and the compiler can count the loads in flight exactly; behind a branch it falls back
        // to waiting for these loads at the first product of the fill
        const int nxt = fill + 1 < nfill ? fill + 1 : fill;
#pragma unroll
        for (int i = 0; i < APW; ++i) areg[i] = *reinterpret_cast<const u32x4*>(a_src[i] + (int64_t)nxt * KA * 512);
        const unsigned char* ab = abuf[fill & 1] + lane * 16;
        static_assert(KA % PD == 0, "ring slots must be static across a fill");
        bf16x8 af[2][MT];                                  // activation fragments: this slice and the next
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
            // keep loads and reads where they are: left alone, the scheduler sinks each one to just before
            // its use and the stream degenerates into load - wait - compute
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < NT; ++i)
#pragma unroll
                for (int j = 0; j < MT; ++j)
                    // gated form: weights first, so that a lane holds one row and consecutive features (what the
                    // packed output wants); plain form: activations first, so that a lane holds one feature and the
                    // 32 lanes of a half wave write 128 contiguous bytes of an output row
                    acc[i][j] = GLU ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, wring[s % PD][i]),
                                                                              af[s & 1][j], acc[i][j], 0, 0, 0)
                                    : __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[s & 1][j], __builtin_bit_cast(bf16x8, wring[s % PD][i]),
                                                                              acc[i][j], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            // refill the ring slot just consumed with the slice PD ahead (clamped at the end: a harmless
            // re-load).  Issued after the products that read the slot, so the slot's registers are dead and
            // the load lands in place: issued before them, every slot needs a copy, and the compiler
            // gathers those copies at the top of the fill, behind a wait for the whole ring.
            const int ahead = slice + PD < total_slices ? slice + PD : total_slices - 1;
#pragma unroll
            for (int i = 0; i < NT; ++i)
                wring[s % PD][i] = load_w(i, ahead);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int i = 0; i < APW; ++i)
            *reinterpret_cast<u32x4*>(&abuf[(fill + 1) & 1][(wave * APW + i) * 1024 + lane * 16]) = areg[i];
    }

    if (GLU && NT == 2) {
        // gate and up of a feature sit in the same lane: silu(gate) * up in registers, rounded to bf16, written as
        // packed operand tiles [M/32][F/16][64][8] of the next projection
        const int F = N / 2;
        bf16_t* act = reinterpret_cast<bf16_t*>(out);
        const int fs = (tn * 128 + wave * 32) / 16;
#pragma unroll
        for (int j = 0; j < MT; ++j) {
            const int mt = m0 / 32 + j;
            if (mt < m_tiles_total) {
                bf16_t* dst = act + ((int64_t)mt * (F / 16) + fs) * 512;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    float r[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        r[i] = silu_mul(acc[0][j][4 * q + i], acc[NT - 1][j][4 * q + i]);
                    }
                    u32x2 pk = {pack2bf(r[0], r[1]), pack2bf(r[2], r[3])};
                    *reinterpret_cast<u32x2*>(dst + ((q >> 1) * 64 + l32 + 32 * (q & 1)) * 8 + 4 * lg) = pk;
                }
            }
        }
        return;
    }
    if (GLU) {
        // up halves travel through LDS to the waves that hold the gate halves; those write
        // silu(gate) * up, rounded to bf16, as packed operand tiles [M/32][F/16][64][8] of the next projection
        const int F = N / 2;
        bf16_t* act = reinterpret_cast<bf16_t*>(out);
        __builtin_amdgcn_s_waitcnt(0xC07F);
        __builtin_amdgcn_s_barrier();                        // every wave is done reading the activations
        float* xbuf = reinterpret_cast<float*>(&abuf[0][0]); // [2 waves][MT][16][64] floats
        static_assert(2 * MT * 16 * 64 * 4 <= 2 * AFR * 1024, "exchange area");
        if (wave >= 2) {
#pragma unroll
            for (int j = 0; j < MT; ++j)
#pragma unroll
                for (int q = 0; q < 16; ++q) xbuf[(((wave - 2) * MT + j) * 16 + q) * 64 + lane] = acc[0][j][q];
        }
        __builtin_amdgcn_s_waitcnt(0xC07F);
        __builtin_amdgcn_s_barrier();
        if (wave < 2) {
            const int fs = (tn * 64 + wave * 32) / 16;
#pragma unroll
            for (int j = 0; j < MT; ++j) {
                const int mt = m0 / 32 + j;
                if (mt < m_tiles_total) {
                    bf16_t* dst = act + ((int64_t)mt * (F / 16) + fs) * 512;
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        float r[4];
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const float g = acc[0][j][4 * q + i];
                            const float u = xbuf[((wave * MT + j) * 16 + 4 * q + i) * 64 + lane];
                            r[i] = silu_mul(g, u);
                        }
                        u32x2 pk = {pack2bf(r[0], r[1]), pack2bf(r[2], r[3])};
                        *reinterpret_cast<u32x2*>(dst + ((q >> 1) * 64 + l32 + 32 * (q & 1)) * 8 + 4 * lg) = pk;
                    }
                }
            }
        }
        return;
    }
    // acc[i][j][4 q + r] <-> row m0 + 32 j + 8 q + 4 lg + r, feature n0 + 32 (wave NT + i) + l32
    // A half wave fills a line of 128 bytes: streamed (LEAVE; where leaves_stream says so; LM head of 96 rows, 58 MB of logits, 224 -> 213 us; QKV
    // and O planes of 96 rows 12.5 + 10.5 -> 12.1 + 9.9, the attention between them 162 -> 160.5, norm and rotary + 0.4 and + 0.2).  The tall and
    // the strip kernel write half lines, which as streams cost the next norm more than they save.
    float* dst = out + (int64_t)sp * M * N;
#pragma unroll
    for (int i = 0; i < NT; ++i) {
        const int n = n0 + (wave * NT + i) * 32 + l32;
#pragma unroll
        for (int j = 0; j < MT; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int m = m0 + j * 32 + 8 * q + 4 * lg + r;
                    if (m >= M) continue;
                    if (LEAVE) store_stream(dst + (int64_t)m * N + n, (float)acc[i][j][4 * q + r]);
                    else dst[(int64_t)m * N + n] = acc[i][j][4 * q + r];
                }
    }
}

// Two work-groups share a CU where the accumulator tile leaves room (up to 96 rows x 256 features, or 128-feature
// strips): more, smaller work-groups resident at once, which evens out a launch whose work-group count is not a
// multiple of the 256 CUs.
template <int MT, int NT, int KA, int PD, bool GLU = false, bool STREAM = false, bool LEAVE = false>
__global__ __launch_bounds__(256, (NT == 1 || MT <= 3) ? 2 : 1) void gemm_bf16_ws_kernel(
    const bf16_t* __restrict__ Ap, const bf16_t* __restrict__ Wp, float* __restrict__ out,
    int M, int N, int K, int k_per_split, int splits, int tiles_m, int tiles_n, int tn0) {
    gemm_bf16_ws_body<MT, NT, KA, PD, GLU, STREAM, LEAVE>(Ap, Wp, out, M, N, K, k_per_split, splits, tiles_m, tiles_n, tn0, blockIdx.x);
}

// Gate/up projection with a short last round: the first n_main work-groups are 160-row ones over the 128-feature
// strips [0, strips_main); the rest are 64-row ones over the remaining strips cut in two (64 features each).  One
// launch: the small work-groups start on whichever CUs free up first instead of waiting for the whole main round.
// A small work-group streams the whole reduction depth of its weight rows whatever its share of the products,
// so the last round is bound by how often the strips are re-read from L2: 64 rows x 64 features (five readers of
// 0.9 MB per half strip) take 26 us where 32 rows x 128 features (ten readers of 1.8 MB) took 35 us.
// (Up-projections of more than 160 rows take the tall kernel by default: what reaches this one is 129 to 160 rows onto 33 to 48
// thousand features, and more rows with the tall kernel switched off.)
__global__ __launch_bounds__(256, 1) void gemm_bf16_ws_glu_mixed_kernel(
    const bf16_t* __restrict__ Ap, const bf16_t* __restrict__ Wp, float* __restrict__ out, int M, int N, int K,
    int tiles_m, int strips_main, int tiles_m2, int strips_tail) {
    const int n_main = tiles_m * strips_main;
    if ((int)blockIdx.x < n_main)
        gemm_bf16_ws_body<5, 2, 8, 8, true, false, false>(Ap, Wp, out, M, N, K, K, 1, tiles_m, strips_main, 0, blockIdx.x);
    else
        gemm_bf16_ws_body<2, 1, 8, 8, true, false, false>(Ap, Wp, out, M, N, K, K, 1, tiles_m2, 2 * strips_tail, 2 * strips_main, blockIdx.x - n_main);
}

// ---- third bf16 kernel: tall tiles, 64 RW rows x 256 features per work-group, both operands through LDS ----
// From a few hundred rows on the weights no longer dominate the traffic, and what bounds a projection is the chip's power:
// alone on the chip a work-group of this kernel runs its CU at 2.3 PFLOP/s / 256, with all CUs busy the clock drops until
// the whole makes 1.2-1.3 PFLOP/s on random operands, whatever the pipeline depth (three fills in flight 1.24 PFLOP/s on the
// LM head at 2304 rows, four and five 1.21; longer fills, raised wave priorities, a persistent grid: no gain).  What counts
// is that the matrix units never wait and that nothing is fetched twice:
//   * eight waves, two per SIMD, so that one multiplies while the other waits for LDS or the barrier.  (Four waves of 128 x 128
//     with a hand-woven stream, alone on their SIMDs, reached 1.07.)  A wave holds 32 RW rows x 64 features.
//   * a fill is two 16-wide slices of both operands, copied global -> LDS by direct-to-LDS loads in the packed orders, a ring
//     of three fills, one barrier per fill.
//   * tiles of two heights in one launch (RW, RWT), so that little of what is multiplied is padding: the shorter ones beside their
//     strip's other tiles where the launch takes several rounds (they share the strip through L2), behind them all in a launch of one or two rounds (they run on the CUs that the tall tiles leave idle).
// GLU: the tile's features are 128 gate rows and the 128 up rows of the same features; a wave holds both for its
// 32 features and writes silu(gate) * up, rounded to bf16, in the packed order of the next projection.
// Measured on MI355X (K = 3584), against the weight-streaming kernel / the four-wave one: gate/up of 37888 at 2304 rows
// 617 / 588 -> 525 us, at 1280 348 / 310 -> 279, at 256 104 -> 77; LM head of 152064 at 2304 rows 2480 / 2340 -> 2050, at 640
// 820 -> 611, at 256 402 -> 308; down (K = 18944) at 2304 rows 282 / 273 -> 243, at 3500 500 -> 411; QKV (4608) 98 -> 71.
constexpr int kTallFills = 3;                             // fills in the LDS ring
constexpr int kTallSlices = 2;                            // 16-wide slices per fill

template <bool GLU, int RW>
__device__ __forceinline__ void gemm_bf16_tall_body(const bf16_t* __restrict__ Ap, const bf16_t* __restrict__ Wp, float* __restrict__ out,
                                                    int M, int N, int K, int k_per_split, int m0, int tn, int sp) {
    extern __shared__ __attribute__((aligned(16))) unsigned char tall_lds[];   // kTallFills fills
    constexpr int KA = kTallSlices, NB = kTallFills;
    constexpr int B_OFF = KA * 2 * RW * 1024;             // weights (2 strips x 4 tiles a slice) behind the 2 RW row tiles
    constexpr int FILL = B_OFF + KA * 8 * 1024;
    const int nfill = k_per_split / (16 * KA), kslices = K / 16, ks0 = sp * (k_per_split / 16);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave >> 2, wn = wave & 3, l16 = lane & 15, lg = lane >> 4;
    const int m_tiles = (M + 31) / 32;

    // A fill is P pieces of 1 KB: the activations' 2 RW row tiles x 2 slices, then (strip, slice, feature tile) of the weights.  Wave w
    // requests pieces w, w + 8, ... ; where they do not come out even, the others take one lane of the last piece once more, so that
    // every wave counts the same loads without a branch (two branches cost 120 cycles a fill).  Row tiles beyond M and a strip beyond N
    // (N an odd multiple of 128) are read as the last one and never stored.
    constexpr int A_P = KA * 2 * RW, P = A_P + KA * 8, EACH = P / 8, EXTRA = P % 8;
    const uint64_t last_lanes = wave < EXTRA ? ~0ull : 1;
    const char* src[EACH + 1];
    int step[EACH + 1];
#pragma unroll
    for (int q = 0; q <= EACH; ++q) {
        const int p = min(wave + 8 * q, P - 1);
        if (p < A_P) {
            const int mt = min(m0 / 32 + p / KA, m_tiles - 1);
            src[q] = reinterpret_cast<const char*>(Ap + ((int64_t)mt * kslices + ks0 + p % KA) * 512);
            step[q] = KA * 1024;
        } else {
            const int w = p - A_P, strip = w / (4 * KA), strip_n = 2 * tn + strip;
            const int strip_g = GLU ? (strip == 0 ? tn : N / 256 + tn) : min(strip_n, N / 128 - 1);
            src[q] = reinterpret_cast<const char*>(Wp + (((int64_t)strip_g * kslices + ks0 + w / 4 % KA) * 4 + w % 4) * 512);
            step[q] = KA * 4096;
        }
    }
    const uint32_t lds0 = (uint32_t)(uintptr_t)SV_LDS_PTR(tall_lds), lane_off = lane * 16;
    int ahead = 0;
    auto request = [&](auto which, uint32_t base) __attribute__((always_inline)) {
        constexpr int Q = decltype(which)::value;
        if constexpr (Q < EACH) dma1(src[Q], lane_off, base + (wave + 8 * Q) * 1024);
        else if constexpr (EXTRA > 0) dma1_lanes(last_lanes, src[Q], lane_off, base + min(wave + 8 * Q, P - 1) * 1024);
    };
    auto advance = [&]() __attribute__((always_inline)) {  // past the end: the last fill again, so that the counts below hold
        if (++ahead < nfill) {
#pragma unroll
            for (int q = 0; q <= EACH; ++q) src[q] += step[q];
        }
    };
    auto wait_fills = [&](auto in_flight) __attribute__((always_inline)) {   // all but the newest in_flight fills have landed
        constexpr int L = decltype(in_flight)::value;
        wait_vmcnt<(EACH + (EXTRA > 0)) * L>();
    };

    // Operands of a fill.  Lane 16 g + r of a 16x16x32 operand holds row r, elements 8 g .. 8 g + 7 of the fill's 32: slice
    // g / 2 of the packed order, half g % 2 of its 16.  Weights: four 16-feature operands, two sets (this fill's, the next
    // one's); activations: 2 RW 16-row operands, in two halves.  The LDS reads are placed by hand, with hand-counted waits: the
    // compiler would wait for every read as soon as a direct-to-LDS load is in flight.  It takes the reads' registers as written
    // at once, so what a half reads is waited for in the basic block that reads it (a branch in between may copy registers
    // still in flight).
    u32x4 a[2][RW], b[2][4];
    const uint32_t in_piece = (lg & 1) * 512 + l16 * 16;
    const uint32_t a_off = lds0 + wm * RW * KA * 1024 + (lg >> 1) * 1024 + in_piece;
    const uint32_t b_off = lds0 + B_OFF + (GLU ? wn * 1024 : (wn >> 1) * KA * 4096 + (wn & 1) * 2048) + (lg >> 1) * 4096 + in_piece;
    constexpr int B_STEP = GLU ? KA * 4096 : 1024;        // from the wave's first 32 features to its second
    uint32_t a_addr = a_off, b_addr = b_off;
    auto read_a = [&](auto half, auto which) __attribute__((always_inline)) {
        constexpr int H = decltype(half)::value, J = decltype(which)::value, X = H * RW + J;
        lds_read16<(X >> 1) * KA * 1024 + (X & 1) * 256>(a[H][J], a_addr);
    };
    auto read_b = [&](auto set, auto which) __attribute__((always_inline)) {
        constexpr int S = decltype(set)::value, I = decltype(which)::value;
        lds_read16<(I >> 1) * B_STEP + (I & 1) * 256>(b[S][I], b_addr);
    };
    auto wait_a = [&](auto half) __attribute__((always_inline)) {
        constexpr int H = decltype(half)::value;
        lds_landed(a[H][0]);
#pragma unroll
        for (int j = 1; j < RW; ++j) lds_landed_too(a[H][j]);
    };
    auto wait_b = [&](auto set) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 4; ++i) lds_landed_too(b[decltype(set)::value][i]);
    };
    floatx4 acc[4][2 * RW];                               // [feature operand][row operand]
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2 * RW; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    // The products of half H of the rows with weight set S, a read after each: in half 0 the activations of half 1, in half 1 the
    // next fill's weights and the activations of its half 0; there also the requests of the fill NB ahead, spread over the products: the
    // texture path takes one every 17 cycles from the whole work-group, and a wave whose request waits there does not
    // multiply.  Weights first, so that a lane holds one
    // row and four consecutive features.
    // The features turn round with each row operand, so that two products in a row differ in one operand only: less power drawn, which is what
    // bounds the large launches (a loop of products alone 2.01 -> 2.05 PFLOP/s; steps of 1280 and 2304 rows 0.3 to 0.9 % shorter, of 20 to 800 within 0.5 % of level).
    auto multiply = [&](auto half, auto set, uint32_t base) __attribute__((always_inline)) {
        constexpr int H = decltype(half)::value, S = decltype(set)::value, NM = 4 * RW, NR = H == 0 ? RW : RW + 4;
        __builtin_amdgcn_sched_barrier(0);
        static_for<NM>([&](auto mi) __attribute__((always_inline)) {
            constexpr int m = decltype(mi)::value, j = m >> 2, i = (j + H * RW) & 1 ? 3 - (m & 3) : m & 3;
            acc[i][H * RW + j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, b[S][i]), __builtin_bit_cast(bf16x8, a[H][j]),
                                                                         acc[i][H * RW + j], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            constexpr int first = m < NR ? m : NR, last = m + 1 == NM ? NR : m + 1 < NR ? m + 1 : NR;
            static_for<last - first>([&](auto rr) __attribute__((always_inline)) {
                constexpr int r = first + decltype(rr)::value;
                if constexpr (H == 0) read_a(std::integral_constant<int, 1>{}, std::integral_constant<int, r>{});
                else if constexpr (r < 4) read_b(std::integral_constant<int, 1 - S>{}, std::integral_constant<int, r>{});
                else read_a(std::integral_constant<int, 0>{}, std::integral_constant<int, r - 4>{});
                __builtin_amdgcn_sched_barrier(0);
            });
            constexpr int NQ = EACH + (EXTRA > 0), q = (m * NQ + NM - 1) / NM;      // request q after product q NM / NQ
            if constexpr (H == 1 && q < NQ && q * NM / NQ == m) {
                request(std::integral_constant<int, q>{}, base);
                __builtin_amdgcn_sched_barrier(0);
            }
        });
    };

    const std::integral_constant<int, 0> i0;
    const std::integral_constant<int, 1> i1;
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        static_for<EACH + 1>([&](auto q) __attribute__((always_inline)) { request(q, lds0 + i * FILL); });
        advance();
    }
    wait_fills(std::integral_constant<int, NB - 1>{});
    __builtin_amdgcn_s_barrier();
    static_for<4>([&](auto r) __attribute__((always_inline)) { read_b(i0, r); });
    static_for<RW>([&](auto r) __attribute__((always_inline)) { read_a(i0, r); });
    wait_a(i0);
    wait_b(i0);
    int slot = 0;
    auto fill = [&](auto set) __attribute__((always_inline)) {
        multiply(i0, set, lds0);
        wait_a(i1);
        // This wave holds all it needs of the fill and its share of the next one has landed; after the barrier so has
        // everyone's, and nobody reads this fill's place in the ring any more.
        wait_fills(std::integral_constant<int, NB - 2>{});
        __builtin_amdgcn_s_barrier();
        const uint32_t base = lds0 + slot * FILL;
        slot = slot + 1 == NB ? 0 : slot + 1;
        a_addr = a_off + slot * FILL;
        b_addr = b_off + slot * FILL;
        multiply(i1, set, base);
        wait_a(i0);
        wait_b(std::integral_constant<int, 1 - decltype(set)::value>{});
        advance();
    };
    int f = 0;
    for (; f + 1 < nfill; f += 2) { fill(i0); fill(i1); }
    if (f < nfill) fill(i0);
    wait_vmcnt<0>();                                      // nothing of this work-group may land in LDS after it has gone

    // acc[i][x][e] <-> row m0 + 32 RW wm + 16 x + l16, feature 4 lg + e of the wave's 16-feature operand i
    if (GLU) {                                            // operands 0, 1: gate rows of 32 features, 2, 3: their up rows
        const int F = N / 2;
        bf16_t* act = reinterpret_cast<bf16_t*>(out);
        const int fs = (tn * 128 + wn * 32) / 16;
#pragma unroll
        for (int x = 0; x < 2 * RW; ++x) {
            const int mt = m0 / 32 + wm * RW + (x >> 1);
            if (mt < m_tiles) {
                bf16_t* dst = act + ((int64_t)mt * (F / 16) + fs) * 512 + ((lg >> 1) * 32 + (x & 1) * 16 + l16) * 8 + 4 * (lg & 1);
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    float r[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        r[e] = silu_mul(acc[i][x][e], acc[2 + i][x][e]);
                    }
                    *reinterpret_cast<u32x2*>(dst + i * 512) = u32x2{pack2bf(r[0], r[1]), pack2bf(r[2], r[3])};
                }
            }
        }
        return;
    }
    if (tn * 256 + wn * 64 >= N) return;
    float* dst = out + (int64_t)sp * M * N + tn * 256 + wn * 64 + 4 * lg;
#pragma unroll
    for (int x = 0; x < 2 * RW; ++x) {
        const int m = m0 + wm * RW * 32 + 16 * x + l16;
        if (m < M) {
#pragma unroll
            for (int i = 0; i < 4; ++i) *reinterpret_cast<floatx4_any*>(dst + (int64_t)m * N + 16 * i) = acc[i][x];
        }
    }
}

// n tiles of 64 RW rows along the rows, then nt of 64 RWT; tail_last: the short ones behind all others.
template <bool GLU, int RW, int RWT>
__global__ __launch_bounds__(512, 2) void gemm_bf16_tall_kernel(const bf16_t* __restrict__ Ap, const bf16_t* __restrict__ Wp,
                                                                float* __restrict__ out, int M, int N, int K, int k_per_split, int splits,
                                                                int n, int nt, int tiles_n, int tail_last) {
    const int n_main = n * tiles_n * splits;
    int tm, logical;
    if (RWT > 0 && tail_last && (int)blockIdx.x >= n_main) {
        logical = xcd_remap(blockIdx.x - n_main, nt * tiles_n * splits);
        tm = n + logical % nt;
        logical /= nt;
    } else {
        const int along = n + (RWT > 0 && !tail_last ? nt : 0);
        logical = xcd_remap(blockIdx.x, along * tiles_n * splits);
        tm = logical % along;
        logical /= along;
    }
    const int sp = logical % splits, tn = logical / splits;
    if (RWT == 0 || tm < n) gemm_bf16_tall_body<GLU, RW>(Ap, Wp, out, M, N, K, k_per_split, tm * 64 * RW, tn, sp);
    else gemm_bf16_tall_body<GLU, RWT == 0 ? RW : RWT>(Ap, Wp, out, M, N, K, k_per_split, n * 64 * RW + (tm - n) * 64 * RWT, tn, sp);
}

// Microseconds a launch of the tall kernel takes, by the same kind of play-through as the weight-streaming plan.  Fitted to the kernel's
// earlier form on 32x32x16 products; for this one it is up to 26 % high: gate/up 37888 x 3584 at 192 / 320 rows 78 / 103 where it takes 72 / 89,
// 28672 x 4096 at 320 90 for 71, down of the 7B shape at 2304 269 for 230; LM heads of 152 thousand features 13 % low (2048 inputs) to 8 % high (5120).  Of the lines that
// weigh it against the other kernels 0.80 and 1.25 were measured with this form, 1.10 with the earlier one.  (The fit: 900
// launches of 17 row counts from 128 to 3500, three shapes and four split counts; nine in ten estimates lay between 0.77 and
// 1.05 of the measured time, and over 63 other launches the tiles it prefers take 2 % longer than the best on average.  Two
// heights against one and a remainder: gate/up of 55296 over K = 5120 at 800 rows, one tile of 320 and two of 256: 445 us,
// three of 256 and one of 64: 468; of 37888 over 3584 at 777 rows 198 us against 224).
// A tile costs its slices at the pace of a CU alone; the chip as a whole sustains kRate; whole rounds take the
// larger of the two (rounded over the corner), a last round that is not full is hidden in part where there are several;
// the weight stream adds to both, as it draws on the same power.
static double gemm_bf16_tall_us(int M, int N, int K, int splits, const TallTiles& tl) {
    static const double kSlice[6] = {0, 0.130, 0.165, 0.208, 0.245, 0.327};            // us per slice of a lone tile of 64 rw rows
    static const double kRate[6] = {1, 0.70e9, 1.00e9, 1.15e9, 1.25e9, 1.25e9};        // flop per us over the chip
    const double slices = (double)K / 16 / splits, wgs = (double)((N + 255) / 256) * splits;
    auto alone = [&](int r) { return kSlice[r] * slices + 4.0; };
    auto share = [&](int r) { return 2.0 * 64 * r * 256 * 16 * slices / kRate[r]; };
    auto corner = [](double x, double y) { return std::sqrt(std::sqrt(x * x * x * x + y * y * y * y)); };
    const double n1 = tl.n * wgs, n2 = tl.nt * wgs, d1 = alone(tl.rw), p1 = share(tl.rw), d2 = tl.nt ? alone(tl.rwt) : 0, p2 = tl.nt ? share(tl.rwt) : 0;
    const double rounds = std::floor(n1 / 256), rem = n1 - 256 * rounds;
    double t = rounds > 0 ? rounds * corner(d1, 256 * p1) : 0;
    const double power = rem * p1 + n2 * p2;
    if (rounds >= 2) {
        if (rem > 0 || n2 > 0) t += std::max(0.5 * d1, power);
    } else {
        const double beside = rem > 0 && n2 > 0 ? (256 - rem) * std::floor(d1 / d2) : 0;    // short tiles that run beside the tall ones
        const double d = (rem > 0 ? d1 : 0) + std::ceil(std::max(0.0, n2 - beside) / 256) * d2;
        if (d > 0) t += corner(d, power);
    }
    const double stream = (double)N * K * 2.0 / 5.5e6;
    return std::sqrt(t * t + stream * stream) + (splits - 1) * (double)M * N * 4.0 / 4.0e6 + 2.3;             // the consumer reads the planes
}

// The tiles that cover M rows with heights 64 rw and 64 rwt (0: one height only): least padding, then most tall ones.  Heights
// of one and two waves' row tiles multiply at a poor rate and come once at most.
static bool gemm_bf16_tall_tiles(int M, int rw, int rwt, TallTiles& tl) {
    const int need = (M + 63) / 64;
    if (rwt == 0) { tl = TallTiles{rw, (need + rw - 1) / rw, 0, 0}; return rw == 3 || rw <= need; }
    int over = rw;
    for (int n = need / rw; n >= 1; --n) {
        const int nt = (need - n * rw + rwt - 1) / rwt, pad = n * rw + nt * rwt - need;
        if (nt < 1 || (rwt < 3 && nt > 1) || pad >= over) continue;
        over = pad;
        tl = TallTiles{rw, n, rwt, nt};
    }
    return over < rw;
}

// Tiles and splits for the tall kernel: the best by the estimate.
TallPlan gemm_bf16_tall_plan(int M, int N, int K, int max_splits) {
    TallPlan best{1, {4, (M + 255) / 256, 0, 0}, 1e30};
    TallTiles tl;
    for (int rw = 3; rw <= 5; ++rw)
        for (int rwt = 0; rwt < rw; ++rwt) {
            if (!gemm_bf16_tall_tiles(M, rw, rwt, tl)) continue;
            for (int s = 1; s <= max_splits; ++s) {
                if ((K / 16) % (kTallSlices * s) != 0) continue;
                const double t = gemm_bf16_tall_us(M, N, K, s, tl);
                if (t < best.us) best = TallPlan{s, tl, t};
            }
        }
    return best;
}

// 256-row tiles and one shorter tile for the rows that are left.
TallTiles gemm_bf16_tall_256(int M) {
    const int need = (M + 63) / 64, rest = need % 4;
    return need <= 3 ? TallTiles{3, 1, 0, 0} : TallTiles{4, need / 4, rest, rest ? 1 : 0};
}

// plain: out [splits][M][N] fp32, N % 128 == 0.  gated: N = 2 F weight rows, out = packed bf16 [ceil(M/32)*32, F],
// F % 128 == 0, splits == 1.  (K / splits) % 32 == 0.
hipError_t gemm_bf16_tall(const bf16_t* Ap, const bf16_t* Wp, float* out, int M, int N, int K, int splits, bool glu, const TallTiles& tl, hipStream_t st) {
    if (splits < 1 || K % splits != 0 || (K / splits) % (16 * kTallSlices) != 0 || N % (glu ? 256 : 128) != 0 || (glu && splits != 1) ||
        tl.rw < 3 || tl.rw > 5 || tl.n < 1 || tl.rwt < 0 || tl.rwt >= tl.rw || tl.nt < 0 || (tl.nt > 0) != (tl.rwt > 0) ||
        64LL * (tl.rw * tl.n + tl.rwt * tl.nt) < M)
        return hipErrorInvalidValue;
    const int tiles_n = (N + 255) / 256, blocks = (tl.n + tl.nt) * tiles_n * splits;
    const int tail_last = tl.n * tiles_n * splits < 2 * 256;
    auto launch = [&](auto kern) -> hipError_t {
        const int lds = kTallFills * kTallSlices * (2 * tl.rw + 8) * 1024;
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kern, dim3(blocks), dim3(512), lds, st, Ap, Wp, out, M, N, K, K / splits, splits, tl.n, tl.nt, tiles_n, tail_last);
        return hipGetLastError();
    };
    auto form = [&](auto g) -> hipError_t {
        constexpr bool G = decltype(g)::value;
        switch (tl.rw * 8 + tl.rwt) {
            case 24: return launch(gemm_bf16_tall_kernel<G, 3, 0>);
            case 25: return launch(gemm_bf16_tall_kernel<G, 3, 1>);
            case 26: return launch(gemm_bf16_tall_kernel<G, 3, 2>);
            case 32: return launch(gemm_bf16_tall_kernel<G, 4, 0>);
            case 33: return launch(gemm_bf16_tall_kernel<G, 4, 1>);
            case 34: return launch(gemm_bf16_tall_kernel<G, 4, 2>);
            case 35: return launch(gemm_bf16_tall_kernel<G, 4, 3>);
            case 40: return launch(gemm_bf16_tall_kernel<G, 5, 0>);
            case 41: return launch(gemm_bf16_tall_kernel<G, 5, 1>);
            case 42: return launch(gemm_bf16_tall_kernel<G, 5, 2>);
            case 43: return launch(gemm_bf16_tall_kernel<G, 5, 3>);
            default: return launch(gemm_bf16_tall_kernel<G, 5, 4>);
        }
    };
    return glu ? form(std::true_type{}) : form(std::false_type{});
}

// ---- fourth bf16 kernel: the tall kernel's scheme in narrow strips, one work-group for all rows ----
// Up to 320 rows a projection is bound by its weight stream and by how many CUs stream it.  The weight-streaming kernel above
// holds the stream in registers, eight slices a wave, and its strips of 128 or 256 features seldom come to the number of CUs; the
// tall kernel's 256-feature strips of the 7B gate/up projection are 148 work-groups.  Here both operands go through an LDS ring of
// fills of one reduction step of 32 in pieces of one 16x16x32 operand, so that a strip can be any multiple of 32 features (gated: of
// 16 gate and 16 up ones): 128, 160 or 224, whichever comes closest to the 256 CUs (widths between them are not built: a width is 16
// kernels, and a shape that just misses one round at one of them puts 183 strips or more on the CUs at the next).  W waves, two of them
// side by side along the features, each RS 16-row operands x FS 16-feature operands, all of a fill's operands in one of two register sets: one
// barrier a fill, the next fill's LDS reads and the ring's requests between the products.
// The request of a ring's fill costs a wave its place at the texture path (17 cycles a piece, one queue per CU): sent in a burst
// behind the barrier, ten row tiles of 160 features took 1536 cycles a fill on an otherwise idle chip, spread 1062 (800 of them
// products).  With the chip full the stream adds to that: fills arrive at 5.7 to 6.2 TB/s where the products are few.
// us alone with weights from HBM, against the kernel that was taken before: gate/up 37888 x 3584 at 5 / 64 / 96 / 128 / 160 / 192 /
// 256 / 320 rows 46.2 / 49.4 / 54.3 / 58.6 / 62.7 / 69.4 / 76.9 / 88.1 -> 44.2 / 44.0 / 45.0 / 47.7 / 52.1 / 56.6 / 68.9 / 76.8; down 3584 x
// 18944 at 5 / 64 / 160 rows 23.8 / 25.6 / 31.8 -> 21.3 / 23.0 / 30.6; QKV 4608 x 3584 6.3 / 7.5 / 13.1 -> 4.6 / 6.7 / 11.1.
// Weights read with the hint of load_stream, us inside a step: gate/up of 5 / 42 / 96 rows 49.3 / 49.9 / 51.7 -> 45.2 / 46.6 / 49.4, of 55296 x 5120 at
// 147 rows 121 -> 106; down of 5 rows 26.1 -> 24.4; LM head of 147 rows 333 -> 308.
// The sums are those of the other two kernels, slice after slice: equal bits at the same splits.
constexpr int strip_fills(int w, int rs, int fs) {        // fills in the ring: two work-groups of four waves share a CU's LDS
    const int n = (w == 4 ? 80 : 160) / (w / 2 * rs + 2 * fs);
    return n < 6 ? n : 6;
}

template <bool GLU, int W, int RS, int FS, bool STREAM>
__global__ __launch_bounds__(64 * W, 2) void gemm_bf16_strip_kernel(const bf16_t* __restrict__ Ap, const bf16_t* __restrict__ Wp, float* __restrict__ out,
                                                                 int M, int N, int K, int k_per_split, int splits) {
    extern __shared__ __attribute__((aligned(16))) unsigned char strip_lds[];   // NB fills; the exchange of the gated form
    constexpr int WM = W / 2, A_P = WM * RS, B_P = 2 * FS, P = A_P + B_P;          // 1 KB pieces of a fill: 16 rows, 16 features x 32
    constexpr int EACH = P / W, EXTRA = P % W, FILL = P * 1024, NB = strip_fills(W, RS, FS);                // a wave requests EACH of them, the first EXTRA waves one more
    const int tiles_n = (N / 2 + 16 * FS - 1) / (16 * FS);
    const int logical = xcd_remap(blockIdx.x, tiles_n * splits);
    const int sp = logical % splits, tn = logical / splits;
    const int nfill = k_per_split / 32, kslices = K / 16, ks0 = sp * (k_per_split / 16);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave >> 1, wn = wave & 1, l16 = lane & 15, lg = lane >> 4;
    const int m_pieces = 2 * ((M + 31) / 32), n_pieces = N / 16;

    // Piece i of a fill, in the lane order of the 16x16x32 operand: lane 16 g + r holds row (feature) r, elements 8 g .. 8 g + 7,
    // which lie in slice g / 2 of the packed order, half g % 2 of its 16.  Dealt to the waves as in the tall kernel.
    const uint64_t last_lanes = wave < EXTRA ? ~0ull : 1;
    const char* src[EACH + 1];
    int step[EACH + 1];
    uint32_t lane_off[EACH + 1];
#pragma unroll
    for (int q = 0; q <= EACH; ++q) {
        const int i = min(wave + W * q, P - 1);
        if (i < A_P) {
            const int x = min(i, m_pieces - 1);
            src[q] = reinterpret_cast<const char*>(Ap) + ((int64_t)(x >> 1) * kslices + ks0) * 1024 + (x & 1) * 256;
            step[q] = 2 * 1024;
        } else {
            const int j = i - A_P;                         // GLU: FS pieces of gate rows, then FS of up rows
            const int x = GLU ? (j < FS ? min(tn * FS + j, n_pieces / 2 - 1) : n_pieces / 2 + min(tn * FS + j - FS, n_pieces / 2 - 1))
                              : min(tn * 2 * FS + j, n_pieces - 1);
            src[q] = reinterpret_cast<const char*>(Wp) + ((int64_t)(x >> 3) * kslices + ks0) * 4096 + ((x >> 1) & 3) * 1024 + (x & 1) * 256;
            step[q] = 2 * 4096;
        }
        lane_off[q] = (lg >> 1) * (step[q] / 2) + (lg & 1) * 512 + l16 * 16;
    }
    const uint32_t lds_base = (uint32_t)(uintptr_t)SV_LDS_PTR(strip_lds);
    int ahead = 0;
    auto request = [&](auto which, uint32_t base) __attribute__((always_inline)) {
        constexpr int Q = decltype(which)::value;
        // pieces Q W .. Q W + W - 1, one a wave: of rows, which every strip reads, or of weights, which only this one does and which come as a
        // stream (STREAM).  Eight waves, bound by their products, do not gain (320 rows: gate/up 85.6 -> 84.1, down 53.1 -> 56.5, LM head 319 -> 323)
        constexpr bool weights = STREAM && Q * W >= A_P, mixed = STREAM && !weights && Q * W + W > A_P;
        if constexpr (Q < EACH) {
            const uint32_t to = base + (wave + W * Q) * 1024;
            if (mixed && wave + W * Q >= A_P) dma1<true>(src[Q], lane_off[Q], to);
            else dma1<weights>(src[Q], lane_off[Q], to);
        } else if constexpr (EXTRA > 0) {
            dma1_lanes<weights>(last_lanes, src[Q], lane_off[Q], base + min(wave + W * Q, P - 1) * 1024);
        }
    };
    auto advance = [&]() __attribute__((always_inline)) {  // past the end: the last fill again, so that the counts below hold
        if (++ahead < nfill) {
#pragma unroll
            for (int q = 0; q <= EACH; ++q) src[q] += step[q];
        }
    };
    auto wait_fills = [&](auto in_flight) __attribute__((always_inline)) {
        constexpr int L = decltype(in_flight)::value;
        wait_vmcnt<(EACH + (EXTRA > 0)) * L>();
    };

    u32x4 a[2][RS], b[2][FS];
    const uint32_t lds0 = lds_base + lane * 16;
    const uint32_t a_off = lds0 + wm * RS * 1024, b_off = lds0 + (A_P + wn * FS) * 1024;
    uint32_t a_addr = a_off, b_addr = b_off;
    auto read = [&](auto set, auto which) __attribute__((always_inline)) {
        constexpr int S = decltype(set)::value, R = decltype(which)::value;
        if constexpr (R < FS) lds_read16<R * 1024>(b[S][R], b_addr);
        else lds_read16<(R - FS) * 1024>(a[S][R - FS], a_addr);
    };
    auto wait_set = [&](auto set) __attribute__((always_inline)) {
        constexpr int S = decltype(set)::value;
        lds_landed(b[S][0]);
#pragma unroll
        for (int i = 1; i < FS; ++i) lds_landed_too(b[S][i]);
#pragma unroll
        for (int j = 0; j < RS; ++j) lds_landed_too(a[S][j]);
    };
    floatx4 acc[FS][RS];
#pragma unroll
    for (int i = 0; i < FS; ++i)
#pragma unroll
        for (int j = 0; j < RS; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};

    const std::integral_constant<int, 0> i0;
    const std::integral_constant<int, 1> i1;
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        static_for<EACH + 1>([&](auto q) __attribute__((always_inline)) { request(q, lds_base + i * FILL); });
        advance();
    }
    wait_fills(std::integral_constant<int, NB - 1>{});
    __builtin_amdgcn_s_barrier();
    static_for<FS + RS>([&](auto r) __attribute__((always_inline)) { read(i0, r); });
    wait_set(i0);
    int slot = 0;
    auto fill = [&](auto set) __attribute__((always_inline)) {
        constexpr int S = decltype(set)::value, NM = FS * RS, NR = FS + RS;
        // this wave holds the whole fill in registers and its share of the next one has landed; after the barrier so has everyone's,
        // and nobody reads this fill's place in the ring any more
        wait_fills(std::integral_constant<int, NB - 2>{});
        __builtin_amdgcn_s_barrier();
        const uint32_t base = lds_base + slot * FILL;
        slot = slot + 1 == NB ? 0 : slot + 1;
        a_addr = a_off + slot * FILL;
        b_addr = b_off + slot * FILL;
        __builtin_amdgcn_sched_barrier(0);
        static_for<NM>([&](auto mi) __attribute__((always_inline)) {
            constexpr int m = decltype(mi)::value, j = m / FS, i = j & 1 ? FS - 1 - m % FS : m % FS;
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, b[S][i]), __builtin_bit_cast(bf16x8, a[S][j]), acc[i][j], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            constexpr int first = m < NR ? m : NR, last = m + 1 == NM ? NR : m + 1 < NR ? m + 1 : NR;
            static_for<last - first>([&](auto rr) __attribute__((always_inline)) {
                read(std::integral_constant<int, 1 - S>{}, std::integral_constant<int, first + decltype(rr)::value>{});
                __builtin_amdgcn_sched_barrier(0);
            });
            constexpr int NQ = EACH + (EXTRA > 0), q = (m * NQ + NM - 1) / NM;      // request q after product q NM / NQ
            if constexpr (q < NQ && q * NM / NQ == m) {
                request(std::integral_constant<int, q>{}, base);
                __builtin_amdgcn_sched_barrier(0);
            }
        });
        wait_set(std::integral_constant<int, 1 - S>{});
        advance();
    };
    int f = 0;
    for (; f + 1 < nfill; f += 2) { fill(i0); fill(i1); }
    if (f < nfill) fill(i0);
    wait_vmcnt<0>();                                      // nothing of this work-group may land in LDS after it has gone

    // acc[i][j][e] <-> row 16 (RS wm + j) + l16, feature 4 lg + e of the wave's 16-feature operand i
    if (GLU) {                                            // even waves hold gate features, odd ones the same features' up halves
        constexpr int RH = (RS + 1) / 2;                  // the even wave finishes the first RH row operands, the odd one the others
        __builtin_amdgcn_s_barrier();                     // everyone's last loads have landed and last reads are over
        floatx4* xbuf = reinterpret_cast<floatx4*>(strip_lds) + wm * FS * RS * 64 + lane;
        static_for<RS>([&](auto jj) __attribute__((always_inline)) {
            constexpr int j = decltype(jj)::value;
            if ((j < RH) != (wn == 0)) {
#pragma unroll
                for (int i = 0; i < FS; ++i) xbuf[(i * RS + j) * 64] = acc[i][j];
            }
        });
        __syncthreads();
        const int F = N / 2;
        bf16_t* act = reinterpret_cast<bf16_t*>(out);
        static_for<RS>([&](auto jj) __attribute__((always_inline)) {
            constexpr int j = decltype(jj)::value;
            const int x = wm * RS + j;
            if ((j < RH) == (wn == 0) && x < m_pieces) {
#pragma unroll
                for (int i = 0; i < FS; ++i) {
                    const floatx4 other = xbuf[(i * RS + j) * 64];
                    float r[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) r[e] = j < RH ? silu_mul(acc[i][j][e], other[e]) : silu_mul(other[e], acc[i][j][e]);
                    const int fs = tn * FS + i;
                    if (fs < F / 16) {
                        u32x2* dst = reinterpret_cast<u32x2*>(act + ((int64_t)(x >> 1) * (F / 16) + fs) * 512 + ((lg >> 1) * 32 + (x & 1) * 16 + l16) * 8 + 4 * (lg & 1));
                        const u32x2 pk = {pack2bf(r[0], r[1]), pack2bf(r[2], r[3])};
                        // streamed from 33 to 160 rows (the down projection of 96 / 147 rows 36.0 -> 31.4 / 68.0 -> 60.6 us); of 320 rows it would
                        // take longer, 52.8 -> 54.8.  By the form, not by leaves_stream: with a branch here 65 to 100 rows lose 1 to 2 % of a step
                        if constexpr (W == 4 && RS > 1) store_stream(dst, pk);
                        else *dst = pk;
                    }
                }
            }
        });
        return;
    }
    float* dst = out + (int64_t)sp * M * N;
#pragma unroll
    for (int j = 0; j < RS; ++j) {
        const int m = 16 * (wm * RS + j) + l16;
        if (m < M) {
#pragma unroll
            for (int i = 0; i < FS; ++i) {
                const int n = (tn * 2 + wn) * 16 * FS + 16 * i;
                if (n < N) *reinterpret_cast<floatx4_any*>(dst + (int64_t)m * N + n + 4 * lg) = acc[i][j];
            }
        }
    }
}

// Microseconds a launch takes, fitted to 400 launches of thirteen shapes (5 to 320 rows, weights from HBM, an idle chip before each;
// rms error 10 %): a lone work-group's fills at their pace and its epilogue, the weight stream beside them -- the two add up at
// nearly twice the stream's rate rather than overlap, and never beat the stream itself.  More work-groups than CUs: in rounds where
// eight waves fill a CU, else two on a CU at 1.35 times their share of one's time (the LM head);
// 296 strips for 5 rows take 58 us where 237 take 44.  The split-K planes, written here and
// read by the consumer, cost less inside a step than their bytes at HBM's rate (they mostly meet in L2): O of the 7B shape at 160 rows
// 2.3 us less a layer in eight parts than in seven, 5.2 less than in four.
static double gemm_bf16_strip_us(int M, int N, int K, int splits, bool glu, const StripTile& s) {
    const int n = gemm_bf16_strips(N, s) * splits, area = s.tiles * s.fs, rounds = n / 256, rem = n % 256;
    const double wg = (double)K / 32 / splits * (0.062 + 0.007 * area) + 0.11 * area, stream = (double)N * K * 2.0 / 1.0e6;
    const double t = n <= 256 ? wg : s.tiles <= 5 ? wg * 1.35 * n / 256 : wg * (rounds + (rem ? 0.5 + rem / 512.0 : 0.0));
    const double planes = glu ? 0.0 : splits == 1 ? (double)M * N * 4.0 / 6.0e6 : (2 * splits - 1) * (double)M * N * 4.0 / 12.0e6;
    const double uneven = n <= 256 || s.tiles > 5 ? 1.0 : std::sqrt((rounds + (rem ? 1 : 0)) * 256.0 / n);       // CUs with one strip more than others
    return std::max(stream / 6.1, t + stream / 11.3) * uneven + planes + 2.3;
}

// The strip for M <= kStripRows rows: the lowest that holds them, width and splits by the estimate (us 1e30: none).
StripPlan gemm_bf16_strip_plan(int M, int N, int K, int min_splits, int max_splits, bool glu) {
    const int need = (M + 31) / 32, tiles = need <= 6 ? need : need <= 8 ? 8 : 10;
    StripPlan best{1, {tiles, 4}, 1e30};
    for (int fs : {4, 5, 7})
        for (int s = min_splits; s <= max_splits; ++s) {
            if (K % (64 * s) != 0) continue;               // (the form in which every kernel of a packed projection can be split)
            const double us = gemm_bf16_strip_us(M, N, K, s, glu, {tiles, fs});
            if (us < best.us) best = {s, {tiles, fs}, us};
        }
    return best;
}

// plain: out [splits][M][N] fp32, N % 128 == 0.  gated: N = 2 F weight rows, out = packed bf16 [ceil(M/32)*32, F], F % 128 == 0,
// splits == 1.  (K / splits) % 32 == 0.  One work-group holds the M rows in tiles of 32 (1 to 5, 6, 8 or 10 of them).
hipError_t gemm_bf16_strip(const bf16_t* Ap, const bf16_t* Wp, float* out, int M, int N, int K, int splits, bool glu, const StripTile& s, bool cold, hipStream_t st) {
    if (splits < 1 || K % splits != 0 || (K / splits) % 32 != 0 || N % (glu ? 256 : 128) != 0 || (glu && splits != 1) || M < 1 || M > 32 * s.tiles)
        return hipErrorInvalidValue;
    auto launch = [&](auto kern, int w, int rs, int fs) -> hipError_t {
        const int tiles_n = gemm_bf16_strips(N, s);
        const int lds = std::max(strip_fills(w, rs, fs) * (w / 2 * rs + 2 * fs) * 1024, glu ? w / 2 * rs * fs * 1024 : 0);
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kern, dim3(tiles_n * splits), dim3(64 * w), lds, st, Ap, Wp, out, M, N, K, K / splits, splits);
        return hipGetLastError();
    };
    auto width = [&](auto g, auto w, auto rs) -> hipError_t {
        constexpr bool G = decltype(g)::value;
        constexpr int W = decltype(w)::value, RS = decltype(rs)::value;
        auto form = [&](auto fs) -> hipError_t {
            constexpr int FS = decltype(fs)::value;
            if (W == 4 && cold) return launch(gemm_bf16_strip_kernel<G, W, RS, FS, W == 4>, W, RS, FS);
            return launch(gemm_bf16_strip_kernel<G, W, RS, FS, false>, W, RS, FS);
        };
        switch (s.fs) {
            case 4: return form(std::integral_constant<int, 4>{});
            case 5: return form(std::integral_constant<int, 5>{});
            case 7: return form(std::integral_constant<int, 7>{});
            default: return hipErrorInvalidValue;
        }
    };
    auto height = [&](auto g) -> hipError_t {
        constexpr std::integral_constant<int, 4> w4;
        constexpr std::integral_constant<int, 8> w8;
        switch (s.tiles) {
            case 1: return width(g, w4, std::integral_constant<int, 1>{});
            case 2: return width(g, w4, std::integral_constant<int, 2>{});
            case 3: return width(g, w4, std::integral_constant<int, 3>{});
            case 4: return width(g, w4, std::integral_constant<int, 4>{});
            case 5: return width(g, w4, std::integral_constant<int, 5>{});
            case 6: return width(g, w8, std::integral_constant<int, 3>{});
            case 8: return width(g, w8, std::integral_constant<int, 4>{});
            case 10: return width(g, w8, std::integral_constant<int, 5>{});
            default: return hipErrorInvalidValue;
        }
    };
    return glu ? height(std::true_type{}) : height(std::false_type{});
}

// Activations [M, K] row-major -> packed [ceil(M/32)][K/16][64 lanes][8]: lane 32*g + r of a fragment holds
// row 32*tile + r, elements 8*g .. 8*g+7 of the slice; rows beyond M are written as zeros.
__global__ void pack_rows_kernel(const bf16_t* __restrict__ src, bf16_t* __restrict__ dst, int M, int K) {
    const int64_t piece = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t total = (int64_t)((M + 31) / 32) * 32 * K / 8;
    if (piece >= total) return;
    const int lane = piece & 63;
    const int64_t frag = piece >> 6;
    const int ks = frag % (K / 16), mt = frag / (K / 16);
    const int row = mt * 32 + (lane & 31), col = ks * 16 + (lane >> 5) * 8;
    u32x4 v = {0, 0, 0, 0};
    if (row < M) v = *reinterpret_cast<const u32x4*>(src + (int64_t)row * K + col);
    *reinterpret_cast<u32x4*>(dst + piece * 8) = v;
}

hipError_t pack_rows(const bf16_t* src, bf16_t* dst, int M, int K, hipStream_t st) {
    const int64_t pieces = (int64_t)((M + 31) / 32) * 32 * K / 8;
    hipLaunchKernelGGL(pack_rows_kernel, dim3((unsigned)((pieces + 255) / 256)), dim3(256), 0, st, src, dst, M, K);
    return hipGetLastError();
}

template <int MT, int NT, int KA, int PD>
static hipError_t launch_ws(const bf16_t* Ap, const bf16_t* Wp, float* out, int M, int N, int K, int splits, bool cold, hipStream_t st) {
    constexpr int BM = 32 * MT, BN = 128 * NT;
    if (N % BN != 0 || (K / splits) % (16 * KA) != 0) return hipErrorInvalidValue;
    const int tiles_m = (M + BM - 1) / BM, tiles_n = N / BN;
    auto launch = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(tiles_m * tiles_n * splits), dim3(256), 0, st, Ap, Wp,
                           out, M, N, K, K / splits, splits, tiles_m, tiles_n, 0);
    };
    auto form = [&](auto stream) {
        // (a branch in the kernel makes its end twice as long: 3.65 -> 3.9 us a launch of five rows)
        if (leaves_stream(M, N < K ? N : K)) launch(gemm_bf16_ws_kernel<MT, NT, KA, PD, false, decltype(stream)::value, true>);
        else launch(gemm_bf16_ws_kernel<MT, NT, KA, PD, false, decltype(stream)::value, false>);
    };
    // one row tile: the weights are read once, as a stream (LM heads of 152 thousand features at 5 / 20 / 42 / 96 rows 193 / 122 / 207 / 219 -> 168 / 107 /
    // 190 / 202 us; QKV and O of 96 rows level).  Several row tiles share them through L2 (O of 5120 x 5120 at 800 rows, so read, 66.5 -> 72.6)
    if (tiles_m == 1 && cold) form(std::true_type{});
    else form(std::false_type{});
    return hipGetLastError();
}

// Gate/up projection fused with SwiGLU: Wp packed [2F, K] (gate rows, then up rows); act_out packed
// [ceil(M/32)*32, F] bf16.  F a multiple of 64.
hipError_t gemm_bf16_ws_glu(const bf16_t* Ap, const bf16_t* Wp, bf16_t* act_out, int M, int F, int K, hipStream_t st) {
    if (F % 64 != 0 || K % 64 != 0) return hipErrorInvalidValue;
    float* out = reinterpret_cast<float*>(act_out);
    if (F % 128 == 0 && K % 128 == 0) {
        // 128-feature strips, gate and up in one wave.  One work-group per CU: the launch runs in rounds of 256,
        // and a last round that is less than half full would leave most CUs idle for a whole work-group's time.
        // Its strips are then given to 64-row work-groups of half a strip each (five times as many, a fifth of the
        // products) at the end of the same launch.
        const int mt = gemm_bf16_ws_row_tiles(M);
        const int tiles_m = (M + 32 * mt - 1) / (32 * mt), strips = F / 128;
        const int rem = (strips * tiles_m) % 256;
        const int strips_tail = mt == 5 && rem > 0 && rem <= 128 ? (rem + tiles_m - 1) / tiles_m : 0;
        const int strips_main = strips - strips_tail;
        const int tiles_m1 = (M + 31) / 32;
        auto launch = [&](auto kern) {
            hipLaunchKernelGGL(kern, dim3(tiles_m * strips), dim3(256), 0, st, Ap, Wp, out, M, 2 * F, K, K, 1, tiles_m, strips, 0);
        };
        if (strips_tail == 0) {
            switch (mt) {
                case 1: launch(gemm_bf16_ws_kernel<1, 2, 8, 8, true>); break;
                case 2: launch(gemm_bf16_ws_kernel<2, 2, 8, 8, true>); break;
                case 3: launch(gemm_bf16_ws_kernel<3, 2, 8, 8, true>); break;
                case 4: launch(gemm_bf16_ws_kernel<4, 2, 8, 8, true>); break;
                default: launch(gemm_bf16_ws_kernel<5, 2, 8, 8, true>); break;
            }
        } else if (strips_main == 0)
            hipLaunchKernelGGL((gemm_bf16_ws_kernel<1, 2, 8, 8, true>), dim3(tiles_m1 * strips_tail), dim3(256), 0, st, Ap, Wp,
                               out, M, 2 * F, K, K, 1, tiles_m1, strips_tail, 0);
        else {
            const int tiles_m2 = (M + 63) / 64;
            hipLaunchKernelGGL(gemm_bf16_ws_glu_mixed_kernel, dim3(tiles_m * strips_main + tiles_m2 * 2 * strips_tail), dim3(256), 0,
                               st, Ap, Wp, out, M, 2 * F, K, tiles_m, strips_main, tiles_m2, strips_tail);
        }
        return hipGetLastError();
    }
    const int tiles_m = (M + 159) / 160, tiles_n = F / 64;
    if (K % 128 == 0)
        hipLaunchKernelGGL((gemm_bf16_ws_kernel<5, 1, 8, 8, true>), dim3(tiles_m * tiles_n), dim3(256), 0, st, Ap, Wp,
                           out, M, 2 * F, K, K, 1, tiles_m, tiles_n, 0);
    else
        hipLaunchKernelGGL((gemm_bf16_ws_kernel<5, 1, 4, 4, true>), dim3(tiles_m * tiles_n), dim3(256), 0, st, Ap, Wp,
                           out, M, 2 * F, K, K, 1, tiles_m, tiles_n, 0);
    return hipGetLastError();
}

// Weight-streaming projection: packed activations, packed weights.  wide: 256 features per work-group.
// 32-row tiles per work-group for M rows: as few work-groups along the rows as five tiles each allow, then no
// more tiles each than those work-groups need (320 rows: 2 x 5; 512 rows: 4 x 4; 64 rows: 1 x 2).
int gemm_bf16_ws_row_tiles(int M) {
    const int tiles = (M + 31) / 32, groups = (tiles + 4) / 5;
    return (tiles + groups - 1) / groups;
}

hipError_t gemm_bf16_ws(const bf16_t* Ap, const bf16_t* Wp, float* out, int M, int N, int K, int splits, bool wide, bool cold,
                        hipStream_t st, int row_tiles) {
    const bool long_fill = (K / splits) % 128 == 0;
    const int mt = row_tiles >= 1 && row_tiles <= 5 ? row_tiles : gemm_bf16_ws_row_tiles(M);
    if (!long_fill) {        // short fills (small models; many splits of a deep reduction at a few rows): narrow strips of
                             // one to four row tiles, else the five-tile form.  96 rows, down of the 7B shape in eight splits of
                             // 18.5 fills, cold weights: five tiles, two of them padding, 39.9 us, three 31.5.
        if (!wide && mt == 1) return launch_ws<1, 1, 4, 4>(Ap, Wp, out, M, N, K, splits, cold, st);
        if (!wide && mt == 2) return launch_ws<2, 1, 4, 4>(Ap, Wp, out, M, N, K, splits, cold, st);
        if (!wide && mt == 3) return launch_ws<3, 1, 4, 4>(Ap, Wp, out, M, N, K, splits, cold, st);
        if (!wide && mt == 4) return launch_ws<4, 1, 4, 4>(Ap, Wp, out, M, N, K, splits, cold, st);
        return wide ? launch_ws<5, 2, 4, 4>(Ap, Wp, out, M, N, K, splits, cold, st) : launch_ws<5, 1, 4, 4>(Ap, Wp, out, M, N, K, splits, cold, st);
    }
    switch (mt * 2 + (wide ? 1 : 0)) {
        case 2: return launch_ws<1, 1, 8, 8>(Ap, Wp, out, M, N, K, splits, cold, st);
        case 3: return launch_ws<1, 2, 8, 8>(Ap, Wp, out, M, N, K, splits, cold, st);
        case 4: return launch_ws<2, 1, 8, 8>(Ap, Wp, out, M, N, K, splits, cold, st);
        case 5: return launch_ws<2, 2, 8, 8>(Ap, Wp, out, M, N, K, splits, cold, st);
        case 6: return launch_ws<3, 1, 8, 8>(Ap, Wp, out, M, N, K, splits, cold, st);
        case 7: return launch_ws<3, 2, 8, 8>(Ap, Wp, out, M, N, K, splits, cold, st);
        case 8: return launch_ws<4, 1, 8, 8>(Ap, Wp, out, M, N, K, splits, cold, st);
        case 9: return launch_ws<4, 2, 8, 8>(Ap, Wp, out, M, N, K, splits, cold, st);
        case 10: return launch_ws<5, 1, 8, 8>(Ap, Wp, out, M, N, K, splits, cold, st);
        default: return launch_ws<5, 2, 8, 8>(Ap, Wp, out, M, N, K, splits, cold, st);
    }
}

// fp32 path (small models): v_mfma_f32_16x16x4_f32, operands straight from global memory.  A wave holds MT x NT tiles of
// 16 rows x 16 features; lane 16 g + r of an operand tile loads four consecutive k (4 g .. 4 g + 3) of its row r in one
// 16-byte piece and feeds them to four MFMAs, the reduction index of an MFMA being only a label as long as both operands
// agree on it.  Two groups of 16 k are in flight.  KW waves of a work-group share the reduction (each takes every KW-th group of 32 k)
// and add their tiles up in LDS; the other waves of the work-group have tiles of their own.  (With four groups of 32 k in flight, all of a
// wave's share up to K = 1024, the code is twice as long and every launch slower: 16 rows, two layers of 512 / 768 / 1024 inputs 98.1 / 118.2 /
// 140.5 us a step against 95.7 / 112.1 / 134.5, 20 rows 99.7 / 123.5 / 145.2 against 97.0 / 116.1 / 138.5.)
// What bounds it at the few rows of a small model's step is one chain of load latencies, so the reduction is spread over
// eight waves: 20 rows, K = 256..1024: 38 us with a scalar 32 x 32 tile per work-group (one FMA per 1.25 LDS reads, 24-64
// work-groups, K walked serially), 5 us now.  Many rows take 64 x 64 tiles per wave.
// And because a launch of such a step is little more than its own start (2.3 us of 4 to 6), the passes between the projections ride in
// them: NORM reads the residual rows and normalises them on the way in (every work-group adds up the squares of its rows), kF32Qkv
// rotates q and k and appends k and v to the cache on the way out, kF32Plain may add to what is there (the residual).  Two layers
// of 20 rows: norm 2.9 + QKV 4.1 + rotary 3.3 -> 5.9 us, norm 2.9 + gate/up 5.2 -> 5.6, the step of 22 launches 91 -> 76 with 15.
// kF32Glu: NT = 2, tile 0 gate rows, tile 1 the up rows of the same features (W has 2 F rows); out [M][F] = silu(gate) * up.
// kF32Qkv: NT = 2, 16 dimensions of a head and their partners half a head away.
// N, K and M are arbitrary: rows and features beyond the end read the last one and are not stored, k beyond the end counts
// as zero.
template <int MT, int NT, int KW, int WAVES, int FORM, bool VEC, bool NORM>
__global__ __launch_bounds__(64 * WAVES) void gemm_f32_kernel(const float* __restrict__ A, const float* __restrict__ W, float* __restrict__ out,
                                                              int M, int N, int K, int tiles_m, int add, F32Norm norm, RopeAppend rope) {
    constexpr int TILES = WAVES / KW;                      // wave tiles per work-group, side by side along the features
    static_assert(TILES == 1 || KW == 1, "the exchange area holds one wave tile");
    static_assert((FORM == kF32Qkv || NORM) ? KW > 1 && VEC : true, "fused forms: small tiles, whole pieces");
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane & 15, g = lane >> 4;
    const int kw = wave % KW, sub = wave / KW;
    const int m0 = (blockIdx.x % tiles_m) * 16 * MT;
    const int tn = (blockIdx.x / tiles_m) * TILES + sub;
    const int half = FORM == kF32Qkv ? rope.hd / 2 : 0, head = FORM == kF32Qkv ? 16 * tn / half : 0, dim = 16 * tn - head * half;
    const int n0 = FORM == kF32Qkv ? head * rope.hd + dim : tn * 16 * (FORM == kF32Glu ? 1 : NT);
    const float* a_row[MT];
    const float* w_row[NT];
#pragma unroll
    for (int j = 0; j < MT; ++j) a_row[j] = A + (int64_t)min(m0 + 16 * j + r, M - 1) * K;
#pragma unroll
    for (int i = 0; i < NT; ++i)
        w_row[i] = W + (int64_t)(FORM == kF32Glu ? i * N + min(n0 + r, N - 1) : FORM == kF32Qkv ? n0 + i * half + r : min(n0 + 16 * i + r, N - 1)) * K;
    floatx4 acc[NT][MT];
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int j = 0; j < MT; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    auto load = [&](const float* row, int k) {
        floatx4 v = {0.f, 0.f, 0.f, 0.f};
        if (VEC) {                                         // K % 4 == 0: a piece lies inside or outside as a whole
            if (k < K) v = *reinterpret_cast<const floatx4_any*>(row + k);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = k + e < K ? row[k + e] : 0.f;
        }
        return v;
    };
    floatx4 a[2][MT], w[2][NT], gain[2];
    auto load_group = [&](int k0) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int k = k0 + 16 * u + 4 * g;
            if (NORM) gain[u] = load(norm.gain, k);
#pragma unroll
            for (int j = 0; j < MT; ++j) a[u][j] = load(a_row[j], k);
#pragma unroll
            for (int i = 0; i < NT; ++i) w[u][i] = load(w_row[i], k);
        }
    };
    load_group(kw * 32);
    // what the wave that adds up row tile kw needs besides, requested with the rest
    const int my_row = min(m0 + 16 * kw + r, M - 1);
    floatx4 before[FORM == kF32Plain ? NT : 1], cs0, cs1;
    int slot = 0;
    if (KW > 1 && kw < MT) {
        if (FORM == kF32Plain && add) {
#pragma unroll
            for (int i = 0; i < NT; ++i)
                if (n0 + 16 * i + 4 * g + 3 < N) before[i] = *reinterpret_cast<const floatx4_any*>(out + (int64_t)my_row * N + n0 + 16 * i + 4 * g);
        }
        if (FORM == kF32Qkv) {
            const float* tab = rope.rope + ((int64_t)my_row * half + dim + 4 * g) * 2;
            cs0 = *reinterpret_cast<const floatx4*>(tab);
            cs1 = *reinterpret_cast<const floatx4*>(tab + 4);
            slot = rope.row_slot[my_row];
        }
    }
    float scale[MT];
    if (NORM) {                                           // wave w: rows w, w + KW, ... of the tile
        constexpr int EACH = 16 * MT / KW;
        __shared__ float scales[16 * MT];
        __builtin_amdgcn_sched_barrier(0);
        float ss[EACH];
#pragma unroll
        for (int i = 0; i < EACH; ++i) ss[i] = 0.f;
        for (int k = lane * 4; k < K; k += 256) {
            floatx4 x[EACH];
#pragma unroll
            for (int i = 0; i < EACH; ++i) x[i] = *reinterpret_cast<const floatx4*>(A + (int64_t)min(m0 + wave + KW * i, M - 1) * K + k);
#pragma unroll
            for (int i = 0; i < EACH; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) ss[i] = fmaf(x[i][e], x[i][e], ss[i]);
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1)
#pragma unroll
            for (int i = 0; i < EACH; ++i) ss[i] += __shfl_xor(ss[i], o);
        if (lane == 0) {
#pragma unroll
            for (int i = 0; i < EACH; ++i) scales[wave + KW * i] = 1.0f / sqrtf(ss[i] / (float)K + norm.eps);
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < MT; ++j) scale[j] = scales[16 * j + r];
    }
    for (int k0 = kw * 32; k0 < K; k0 += 32 * KW) {
        if (k0 != kw * 32) load_group(k0);
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            if (NORM) {
#pragma unroll
                for (int j = 0; j < MT; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e) a[u][j][e] = a[u][j][e] * scale[j] * gain[u][e];
            }
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int i = 0; i < NT; ++i)
#pragma unroll
                    for (int j = 0; j < MT; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[u][i][e], a[u][j][e], acc[i][j], 0, 0, 0);
        }
    }
    auto put = [&](int m, int n, floatx4 v) {              // four features of a row
        if (m >= M) return;
        float* dst = out + (int64_t)m * N + n;
        if (n + 3 < N) *reinterpret_cast<floatx4_any*>(dst) = v;
        else
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (n + e < N) dst[e] = v[e];
    };
    auto rest = [&](int m, int n) {                        // what is there, where fewer than four features are left
        floatx4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (m < M && n + e < N) v[e] = out[(int64_t)m * N + n + e];
        return v;
    };
    auto gated = [&](const floatx4& gate, const floatx4& up) {
        return floatx4{silu_mul(gate[0], up[0]), silu_mul(gate[1], up[1]), silu_mul(gate[2], up[2]), silu_mul(gate[3], up[3])};
    };
    if (KW > 1) {
        __shared__ floatx4 part[KW > 1 ? KW : 1][NT * MT][64];
#pragma unroll
        for (int i = 0; i < NT; ++i)
#pragma unroll
            for (int j = 0; j < MT; ++j) part[kw][i * MT + j][lane] = acc[i][j];
        __syncthreads();
        // wave j adds up and stores row tile j; the features that belong together stay together
        if (kw < MT) {
            const int m = m0 + 16 * kw + r;
            floatx4 s[NT];
#pragma unroll
            for (int i = 0; i < NT; ++i) {
                s[i] = part[0][i * MT + kw][lane];
#pragma unroll
                for (int q = 1; q < KW; ++q) s[i] += part[q][i * MT + kw][lane];
            }
            if (FORM == kF32Glu) {
                put(m, n0 + 4 * g, gated(s[0], s[NT - 1]));
            } else if (FORM == kF32Qkv) {
                if (m >= M) return;
                const int d = dim + 4 * g;
                const floatx4 x1 = s[0], x2 = s[NT - 1];
                if (head >= rope.Hq + rope.Hkv) {          // V as it is
                    float* pool = reinterpret_cast<float*>(rope.pool);
                    const int page = slot / rope.geom.page_size, tok = slot % rope.geom.page_size, kh = head - rope.Hq - rope.Hkv;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        pool[kv_v_index(rope.geom, rope.layer, page, kh, tok, d + e)] = x1[e];
                        pool[kv_v_index(rope.geom, rope.layer, page, kh, tok, d + half + e)] = x2[e];
                    }
                    return;
                }
                const floatx4 c = {cs0[0], cs0[2], cs1[0], cs1[2]}, sn = {cs0[1], cs0[3], cs1[1], cs1[3]};
                const floatx4 o1 = x1 * c - x2 * sn, o2 = x2 * c + x1 * sn;
                float *d1, *d2;
                if (head < rope.Hq) {
                    d1 = reinterpret_cast<float*>(rope.q_out) + ((int64_t)m * rope.Hq + head) * rope.hd + d;
                    d2 = d1 + half;
                } else {
                    float* pool = reinterpret_cast<float*>(rope.pool);
                    const int page = slot / rope.geom.page_size, tok = slot % rope.geom.page_size;
                    d1 = pool + kv_k_index(rope.geom, rope.layer, page, head - rope.Hq, tok, d);
                    d2 = pool + kv_k_index(rope.geom, rope.layer, page, head - rope.Hq, tok, d + half);
                }
                *reinterpret_cast<floatx4*>(d1) = o1;
                *reinterpret_cast<floatx4*>(d2) = o2;
            } else {
#pragma unroll
                for (int i = 0; i < NT; ++i) {
                    const int n = n0 + 16 * i + 4 * g;
                    if (add) s[i] += n + 3 < N ? before[i] : rest(m, n);
                    put(m, n, s[i]);
                }
            }
        }
        return;
    }
    // acc[i][j][e] <-> feature n0 + 16 i + 4 g + e, row m0 + 16 j + r
#pragma unroll
    for (int j = 0; j < MT; ++j) {
        const int m = m0 + 16 * j + r;
        if (FORM == kF32Glu) put(m, n0 + 4 * g, gated(acc[0][j], acc[NT - 1][j]));
        else
#pragma unroll
            for (int i = 0; i < NT; ++i) {
                const int n = n0 + 16 * i + 4 * g;
                put(m, n, add ? acc[i][j] + rest(m, n) : acc[i][j]);
            }
    }
}

// 64-row wave tiles once they make a work-group for every other CU; below that eight waves share a reduction, on tiles of 32 rows, or of 16
// while each of those has a CU to itself: half the products (a wave's 64 on K = 1024 take 1.9 us of the matrix unit) and half the
// loads of a work-group.  20 rows, K = 256 and 1024 in turn: 6.4 -> 4.9 us a launch.  Up to 16 rows always: a 32-row tile has the same
// work-groups there and rows that are not there in its second half (16 rows, feed-forward and vocabulary of nine times the inputs, 512 / 768
// inputs: 132.6 / 170.0 us a two-layer step with 32-row tiles, 127.8 / 163.5 with 16-row ones).
static bool f32_large(int M, int N, bool glu) {
    const int f = glu ? 64 : 256;
    return (long long)((M + 63) / 64) * ((N + f - 1) / f) >= 128;
}

static bool f32_low(int M, int N, int feats) { return (long long)((M + 15) / 16) * ((N + feats - 1) / feats) <= 256; }

// Where the norm and what follows QKV ride in the projection: 16-row tiles only, since every work-group goes over its rows a second time
// and more work-groups than CUs would do so in turn (without that line 256 inputs at 320 / 640 rows 154 / 230 us a two-layer step with launches
// of their own against 156 / 238 fused, 512 at 160 221 against 243).  Within it, launches of their own against fused at 1 / 5 / 10 / 16 / 20 / 32 / 48 rows: 512
// inputs 91 / 96 / 98 / 101 / 103 / 103 / 108 against 85 / 89 / 93 / 95 / 97 / 98 / 104, 768 inputs 105 / 107 / 111 / 115 / 119 / 122 / 139 against 100 / 104 / 108 /
// 112 / 117 / 120 / 136, 1024 inputs 123 / 125 / 135 / 135 / 140 / 142 / 163 against 119 / 123 / 128 / 134 / 138 / 141 / 158.  Longer rows, of which a
// work-group would read 16 one after the other, keep the launches: the gain is down to 1 us in 1024.
bool gemm_f32_fuses(int M, int N, int K, F32Form form) {
    return K % 4 == 0 && K <= 1024 && f32_low(M, N, form == kF32Qkv ? 32 : 16);
}

template <int FORM>
static hipError_t launch_f32(const float* A, const float* W, float* out, int M, int N, int K, bool add, const F32Norm& norm, const RopeAppend& rope,
                             hipStream_t st) {
    constexpr bool GLU = FORM == kF32Glu;
    auto launch = [&](auto kern, int rows, int feats, int threads) {
        const int tiles_m = (M + rows - 1) / rows, tiles_n = (N + feats - 1) / feats;
        hipLaunchKernelGGL(kern, dim3(tiles_m * tiles_n), dim3(threads), 0, st, A, W, out, M, N, K, tiles_m, add ? 1 : 0, norm, rope);
        return hipGetLastError();
    };
    constexpr int NTB = GLU ? 2 : 4, NTS = FORM == kF32Plain ? 1 : 2, FB = GLU ? 64 : 256, FS = FORM == kF32Qkv ? 32 : 16;
    const bool low = f32_low(M, N, FS);
    if (norm.gain) {
        if (!gemm_f32_fuses(M, N, K, (F32Form)FORM)) return hipErrorInvalidValue;
        return launch(gemm_f32_kernel<1, NTS, 8, 8, FORM, true, true>, 16, FS, 512);
    }
    if constexpr (FORM == kF32Qkv) return hipErrorInvalidValue;
    else {
        const bool vec = K % 4 == 0;
        if (f32_large(M, N, GLU))
            return vec ? launch(gemm_f32_kernel<4, NTB, 1, 4, FORM, true, false>, 64, FB, 256) : launch(gemm_f32_kernel<4, NTB, 1, 4, FORM, false, false>, 64, FB, 256);
        if (low || M <= 16) return vec ? launch(gemm_f32_kernel<1, NTS, 8, 8, FORM, true, false>, 16, FS, 512) : launch(gemm_f32_kernel<1, NTS, 8, 8, FORM, false, false>, 16, FS, 512);
        return vec ? launch(gemm_f32_kernel<2, NTS, 8, 8, FORM, true, false>, 32, FS, 512) : launch(gemm_f32_kernel<2, NTS, 8, 8, FORM, false, false>, 32, FS, 512);
    }
}

template <int MT, int NT, int WM, int WN>
static hipError_t launch_bf16(const bf16_t* A, const bf16_t* W, float* out, int M, int N, int K, int splits,
                              hipStream_t st) {
    constexpr int BM = 16 * MT * WM, BN = 16 * NT * WN;
    const int tiles_m = (M + BM - 1) / BM, tiles_n = N / BN;
    const size_t lds = (size_t)2 * (BM + BN) * LDS_PITCH * sizeof(bf16_t);
    auto kern = gemm_bf16_kernel<MT, NT, WM, WN>;
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    hipLaunchKernelGGL(kern, dim3(tiles_m * tiles_n * splits), dim3(64 * WM * WN), lds, st, A, W, out, M, N, K,
                       K / splits, splits, tiles_m, tiles_n);
    return hipGetLastError();
}

// dst (packed) <- src [N, K] row-major.  Packed order: [N/128][K/16][4 tiles of 32 rows][64 lanes][8],
// lane 32*g + r of a tile holding row r, elements 8*g .. 8*g+7 of the 16-wide k slice.
__global__ void pack_weight_kernel(const bf16_t* __restrict__ src, bf16_t* __restrict__ dst, int N, int K) {
    const int64_t piece = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;          // one 16-byte piece
    const int64_t total = (int64_t)N * K / 8;
    if (piece >= total) return;
    const int lane = piece & 63;
    int64_t frag = piece >> 6;
    const int within = frag & 3;
    frag >>= 2;
    const int ks = frag % (K / 16);
    const int grp = frag / (K / 16);
    const int row = (grp * 4 + within) * 32 + (lane & 31), col = ks * 16 + (lane >> 5) * 8;
    *reinterpret_cast<u32x4*>(dst + piece * 8) = *reinterpret_cast<const u32x4*>(src + (int64_t)row * K + col);
}

hipError_t pack_weight(const bf16_t* src, bf16_t* dst, int N, int K, hipStream_t st) {
    const int64_t pieces = (int64_t)N * K / 8;
    hipLaunchKernelGGL(pack_weight_kernel, dim3((unsigned)((pieces + 255) / 256)), dim3(256), 0, st, src, dst, N, K);
    return hipGetLastError();
}

int gemm_bf16_variant_ok(int variant, int N) { return variant >= 0 && variant <= 2 && N % 128 == 0; }

int gemm_bf16_shape_ok(int N, int K, int splits) {
    return N > 0 && K > 0 && splits > 0 && N % 128 == 0 && K % (BK * splits) == 0;
}

hipError_t gemm_bf16(const bf16_t* A, const bf16_t* W, float* out, int M, int N, int K, int splits, int variant,
                     hipStream_t st) {
    switch (variant) {
        case 1: return launch_bf16<2, 4, 2, 2>(A, W, out, M, N, K, splits, st);    // 64 x 128
        case 2: return launch_bf16<4, 4, 4, 2>(A, W, out, M, N, K, splits, st);    // 256 x 128, 8 waves
        default: return launch_bf16<4, 4, 2, 2>(A, W, out, M, N, K, splits, st);   // 128 x 128
    }
}

hipError_t gemm_f32(const float* A, const float* W, float* out, int M, int N, int K, bool add, const F32Norm& norm, hipStream_t st) {
    return launch_f32<kF32Plain>(A, W, out, M, N, K, add, norm, RopeAppend{}, st);
}

hipError_t gemm_f32_glu(const float* A, const float* W, float* act, int M, int F, int K, const F32Norm& norm, hipStream_t st) {
    return launch_f32<kF32Glu>(A, W, act, M, F, K, false, norm, RopeAppend{}, st);
}

hipError_t gemm_f32_qkv(const float* h, const float* W, int K, const F32Norm& norm, const RopeAppend& rope, hipStream_t st) {
    if (rope.dtype != 0 || rope.hd % 32 != 0) return hipErrorInvalidValue;
    return launch_f32<kF32Qkv>(h, W, nullptr, rope.T, (rope.Hq + 2 * rope.Hkv) * rope.hd, K, false, norm, rope, st);
}

}  // namespace sv
