// Shared device-side definitions for the gfx950 kernels of the verification step.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <utility>

namespace sv {

constexpr int kWave = 64;          // CDNA wavefront
constexpr int kVBlk = 32;          // keys per tile of a KV page

typedef uint16_t bf16_t;           // raw bf16 bits
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float floatx4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;

typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(2))) float floatx2;

// The same pieces at any address their elements may have, for buffers that a caller brings (logits, draft probabilities, gains,
// fp32 matrices may start anywhere inside an allocation).  Global memory takes such accesses: one wide load or store as well.
typedef floatx4 floatx4_any __attribute__((aligned(4)));
typedef u32x2 u32x2_any __attribute__((aligned(2)));

// float -> bf16, round to nearest even: gfx950's v_cvt_pk_bf16_f32.
__device__ __forceinline__ bf16_t f2bf(float f) { return __builtin_bit_cast(bf16_t, (__bf16)f); }
__device__ __forceinline__ float bf2f(bf16_t h) { return __uint_as_float(((uint32_t)h) << 16); }
__device__ __forceinline__ uint32_t pack2bf(float lo, float hi) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(floatx2{lo, hi}, bf16x2));
}

// What a launch leaves for later ones and does not read again itself, written with the non-temporal hint.  It is kept for what it measures: the
// launches that follow, streaming weights or keys, are the faster ones (down of 96 rows 36.0 -> 31.4 us).  The counters do not say why: launches
// run one by one write and read the same bytes with it and without.  For stores that fill whole 128-byte lines at once, or whole halves that are
// put together before they leave; not the pieces of 8 and 16 bytes of a packed row (the norm's operands so written: 24 -> 41 us at 2304 rows).
template <typename T> __device__ __forceinline__ void store_stream(T* p, T v) { __builtin_nontemporal_store(v, p); }
// Few rows leave little behind, and the launch that reads it, all of it one chain of latencies, does better to find it in L2 (after streamed
// planes the norm of five rows takes 4.8 us for 4.1, rotary 7.7 for 6.1).  The line is where steps are level, ordinary against streamed stores at 5 /
// 20 / 49 / 65 / 100 rows: 1024 wide, 12 layers 608 / 620 / 685 / 753 / 817 against 643 / 648 / 701 / 765 / 811 us, 2048 wide, 4 layers 286 / 299 / 346 / 378 / 408 against
// 292 / 305 / 346 / 375 / 402, 3584 wide, 3 layers 519 / 549 / 615 / 651 / 695 against 524 / 549 / 596 / 624 / 676.
__host__ __device__ __forceinline__ bool leaves_stream(int64_t rows, int width) { return rows * width >= 96 * 1024; }

// What is read once in a launch, and by one work-group only, read with the same hint (not what several work-groups share: see the kernels).
// For what comes from HBM: a pass that reads less than kCacheBytes finds it in the chip's memory-side cache, where the one before left it, and
// ordinary loads are the faster ones then ("cold" names passes that read more).  Steps of a 1024-wide model, 4 / 6 / 8 / 10 / 14 layers, 162 / 210 / 258 / 307 /
// 403 MB of weights, 5 rows: 210 / 303 / 417 / 528 / 735 us with ordinary loads, 223 / 319 / 417 / 510 / 701 streamed; 4 layers and 49 / 196 / 786 MB of
// cached keys and values (4 / 16 / 64 requests) 221 / 320 / 512 against 238 / 319 / 486.
constexpr size_t kCacheBytes = (size_t)256 << 20;
template <typename T> __device__ __forceinline__ T load_stream(const T* p) { return __builtin_nontemporal_load(p); }
constexpr int kStreamLoad = 2;                              // the same hint in the cache-policy operand of the load builtins

// Storage-type traits: T is float (fp32 model) or bf16_t (bf16 model).
template <typename T> struct Store;
template <> struct Store<float> {
    static __device__ __forceinline__ float load(const float* p) { return *p; }
    static __device__ __forceinline__ void load4(const float* p, float* v) {       // any p
        const floatx4 x = *reinterpret_cast<const floatx4_any*>(p);
        v[0] = x[0]; v[1] = x[1]; v[2] = x[2]; v[3] = x[3];
    }
    static __device__ __forceinline__ void store(float* p, float v) { *p = v; }
    static __device__ __forceinline__ void store4(float* p, const float* v) {      // p 16-byte aligned
        *reinterpret_cast<floatx4*>(p) = floatx4{v[0], v[1], v[2], v[3]};
    }
    static __device__ __forceinline__ void stream4(float* p, const float* v, bool stream) {
        if (stream) store_stream(reinterpret_cast<floatx4*>(p), floatx4{v[0], v[1], v[2], v[3]});
        else store4(p, v);
    }
};
template <> struct Store<bf16_t> {
    static __device__ __forceinline__ float load(const bf16_t* p) { return bf2f(*p); }
    static __device__ __forceinline__ void load4(const bf16_t* p, float* v) {      // any p
        const u32x2 x = *reinterpret_cast<const u32x2_any*>(p);
        v[0] = __uint_as_float(x[0] << 16); v[1] = __uint_as_float(x[0] & 0xffff0000u);
        v[2] = __uint_as_float(x[1] << 16); v[3] = __uint_as_float(x[1] & 0xffff0000u);
    }
    static __device__ __forceinline__ void store(bf16_t* p, float v) { *p = f2bf(v); }
    static __device__ __forceinline__ void store4(bf16_t* p, const float* v) {     // p 8-byte aligned
        *reinterpret_cast<u32x2*>(p) = u32x2{pack2bf(v[0], v[1]), pack2bf(v[2], v[3])};
    }
    static __device__ __forceinline__ void stream4(bf16_t* p, const float* v, bool stream) {
        if (stream) store_stream(reinterpret_cast<u32x2*>(p), u32x2{pack2bf(v[0], v[1]), pack2bf(v[2], v[3])});
        else store4(p, v);
    }
};

// ---- paged KV layout -------------------------------------------------------
// pool[layer][page][K | V][kv_head][tile of 32 keys], each tile stored in the order the 16x16x32 MFMA
// reads its operands, so that a wave fetches one operand fragment (64 lanes x 8 elements) as one
// contiguous, fully used 1 KB (bf16) piece:
//   K tile: fragments [key block kb = 0,1][head_dim slice kk = 0 .. hd/32-1], fragment element
//           (lane = 16*g + r, e) = K[key 16*kb + r][dim 32*kk + 8*g + e]
//   V tile: fragments [ht = 0 .. hd/16-1], fragment element (lane = 16*g + r, j) = V[key][dim 16*ht + r]
//           with key = 4*g + j for j < 4 and 16 + 4*g + (j-4) otherwise -- the order in which the
//           score tile leaves the MFMA (a lane holds 4 consecutive keys of each 16-key block).
struct KvGeom {
    int n_kv_heads, head_dim, page_size;
    int64_t page_elems;    // 2 * n_kv_heads * page_size * head_dim
    int64_t layer_elems;   // num_pages * page_elems
};
__host__ __device__ __forceinline__ int64_t kv_k_index(const KvGeom& g, int layer, int page, int head, int tok, int dim) {
    const int t = tok % kVBlk, kb = t / 16, r = t % 16;
    const int kk = dim / 32, grp = (dim % 32) / 8, e = dim % 8;
    return (int64_t)layer * g.layer_elems + (int64_t)page * g.page_elems +
           ((int64_t)head * g.page_size + (tok / kVBlk) * kVBlk) * g.head_dim +
           ((kb * (g.head_dim / 32) + kk) * 64 + grp * 16 + r) * 8 + e;
}
__host__ __device__ __forceinline__ int64_t kv_v_index(const KvGeom& g, int layer, int page, int head, int tok, int dim) {
    const int t = tok % kVBlk, half = t / 16, grp = (t % 16) / 4, j = half * 4 + t % 4;
    const int ht = dim / 16, r = dim % 16;
    return (int64_t)layer * g.layer_elems + (int64_t)page * g.page_elems +
           (int64_t)g.n_kv_heads * g.page_size * g.head_dim +
           ((int64_t)head * g.page_size + (tok / kVBlk) * kVBlk) * g.head_dim +
           ((ht * 64) + grp * 16 + r) * 8 + j;
}

// Activations that feed a projection, [rows, K]: row-major, or (packed) in the fragment order the
// weight-streaming kernel reads -- [rows/32][K/16][64 lanes][8], lane 32*g + r of a fragment holding row r of
// the 32-row tile, elements 8*g .. 8*g+7 of the 16-wide slice.
__host__ __device__ __forceinline__ int64_t act_index(int row, int col, int K, bool packed) {
    if (!packed) return (int64_t)row * K + col;
    return ((((int64_t)(row >> 5) * (K >> 4) + (col >> 4)) * 64) + ((col >> 3) & 1) * 32 + (row & 31)) * 8 + (col & 7);
}

// Index of new row j (0 = x0, then chain 0's drafts, chain 1's ...) -> chain, index in chain.
__host__ __device__ __forceinline__ int row_chain(int j, int k) { return j == 0 ? -1 : (j - 1) / k; }
__host__ __device__ __forceinline__ int row_index_in_chain(int j, int k) { return j == 0 ? 0 : (j - 1) % k + 1; }
// Does new row i attend new row j?  (x0, and the earlier drafts of its own chain.)
__host__ __device__ __forceinline__ bool row_sees(int i, int j, int k) {
    if (j == 0) return true;
    if (i == 0) return false;
    return (i - 1) / k == (j - 1) / k && j <= i;
}

// ---- waits and direct-to-LDS loads ----
#define SV_LDS_PTR(p) ((__attribute__((address_space(3))) void*)(p))

// s_waitcnt immediates (gfx9 encoding: vmcnt in bits 3:0 and 15:14, expcnt 6:4, lgkmcnt 11:8; all-ones = no wait)
template <int N> __device__ __forceinline__ void wait_vmcnt() {
    __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}

// LDS reads placed by hand, with hand-placed waits: the compiler would wait for every request that is in flight into LDS before a read of
// it.  It takes the registers as written at once, so what is read is waited for in the basic block that reads it (a branch in between may
// copy registers still in flight).
template <int OFF> __device__ __forceinline__ void lds_read16(u32x4& d, uint32_t addr) {
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(d) : "v"(addr), "n"(OFF));
}
__device__ __forceinline__ void lds_landed(u32x4& d) { asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(d)); }
__device__ __forceinline__ void lds_landed_too(u32x4& d) { asm volatile("" : "+v"(d)); }     // no use of d moves above the wait

// 1 KB from global memory straight into LDS: lane l's 16 bytes at base + lane_off go to LDS address lds + 16 l (base and lds the same for
// all lanes).  dma1_lanes: only the lanes of a mask that is not empty.
// Both write m0, and the second exec: reserved registers, which the compiler takes no clobber for.  So they are for kernels in which
// nothing else uses m0 (no builtin that loads into LDS, whose m0 the compiler may carry from one to the next), and dma1_lanes for places
// that all 64 lanes of the wave reach: exec is all ones before it and after it.
// STREAM: with the hint of load_stream.
template <bool STREAM = false>
__device__ __forceinline__ void dma1(const char* base, uint32_t lane_off, uint32_t lds) {
    if constexpr (STREAM) asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt" : : "s"(lds), "v"(lane_off), "s"(base) : "memory");
    else asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(lds), "v"(lane_off), "s"(base) : "memory");
}
template <bool STREAM = false>
__device__ __forceinline__ void dma1_lanes(uint64_t lanes, const char* base, uint32_t lane_off, uint32_t lds) {
    if constexpr (STREAM)
        asm volatile("s_mov_b32 m0, %0\n\ts_mov_b64 exec, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt\n\ts_mov_b64 exec, -1"
                     : : "s"(lds), "v"(lane_off), "s"(base), "s"(lanes) : "memory");
    else
        asm volatile("s_mov_b32 m0, %0\n\ts_mov_b64 exec, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2\n\ts_mov_b64 exec, -1"
                     : : "s"(lds), "v"(lane_off), "s"(base), "s"(lanes) : "memory");
}

// KB F (0 to 3) of 4 KB that lie together on both sides, in order: the first sets m0, the others add their offset to it and to base.
template <int F, bool STREAM = false>
__device__ __forceinline__ void dma_piece(const char* base, uint32_t lane_off, uint32_t lds) {
    if constexpr (F == 0) dma1<STREAM>(base, lane_off, lds);
    else if constexpr (STREAM) asm volatile("global_load_lds_dwordx4 %0, %1 offset:%2 nt" : : "v"(lane_off), "s"(base), "n"(F * 1024) : "memory");
    else asm volatile("global_load_lds_dwordx4 %0, %1 offset:%2" : : "v"(lane_off), "s"(base), "n"(F * 1024) : "memory");
}
// 16 bytes per lane from base + lane_off + off, off the same for all lanes, through a buffer descriptor over [base, base + bytes).
// base: the same for all lanes.  The caller keeps off inside the range: only lane_off is checked against it.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void* base, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, bytes, 0x00020000);
}
template <int POLICY = 0>
__device__ __forceinline__ u32x4 buffer_load16(__amdgpu_buffer_rsrc_t d, uint32_t lane_off, uint32_t off) {
    return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(d, lane_off, off, POLICY));
}

// f(std::integral_constant<int, 0>{}), ... , f(std::integral_constant<int, N - 1>{}): a loop whose index is a constant expression
template <typename F, int... I> __device__ __forceinline__ void static_for_each(F f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F> __device__ __forceinline__ void static_for(F f) { static_for_each(f, std::make_integer_sequence<int, N>{}); }

// Work-groups are dealt to the 8 XCDs round-robin by id.  Give XCD x a contiguous range of logical
// ids instead, so that neighbours in logical order share an L2.
__device__ __forceinline__ int xcd_remap(int id, int n) {
    const int q = n >> 3, r = n & 7;
    const int x = id & 7, local = id >> 3;
    return x * q + (x < r ? x : r) + local;
}

// silu(g) * u = g / (1 + e^-g) * u.  Bounded by the vector ALU in the gated projections' epilogues, where it is all that a CU does:
// the library's exponential and division, each correct from the smallest to the largest float, take some 45 issue slots, this 24.
// e^-g = 2^n 2^f: the product of -g and log2 e in two parts (log2 e rounded to 24 bits, and what that leaves out), n its nearest whole
// number, f the rest; clamped instead of selected beyond the range of floats.  The quotient g r from the hardware's reciprocal r, then
// one Newton step q + (g - d q) r.  Both sides are scaled by 1/4, so that the reciprocal of a large denominator is no denormal.  Against 64
// bits on normal gates and ones over [-20, 20]: 0.63 (largest 2.8) units of 2^-24, as g / (1.0f + expf(-g)) * u gives.
__device__ __forceinline__ float silu_mul(float g, float u) {
    const float t = __builtin_amdgcn_fmed3f(g * -1.44269504088896340736f, -150.0f, 150.0f);
    const float rest = __builtin_fmaf(g, -1.92596299e-8f, __builtin_fmaf(g, -1.44269504088896340736f, -t));
    const float n = __builtin_rintf(t);
    const float d = 0.25f + __builtin_amdgcn_ldexpf(__builtin_amdgcn_exp2f((t - n) + rest), (int)n - 2);
    const float r = __builtin_amdgcn_rcpf(d), g4 = 0.25f * g, q = g4 * r;
    return __builtin_amdgcn_div_fixupf(__builtin_fmaf(__builtin_fmaf(-d, q, g4), r, q), d, g4) * u;
}

template <typename T> __device__ __forceinline__ T wave_max(T v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) { T w = __shfl_xor(v, o); v = w > v ? w : v; }
    return v;
}
template <typename T> __device__ __forceinline__ T wave_sum(T v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// Largest of 64 lanes' unsigned values, in all lanes: six DPP steps (within rows of 16 lanes, then across rows) and a read of
// lane 63, no LDS-crossbar latency on the way.
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, true));            // row_shr:1
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, true));            // row_shr:2
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, true));            // row_shr:4
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, true));            // row_shr:8
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x142, 0xa, 0xf, false));      // row_bcast:15
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x143, 0xc, 0xf, false));      // row_bcast:31
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

}  // namespace sv
