// Projections of a few rows, with the passes between them in the launch: what the last requests of a rollout run.
//
// A step of up to sixteen rows is its weight stream and, between the streams, launches that are one chain of latencies each: norm, rotary and
// split-K planes are a few kilobytes, and every one of them waits for the launch before it to drain and starts from cold.  Here a
// projection takes them along: QKV and gate/up normalise the residual rows on the way in, QKV rotates and appends on the way out, O and
// down add to the residual themselves.  Six launches a layer where there were nine.
//
//   * A work-group of eight waves owns NT 16-feature operands and the whole reduction, so that no planes are left behind: wave w takes the
//     32-wide steps w, w + 8, ... of it (together the waves sweep one contiguous range of the packed weights), and the eight
//     partial tiles are added up in LDS.  Weights go from HBM straight into the operand registers, U steps of each wave in flight;
//     nothing but the rows is shared.
//   * NORM: the waves normalise the rows (M <= 8) into LDS as bf16, while the weights of the first steps are on their way: the rows and gains are
//     requested ahead of them, since loads return in order.
// The work-groups of the 7B and 32B shapes come to the number of CUs or less: 16 features of O and down (224), 16 and their rotary partners of QKV (144, 224), 5 or
// 7 times 16 gate and up features (237 and 247).  Narrower models have no gate/up of less than 64 features a work-group, 76 of them for 4864 gate features: the
// launches it replaces made no more, and with its norm it saves them 0.4 to 4 us a layer.
#include <algorithm>
#include <type_traits>
#include "common.h"
#include "kernels.h"

namespace sv {

constexpr int kFewWaves = 8;

template <int NT, int U, int FORM, bool NORM, bool STREAM, int OCC>
__global__ __launch_bounds__(64 * kFewWaves, OCC) void few_rows_kernel(const void* __restrict__ in, const bf16_t* __restrict__ Wp, void* __restrict__ out, int M,
                                                                       int N, int K, FewNorm norm, RopeAppend rope) {
    extern __shared__ __attribute__((aligned(16))) unsigned char few_lds[];        // NORM: the rows, then (all forms) the waves' tiles
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane & 15, g = lane >> 4;
    const int steps = K / 32, kslices = K / 16, n_my = (steps - wave + kFewWaves - 1) / kFewWaves;        // (K >= 256: every wave has one)
    constexpr int FS = NT / 2;
    const int half = FORM == kFewQkv ? rope.hd / 2 : 0, head = FORM == kFewQkv ? 16 * (int)blockIdx.x / half : 0, dim = 16 * (int)blockIdx.x - head * half;
    auto operand = [&](int i) {                            // 16-feature operand i of this work-group, among those of the matrix
        if (FORM == kFewQkv) return (head * rope.hd + dim + i * half) / 16;
        if (FORM == kFewGlu) return (i < FS ? 0 : N / 32) + min((int)blockIdx.x * FS + i % FS, N / 32 - 1);        // beyond the end: the last one, not stored
        return (int)blockIdx.x * NT + i;
    };
    const char* base[NT];
#pragma unroll
    for (int i = 0; i < NT; ++i) {
        const int x = operand(i);
        base[i] = reinterpret_cast<const char*>(Wp) + (int64_t)(x >> 3) * kslices * 4096 + ((x >> 1) & 3) * 1024 + (x & 1) * 256;
    }
    // lane 16 g + r of a 16x16x32 operand: row r, elements 8 g .. 8 g + 7 of the step: slice g / 2 of the packed order, half g % 2 of its 16
    const uint32_t w_lane = (g >> 1) * 4096 + (g & 1) * 512 + r * 16;
    const int row = min(r, M - 1);
    const uint32_t a_lane = (g >> 1) * 1024 + (g & 1) * 512 + row * 16;
    auto step_of = [&](int t) { return wave + kFewWaves * min(t, n_my - 1); };                            // past the end: the last one again
    u32x4 w[U][NT], a[U];
    auto load = [&](int t, auto slot) __attribute__((always_inline)) {
        constexpr int S = decltype(slot)::value;
        const int64_t s = step_of(t);
#pragma unroll
        for (int i = 0; i < NT; ++i) {
            const u32x4* p = reinterpret_cast<const u32x4*>(base[i] + s * 8192 + w_lane);
            w[S][i] = STREAM ? load_stream(p) : *p;
        }
        if (!NORM) a[S] = *reinterpret_cast<const u32x4*>(reinterpret_cast<const char*>(in) + s * 2048 + a_lane);
    };
    auto fence = []() __attribute__((always_inline)) { __builtin_amdgcn_sched_barrier(0); };

    const int pitch = K + 32;                              // elements of a normalised row in LDS
    bf16_t* rows = reinterpret_cast<bf16_t*>(few_lds);
    if (NORM) {                                            // wave w: columns 256 (w + 8 u) .. + 255 of every row
        constexpr int NU = 3;                              // K <= 256 * 8 * 3
        __shared__ float squares[kFewWaves][kFewWaves];    // [row][wave]
        const floatx4* h = reinterpret_cast<const floatx4*>(in);
        const int nq = K / 4;
        floatx4 x[NU][kFewWaves];
        float gain[NU][4];
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const int at0 = (u * kFewWaves + wave) * 64;
            if (at0 >= nq) break;
            const int at = min(at0 + lane, nq - 1);
#pragma unroll
            for (int m = 0; m < kFewWaves; ++m)
                if (m < M) x[u][m] = h[(int64_t)m * nq + at];
            Store<bf16_t>::load4(norm.gain + 4 * at, gain[u]);
        }
        fence();
        static_for<U>([&](auto u) __attribute__((always_inline)) { load(decltype(u)::value, u); });
        fence();
        float ss[kFewWaves];
#pragma unroll
        for (int m = 0; m < kFewWaves; ++m) ss[m] = 0.f;
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            if ((u * kFewWaves + wave) * 64 >= nq) break;
            if ((u * kFewWaves + wave) * 64 + lane < nq)
#pragma unroll
                for (int m = 0; m < kFewWaves; ++m)
                    if (m < M)
#pragma unroll
                        for (int e = 0; e < 4; ++e) ss[m] = fmaf(x[u][m][e], x[u][m][e], ss[m]);
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1)
#pragma unroll
            for (int m = 0; m < kFewWaves; ++m) ss[m] += __shfl_xor(ss[m], o);
        if (lane == 0)
#pragma unroll
            for (int m = 0; m < kFewWaves; ++m) squares[m][wave] = ss[m];
        __syncthreads();
#pragma unroll
        for (int m = 0; m < kFewWaves; ++m) {
            if (m >= M) break;
            float tot = 0.f;
#pragma unroll
            for (int q = 0; q < kFewWaves; ++q) tot += squares[m][q];
            const float scale = 1.0f / sqrtf(tot / (float)K + norm.eps);
#pragma unroll
            for (int u = 0; u < NU; ++u) {
                const int at = (u * kFewWaves + wave) * 64 + lane;
                if (at < nq) {
                    float o[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[e] = x[u][m][e] * scale * gain[u][e];
                    Store<bf16_t>::store4(rows + m * pitch + 4 * at, o);
                }
            }
        }
        __syncthreads();
    } else {
        static_for<U>([&](auto u) __attribute__((always_inline)) { load(decltype(u)::value, u); });
    }
    // what the waves that finish a tile need besides
    floatx4 before = {0.f, 0.f, 0.f, 0.f}, cs0 = before, cs1 = before;
    int slot_at = 0;
    if (FORM == kFewAdd && wave < NT) before = *reinterpret_cast<const floatx4*>(reinterpret_cast<const float*>(out) + (int64_t)row * N + 16 * operand(wave) + 4 * g);
    if (wave == 0) {
        if (FORM == kFewQkv) {
            const float* tab = rope.rope + ((int64_t)row * half + dim + 4 * g) * 2;
            cs0 = *reinterpret_cast<const floatx4*>(tab);
            cs1 = *reinterpret_cast<const floatx4*>(tab + 4);
            slot_at = rope.row_slot[row];
        }
    }
    floatx4 acc[NT];
#pragma unroll
    for (int i = 0; i < NT; ++i) acc[i] = floatx4{0.f, 0.f, 0.f, 0.f};
    auto multiply = [&](int t, auto slot) __attribute__((always_inline)) {
        constexpr int S = decltype(slot)::value;
        u32x4 x;
        if (NORM) x = *reinterpret_cast<const u32x4*>(rows + row * pitch + step_of(t) * 32 + 8 * g);
        else x = a[S];
#pragma unroll
        for (int i = 0; i < NT; ++i)
            acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w[S][i]), __builtin_bit_cast(bf16x8, x), acc[i], 0, 0, 0);
    };
    int t = 0;
    for (; t + U < n_my; t += U)
        static_for<U>([&](auto u) __attribute__((always_inline)) {
            fence();
            multiply(t + decltype(u)::value, u);
            fence();
            load(t + decltype(u)::value + U, u);
        });
    fence();
    static_for<U>([&](auto u) __attribute__((always_inline)) {
        if (t + decltype(u)::value < n_my) multiply(t + decltype(u)::value, u);
    });

    // acc[i][e] <-> row r, feature 4 g + e of operand i.  The eight waves' tiles are added up in their order.
    if (NORM) __syncthreads();                             // the rows have been read
    floatx4* part = reinterpret_cast<floatx4*>(few_lds);
#pragma unroll
    for (int i = 0; i < NT; ++i) part[(wave * NT + i) * 64 + lane] = acc[i];
    __syncthreads();
    auto total = [&](int i) {
        floatx4 s = part[i * 64 + lane];
#pragma unroll
        for (int q = 1; q < kFewWaves; ++q) s += part[(q * NT + i) * 64 + lane];
        return s;
    };
    if (FORM == kFewGlu) {
        const int fs = (int)blockIdx.x * FS + wave;
        if (wave < FS && fs < N / 32 && r < M) {
            const floatx4 gate = total(wave), up = total(FS + wave);
            float o[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = silu_mul(gate[e], up[e]);
            Store<bf16_t>::store4(reinterpret_cast<bf16_t*>(out) + (int64_t)fs * 512 + ((g >> 1) * 32 + r) * 8 + 4 * (g & 1), o);
        }
        return;
    }
    if (r >= M) return;
    if (FORM == kFewAdd) {
        if (wave < NT) *reinterpret_cast<floatx4*>(reinterpret_cast<float*>(out) + (int64_t)r * N + 16 * operand(wave) + 4 * g) = before + total(wave);
        return;
    }
    if (wave != 0) return;
    if (FORM == kFewQkv) {
        const floatx4 x1 = total(0), x2 = total(NT - 1);
        const int d = dim + 4 * g, page = slot_at / rope.geom.page_size, tok = slot_at % rope.geom.page_size;
        bf16_t* pool = reinterpret_cast<bf16_t*>(rope.pool);
        if (head >= rope.Hq + rope.Hkv) {                  // V as it is
            const int kh = head - rope.Hq - rope.Hkv;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                Store<bf16_t>::store(pool + kv_v_index(rope.geom, rope.layer, page, kh, tok, d + e), x1[e]);
                Store<bf16_t>::store(pool + kv_v_index(rope.geom, rope.layer, page, kh, tok, d + half + e), x2[e]);
            }
            return;
        }
        const float c[4] = {cs0[0], cs0[2], cs1[0], cs1[2]}, sn[4] = {cs0[1], cs0[3], cs1[1], cs1[3]};
        float o1[4], o2[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            o1[e] = x1[e] * c[e] - x2[e] * sn[e];
            o2[e] = x2[e] * c[e] + x1[e] * sn[e];
        }
        bf16_t *d1, *d2;
        if (head < rope.Hq) {
            d1 = reinterpret_cast<bf16_t*>(rope.q_out) + ((int64_t)r * rope.Hq + head) * rope.hd + d;
            d2 = d1 + half;
        } else {
            d1 = pool + kv_k_index(rope.geom, rope.layer, page, head - rope.Hq, tok, d);
            d2 = pool + kv_k_index(rope.geom, rope.layer, page, head - rope.Hq, tok, d + half);
        }
        Store<bf16_t>::store4(d1, o1);
        Store<bf16_t>::store4(d2, o2);
    }
}

constexpr int kFewShort = 8192;                           // reductions up to here are a handful of steps for each wave
constexpr int kFewNarrow = 2560;                          // features of fewer than 160 work-groups of 16
// can the launch that O or down replaces cut the reduction into eight parts or more?
static bool splits_well(int K) {
    for (int s = 8; s <= 16; ++s)
        if (K % (64 * s) == 0) return true;
    return false;
}
static int few_features(int F) {                          // 16-feature gate operands of a work-group; 0: with none of the widths one round of work-groups
    for (int fs : {4, 5, 7})
        if ((F / 16 + fs - 1) / fs <= 256) return fs;
    return 0;
}

// Up to eight rows, whose 16-byte pieces share a cache line, QKV and gate/up are ahead of the launches that they replace; O and down are level with theirs by
// themselves, and ahead by the planes that the next launch need not add up, which lets it normalise.  us a launch, weights from HBM, one, five and eight rows
// against the launches that they replace at five: QKV of 4608 x 3584 normalised, rotated and appended 9.5 / 10.7 / 12.0 against 4.5 + 7.4 + 4.8, of 7168 x 5120
// 14.7 / 16.3 / 17.4 against 4.8 + 13.3 + 4.7; gate/up of 37888 x 3584 43.5 / 44.5 / 45.6 against 4.5 + 43.4, of 55296 x 5120 85.7 / 87.2 / 88.0
// against 4.8 + 85.5; O of 3584 x 3584 6.1 against 6.7, of 5120 x 5120 10.7 against 10.6; down of 3584 x 18944 23.4 against 23.1, of 5120 x 27648 48.1
// against 49.3.  Nine to sixteen: QKV after a norm of its own 9.2 against 7.4 + 4.8 and O 6.7 against 6.7 (with no planes for the norm to read), but O of
// 5120 x 5120 11.7 against 10.6 and down 26.3 against 23.1 and 53.5 against 49.3.  More work-groups than CUs: no (QKV of 10240 and 15360 features, steps of
// 12 and 16 rows level to 0.6 % longer).  Steps of five rows of smaller models, whose streams are shorter: 896 wide 691 -> 566 us (12 layers), 1024 wide 630 -> 539,
// 2048 wide 537 -> 479 and 659 -> 563 (8 layers), 4096 wide 696 -> 656 (6 layers), 8192 wide 992 -> 970 (3).
// O and down of narrow models: with one CU to 16 features and the whole reduction, long reductions are bound by what a CU draws, where split-K fills
// the chip.  us a layer that the launch saves (all that it replaces; 240 shapes of 256 to 3072 features x 1024 to 24576 inputs) at five / eight / sixteen
// rows: 1024 features x 4096 inputs 2.8 / 2.1 / 1.0, x 6144 -1.0 / -1.2 / -1.5, x 8192 -1.6 / -2.3 / -2.3, x 16384 -5.5 / -5.9; 2048 x 6144 0.2 / -0.3 / -0.7,
// x 8960 -1.6 / -2.0, x 16384 -2.3 / -3.1; 512 x 10240 1.1 / 0.1, x 12288 -2.4 / -3.2; 2560 x 16384 1.0 / 0.7, and from there on -1 to 2.  Reductions that split into four
// parts at most (11008 and 4864 inputs) 4 to 7 / 3.5 to 6.5 / 2.7 at any width.
bool few_rows_ok(int M, int N, int K, FewForm form, bool norm) {
    if (M < 1 || M > 16 || K % 64 != 0 || K < 32 * kFewWaves || N % 128 != 0) return false;
    if (norm && (M > kFewWaves || K > 256 * kFewWaves * 3)) return false;
    if (form != kFewGlu && N > 256 * 32) return false;
    if (form == kFewAdd && M > kFewWaves && (K > kFewShort || N > 256 * 16)) return false;
    if (form == kFewAdd && splits_well(K) && (M > kFewWaves ? K > 4096 && N < kFewNarrow : K > 6144 && N < kFewNarrow && (K > 10240 || N > 512))) return false;
    return form != kFewGlu || few_features(N / 2) > 0;
}

template <int FORM, bool NORM, int NT, int U, int OCC>
static hipError_t launch_few(int blocks, const void* in, const bf16_t* W, void* out, int M, int N, int K, const FewNorm& norm, const RopeAppend& rope, bool cold, hipStream_t st) {
    auto launch = [&](auto kern) -> hipError_t {
        const int lds = std::max(NORM ? M * (K + 32) * 2 : 0, kFewWaves * NT * 1024);
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kern, dim3(blocks), dim3(64 * kFewWaves), lds, st, in, W, out, M, N, K, norm, rope);
        return hipGetLastError();
    };
    return cold ? launch(few_rows_kernel<NT, U, FORM, NORM, true, OCC>) : launch(few_rows_kernel<NT, U, FORM, NORM, false, OCC>);
}

hipError_t few_rows_qkv(const void* in, const bf16_t* W, int K, const FewNorm& norm, const RopeAppend& rope, bool cold, hipStream_t st) {
    const int N = (rope.Hq + 2 * rope.Hkv) * rope.hd;
    if (!few_rows_ok(rope.T, N, K, kFewQkv, norm.gain != nullptr) || rope.hd % 32 != 0) return hipErrorInvalidValue;
    return norm.gain ? launch_few<kFewQkv, true, 2, 7, 2>(N / 32, in, W, nullptr, rope.T, N, K, norm, rope, cold, st)
                     : launch_few<kFewQkv, false, 2, 7, 2>(N / 32, in, W, nullptr, rope.T, N, K, norm, rope, cold, st);
}

// Features of a work-group: 16, or 32 where those would be more work-groups than CUs (5120 features over 27648 inputs in 320 of them 57.8 us, in 160 48.3; 3584
// over 18944 in 224 23.4, in 112 33.2: a CU alone draws 36 KB a us from HBM and no more).  Steps in flight: with 7 for 12 O of 3584 inputs 7.2 -> 6.1
// us (14 steps a wave: nothing is read twice past the end), with 16 for 12 and 24 the long reductions 23.9 and 25.2 -> 23.3.
hipError_t few_rows_add(const bf16_t* act, const bf16_t* W, float* h, int M, int N, int K, bool cold, hipStream_t st) {
    if (!few_rows_ok(M, N, K, kFewAdd, false)) return hipErrorInvalidValue;
    auto launch = [&](auto nt, auto u, auto occ) {
        constexpr int NT = decltype(nt)::value;
        return launch_few<kFewAdd, false, NT, decltype(u)::value, decltype(occ)::value>(N / (16 * NT), act, W, h, M, N, K, FewNorm{}, RopeAppend{}, cold, st);
    };
    constexpr std::integral_constant<int, 1> i1;
    constexpr std::integral_constant<int, 2> i2;
    if (N <= 256 * 16) return K > kFewShort ? launch(i1, std::integral_constant<int, 16>{}, i2) : launch(i1, std::integral_constant<int, 7>{}, std::integral_constant<int, 4>{});
    return K > kFewShort ? launch(i2, std::integral_constant<int, 12>{}, i2) : launch(i2, std::integral_constant<int, 5>{}, i2);
}

hipError_t few_rows_glu(const float* h, const bf16_t* W, bf16_t* act, int M, int F, int K, const FewNorm& norm, bool cold, hipStream_t st) {
    if (!few_rows_ok(M, 2 * F, K, kFewGlu, true)) return hipErrorInvalidValue;
    const int fs = few_features(F), blocks = (F / 16 + fs - 1) / fs;
    if (fs == 4) return launch_few<kFewGlu, true, 8, 2, 2>(blocks, h, W, act, M, 2 * F, K, norm, RopeAppend{}, cold, st);
    if (fs == 5) return launch_few<kFewGlu, true, 10, 2, 2>(blocks, h, W, act, M, 2 * F, K, norm, RopeAppend{}, cold, st);
    return launch_few<kFewGlu, true, 14, 2, 2>(blocks, h, W, act, M, 2 * F, K, norm, RopeAppend{}, cold, st);
}

}  // namespace sv
