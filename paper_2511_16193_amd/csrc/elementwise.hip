// The memory-bound glue of the forward pass: row preparation (positions, cache slots, rotary table),
// embedding gather, residual-add + RMSNorm (which also sums split-K partial products), rotary embedding
// + KV append into the paged cache, SwiGLU, and dense <-> paged KV copies.
#include "common.h"
#include "kernels.h"

namespace sv {

// One group per new row t, row j of its request.  Position = L + index-in-chain, cache slot = L + j.  What every layer
// asks of a row (physical slot, where its attention partials lie) is worked out here once, so that no layer's kernel
// follows request -> sequence -> page table again.  The rotary angle pos * theta^(-2i/hd) is formed in double: at
// positions of tens of thousands a float angle is off by ~1e-3 rad, which is visible after rounding q and k to bf16.
// The row's embedding becomes the residual stream in the same launch.
template <typename E>
__global__ __launch_bounds__(256) void prep_rows_kernel(RowPrep p) {
    const int t = blockIdx.x;
    int b;
    if (p.n > 0) b = t / p.n;
    else {                                                 // requests of different sizes: exactly one holds row t
        __shared__ int owner;
        for (int i = threadIdx.x; i < p.B; i += 256) {
            const int t0 = p.req[i * kReqInts], n = p.req[i * kReqInts + 1];
            if (t >= t0 && t < t0 + n) owner = i;
        }
        __syncthreads();
        b = owner;
    }
    const int32_t* rq = p.req + b * kReqInts;
    const int j = t - rq[0], n = rq[1], seq = rq[7];
    int tok;
    if (p.tok_matrix) tok = p.tok_matrix[(int64_t)rq[8] * p.tok_ld + rq[9] + j];
    else              // (a pass over given residual rows brings no tokens at all)
        tok = !p.last_tokens ? 0 : j == 0 ? p.last_tokens[b] : p.drafts[(int64_t)b * (n - 1) + (j - 1)];
    // ids arrive in device memory from another process and cannot be checked on the host: an id outside the
    // vocabulary is embedded as the nearest valid one (the sampler rejects such a draft whatever its row yields)
    tok = min(max(tok, 0), p.vocab - 1);
    const int L = p.seq_len[seq];
    if (p.embed) {
        const E* src = reinterpret_cast<const E*>(p.embed) + (int64_t)tok * p.d;
        float* dst = p.h + (int64_t)t * p.d;
        for (int i = threadIdx.x * 4; i < p.d; i += 1024) {                  // d % 4 == 0
            const floatx4 v = {Store<E>::load(src + i), Store<E>::load(src + i + 1), Store<E>::load(src + i + 2), Store<E>::load(src + i + 3)};
            *reinterpret_cast<floatx4*>(dst + i) = v;
        }
    }
    if (threadIdx.x == 0) {
        const int slot = L + j;
        p.row_slot[t] = p.page_table[(int64_t)seq * p.max_pages_per_seq + slot / p.page_size] * p.page_size + slot % p.page_size;
        reinterpret_cast<int4*>(p.row_info)[t] = int4{seq, j, n, L};
        // pieces that start below the live end (they were cut from the host's upper bound of the length)
        const int nch = rq[3] > 1 ? min(rq[3], (L + n + rq[2] - 1) / rq[2]) : 0;
        reinterpret_cast<int4*>(p.row_part)[t] = int4{rq[4] + j * p.group, rq[5], rq[6], nch};
    }
    const int half = p.head_dim / 2;
    const int pos = L + row_index_in_chain(j, p.k);
    for (int i = threadIdx.x; i < half; i += 256) {
        const double inv_freq = pow((double)p.rope_theta, -2.0 * (double)i / (double)p.head_dim);
        double s, c;
        sincos((double)pos * inv_freq, &s, &c);
        p.rope[((int64_t)t * half + i) * 2 + 0] = (float)c;
        p.rope[((int64_t)t * half + i) * 2 + 1] = (float)s;
    }
}

// One work-group of NTH threads per row.  Each thread owns up to NV float4 pieces of the row; the loads of the residual, of
// the gain and of a batch of split-K partial products (plane order kept in the additions) are issued before the first
// use, so the row costs a few memory round trips rather than one per element.
// With `inv` set the addend is not S planes but the weighted sum of the row's top_k expert outputs
// (part = expert outputs [padded row][d], row of assignment j at inv[t*top_k + j], weight wts[t*top_k + j]),
// accumulated in slot order.
// A row's packed output is 16-byte pieces of cache lines that it shares with its neighbours: rows that follow each other go to one
// XCD, whose L2 puts the lines together (dealt round-robin, 320 rows of 3584 wrote 8.7 MiB where they hold 6.5): 320 / 2304 / 3520 rows
// 10.0 / 30.5 / 41 -> 8.7 / 24.5 / 32 us.  The residual leaves as a stream: 320 / 800 / 2304 rows 8.5 / 16.5 / 23.3 -> 8.2 / 16.1 / 22.8 us, and the
// gate/up weights of 147 rows after it 121 -> 115.
template <typename T, int NV, int NTH>
__global__ __launch_bounds__(NTH) void add_rmsnorm_kernel(float* __restrict__ h, const float* __restrict__ part, int S,
                                                          int64_t part_stride, const T* __restrict__ w,
                                                          T* __restrict__ a, int d, float eps, bool packed,
                                                          const int32_t* __restrict__ inv, const float* __restrict__ wts,
                                                          int top_k, LastRows last) {
    constexpr int U = NV == 1 ? 8 : 4;                   // planes, or expert rows, in flight
    __shared__ float red[NTH / 64];
    const int t_out = xcd_remap(blockIdx.x, gridDim.x);
    const int t = last.of ? last.of[t_out * kReqInts] + last.of[t_out * kReqInts + 1] - 1 : t_out;
    const int ta = last.dense ? t_out : t;               // row of what is added
    const bool stream = leaves_stream(gridDim.x, d);
    const int nq = d >> 2;                               // float4 pieces per row
    floatx4* hr = reinterpret_cast<floatx4*>(h + (int64_t)t * d);
    const floatx4 zero = {0.f, 0.f, 0.f, 0.f};
    floatx4 x[NV];
    float gain[NV][4];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        const int i = threadIdx.x + v * NTH;
        x[v] = i < nq ? hr[i] : zero;
        if (i < nq) Store<T>::load4(w + 4 * i, gain[v]);
    }
    if (inv) {
        floatx4 acc[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) acc[v] = zero;
        for (int j0 = 0; j0 < top_k; j0 += U) {
            floatx4 y[U][NV];
            float wj[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int j = j0 + u < top_k ? j0 + u : j0;
                wj[u] = j0 + u < top_k ? wts[(int64_t)ta * top_k + j] : 0.f;
                const floatx4* pr = reinterpret_cast<const floatx4*>(part + (int64_t)inv[(int64_t)ta * top_k + j] * d);
#pragma unroll
                for (int v = 0; v < NV; ++v) {
                    const int i = threadIdx.x + v * NTH;
                    y[u][v] = ((i < nq) & (j0 + u < top_k)) ? pr[i] : zero;
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (j0 + u < top_k) {
#pragma unroll
                    for (int v = 0; v < NV; ++v)
#pragma unroll
                        for (int e = 0; e < 4; ++e) acc[v][e] = fmaf(wj[u], y[u][v][e], acc[v][e]);
                }
        }
#pragma unroll
        for (int v = 0; v < NV; ++v) x[v] = x[v] + acc[v];
    } else {
        for (int s0 = 0; s0 < S; s0 += U) {
            floatx4 y[U][NV];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const floatx4* pr = reinterpret_cast<const floatx4*>(part + (s0 + u < S ? s0 + u : s0) * part_stride + (int64_t)ta * d);
#pragma unroll
                for (int v = 0; v < NV; ++v) {
                    const int i = threadIdx.x + v * NTH;
                    y[u][v] = ((i < nq) & (s0 + u < S)) ? pr[i] : zero;
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int v = 0; v < NV; ++v) x[v] = x[v] + y[u][v];
        }
    }
    float ss = 0.f;
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        const int i = threadIdx.x + v * NTH;
        if (i < nq) {
            if ((S > 0 || inv) && (!last.of || last.dense)) {
                if (stream) store_stream(hr + i, x[v]);
                else hr[i] = x[v];
            }
            ss = fmaf(x[v][0], x[v][0], ss);
            ss = fmaf(x[v][1], x[v][1], ss);
            ss = fmaf(x[v][2], x[v][2], ss);
            ss = fmaf(x[v][3], x[v][3], ss);
        }
    }
    ss = wave_sum(ss);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
    __syncthreads();
    float tot = red[0];
#pragma unroll
    for (int i = 1; i < NTH / 64; ++i) tot += red[i];
    const float r = 1.0f / sqrtf(tot / (float)d + eps);
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        const int i = threadIdx.x + v * NTH;
        if (i < nq) {
            float o[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = x[v][e] * r * gain[v][e];
            // four consecutive columns are contiguous in either output order
            Store<T>::store4(a + act_index(last.row0 + t_out, 4 * i, d, packed), o);
        }
    }
}

// q and k heads are rotated, k and v heads go to the row's cache slot.  Four consecutive dimensions (and their partners
// half a head away) per thread, a row spread over gridDim.y work-groups: 16-byte reads of the partial planes, four planes in
// flight, and of the rotary table, one 8- or 16-byte store per four q or K values (four consecutive dimensions of a key are
// contiguous in the cache's K tiles); V is stored transposed, one element at a time.  head_dim % 8 == 0 (it is 64 or 128).
// Rows that follow each other are a request's or a prompt's next tokens as a rule, with V elements two bytes apart: they go to one
// XCD (320 / 800 / 3520 rows 7.7 / 15.5 / 28 -> 7.1 / 14.1 / 25.5 us, writes of 800 rows 21.0 -> 12.1 MiB).
// q, whole half heads a store, is streamed as well (320 / 777 rows 7.15 / 8.45 -> 6.7 / 7.9); K's pieces of 8 bytes and V's of 2 are not.
// Five rows, eight planes: 4.8 us; with one work-group per row and the planes one after the other 10.5.
template <typename T>
__global__ __launch_bounds__(256) void rope_append_vec_kernel(RopeAppend p) {
    const int t = xcd_remap(blockIdx.x, gridDim.x);       // (an XCD by x for every y: y's features are other cache lines)
    const int hd = p.hd, half = hd / 2, upq = half / 4;   // units of four pairs per head
    const int nheads = p.Hq + 2 * p.Hkv;
    const int ncol = nheads * hd;
    const int64_t stride = (int64_t)p.T * ncol;
    const int u = blockIdx.y * 256 + threadIdx.x;
    if (u >= nheads * upq) return;
    const int slot = p.row_slot[t];
    const int page = slot / p.geom.page_size, tok = slot % p.geom.page_size;
    T* pool = reinterpret_cast<T*>(p.pool);
    const int head = u / upq, i = (u % upq) * 4;
    const float* src = p.qkv_part + (int64_t)t * ncol + head * hd + i;
    const floatx4 r0 = *reinterpret_cast<const floatx4*>(p.rope + ((int64_t)t * half + i) * 2);
    const floatx4 r1 = *reinterpret_cast<const floatx4*>(p.rope + ((int64_t)t * half + i) * 2 + 4);
    floatx4 x1 = {0.f, 0.f, 0.f, 0.f}, x2 = {0.f, 0.f, 0.f, 0.f};
    for (int s0 = 0; s0 < p.S; s0 += 4) {
        floatx4 y1[4], y2[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float* ps = src + min(s0 + q, p.S - 1) * stride;
            y1[q] = *reinterpret_cast<const floatx4*>(ps);
            y2[q] = *reinterpret_cast<const floatx4*>(ps + half);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (s0 + q < p.S) { x1 += y1[q]; x2 += y2[q]; }
    }
    if (head < p.Hq + p.Hkv) {
        const float c[4] = {r0[0], r0[2], r1[0], r1[2]}, sn[4] = {r0[1], r0[3], r1[1], r1[3]};
        float o1[4], o2[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            o1[e] = x1[e] * c[e] - x2[e] * sn[e];
            o2[e] = x2[e] * c[e] + x1[e] * sn[e];
        }
        if (head < p.Hq) {
            T* q = reinterpret_cast<T*>(p.q_out) + ((int64_t)t * p.Hq + head) * hd;
            const bool stream = leaves_stream(p.T, p.Hq * hd);
            Store<T>::stream4(q + i, o1, stream);
            Store<T>::stream4(q + i + half, o2, stream);
        } else {
            const int kh = head - p.Hq;
            Store<T>::store4(pool + kv_k_index(p.geom, p.layer, page, kh, tok, i), o1);
            Store<T>::store4(pool + kv_k_index(p.geom, p.layer, page, kh, tok, i + half), o2);
        }
    } else {
        const int kh = head - p.Hq - p.Hkv;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            Store<T>::store(pool + kv_v_index(p.geom, p.layer, page, kh, tok, i + e), x1[e]);
            Store<T>::store(pool + kv_v_index(p.geom, p.layer, page, kh, tok, i + half + e), x2[e]);
        }
    }
}

// Row-major bf16 models (packed and fp32 ones have the product in the epilogue of their gate/up projection).
__global__ __launch_bounds__(256) void swiglu_kernel(const float* __restrict__ part, int S, int64_t stride,
                                                     bf16_t* __restrict__ act, int F, bool packed) {
    const int t = blockIdx.y;
    const int f = blockIdx.x * 256 + threadIdx.x;
    if (f >= F) return;
    const float* src = part + (int64_t)t * 2 * F;
    float g = 0.f, u = 0.f;
    for (int s = 0; s < S; ++s) {
        g += src[s * stride + f];
        u += src[s * stride + F + f];
    }
    act[act_index(t, f, F, packed)] = f2bf(silu_mul(g, u));
}

template <typename T>
__global__ void kv_copy_kernel(T* pool, KvGeom g, int layer, const int32_t* __restrict__ pages, int pos0, T* k, T* v,
                               bool to_pool) {
    const int i = blockIdx.x, pos = pos0 + i;
    const int page = pages[pos / g.page_size], tok = pos % g.page_size;
    const int per = g.n_kv_heads * g.head_dim;
    for (int e = threadIdx.x; e < per; e += blockDim.x) {
        const int h = e / g.head_dim, d = e % g.head_dim;
        const int64_t ki = kv_k_index(g, layer, page, h, tok, d), vi = kv_v_index(g, layer, page, h, tok, d);
        if (to_pool) {
            pool[ki] = k[(int64_t)i * per + e];
            pool[vi] = v[(int64_t)i * per + e];
        } else {
            k[(int64_t)i * per + e] = pool[ki];
            v[(int64_t)i * per + e] = pool[vi];
        }
    }
}

__global__ void set_i32_kernel(int32_t* p, int32_t v) { *p = v; }
__global__ void add_rows_kernel(int32_t* seq_len, const int32_t* req, int B) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b < B) seq_len[req[b * kReqInts + 7]] += req[b * kReqInts + 1];
}

// ---------------------------------------------------------------- launchers ---

hipError_t prep_rows(const RowPrep& p, hipStream_t st) {
    if (p.dtype == 1) hipLaunchKernelGGL(prep_rows_kernel<bf16_t>, dim3(p.T), dim3(256), 0, st, p);
    else hipLaunchKernelGGL(prep_rows_kernel<float>, dim3(p.T), dim3(256), 0, st, p);
    return hipGetLastError();
}

constexpr int kWideNormRows = 640;

template <typename T>
static hipError_t add_rmsnorm_t(float* h, const float* part, int S, const T* w, T* a, int T_, int d, float eps, bool packed,
                                const int32_t* inv, const float* wts, int top_k, const LastRows& last, hipStream_t st) {
    const int64_t stride = (int64_t)(last.dense ? last.n : T_) * d;
    const int nq = d / 4;
    if (d % 4 != 0 || nq > 256 * 8) return hipErrorInvalidValue;
    const dim3 grid(last.of ? last.n : T_);
    auto launch = [&](auto kern, int threads) {
        hipLaunchKernelGGL(kern, grid, dim3(threads), 0, st, h, part, S, stride, w, a, d, eps, packed, inv, wts, top_k, last);
    };
    // Few rows: the more threads the fewer round trips (five rows of 896 pieces: 6.0 us with 256 threads, 4.7 with 1024).
    // Many: as few idle lanes and registers as the width allows (800 rows of 1280 pieces and four planes in flight: eight
    // pieces for each of 256 threads 31.8 us, three for each of 512 17.8).
    // In between the two are level and the line's place matters little: us of a layer's three norms, 1024 threads against 512, at
    // 160 / 320 / 480 / 640 / 800 / 1280 rows: 896 pieces 18.5 / 25.2 / 29.4 / 40.2 / 41.1 / 56.3 against 19.0 / 25.3 / 29.5 / 38.9 /
    // 37.8 / 54.0; 1280 pieces 22.5 / 32.7 / 31.4 / 50.6 / 54.1 / 72.4 against 24.0 / 32.6 / 32.3 / 51.4 / 54.2 / 73.2.
    const bool wide = (int)grid.x <= kWideNormRows;
    if (nq <= 512) launch(add_rmsnorm_kernel<T, 1, 512>, 512);
    else if (nq <= 1024 && wide) launch(add_rmsnorm_kernel<T, 1, 1024>, 1024);
    else if (nq <= 1024) launch(add_rmsnorm_kernel<T, 2, 512>, 512);
    else if (wide) launch(add_rmsnorm_kernel<T, 2, 1024>, 1024);
    else if (nq <= 1536) launch(add_rmsnorm_kernel<T, 3, 512>, 512);
    else launch(add_rmsnorm_kernel<T, 4, 512>, 512);
    return hipGetLastError();
}

hipError_t add_rmsnorm(float* h, const float* part, int S, const void* w, void* a, int dtype, int T, int d, float eps,
                       bool packed, hipStream_t st, const LastRows& last) {
    if (dtype == 1)
        return add_rmsnorm_t<bf16_t>(h, part, S, (const bf16_t*)w, (bf16_t*)a, T, d, eps, packed, nullptr, nullptr, 0, last, st);
    return add_rmsnorm_t<float>(h, part, S, (const float*)w, (float*)a, T, d, eps, packed, nullptr, nullptr, 0, last, st);
}

hipError_t add_rmsnorm_experts(float* h, const float* y, const int32_t* inv, const float* wts, int top_k, const void* w, void* a,
                               int T, int d, float eps, bool packed, hipStream_t st, const LastRows& last) {
    return add_rmsnorm_t<bf16_t>(h, y, 0, (const bf16_t*)w, (bf16_t*)a, T, d, eps, packed, inv, wts, top_k, last, st);
}

hipError_t rope_append(const RopeAppend& p, hipStream_t st) {
    if (p.hd % 8 != 0) return hipErrorInvalidValue;
    const dim3 grid(p.T, ((p.Hq + 2 * p.Hkv) * (p.hd / 8) + 255) / 256);
    if (p.dtype == 1) hipLaunchKernelGGL(rope_append_vec_kernel<bf16_t>, grid, dim3(256), 0, st, p);
    else hipLaunchKernelGGL(rope_append_vec_kernel<float>, grid, dim3(256), 0, st, p);
    return hipGetLastError();
}

hipError_t swiglu(const float* gu_part, int S, void* act, int T, int F, bool packed, hipStream_t st) {
    hipLaunchKernelGGL(swiglu_kernel, dim3((F + 255) / 256, T), dim3(256), 0, st, gu_part, S, (int64_t)T * 2 * F, (bf16_t*)act, F, packed);
    return hipGetLastError();
}

hipError_t kv_copy(void* pool, const KvGeom& geom, int layer, const int32_t* page_table_row, int pos0, int n, void* k,
                   void* v, int dtype, bool to_pool, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    if (dtype == 1)
        hipLaunchKernelGGL(kv_copy_kernel<bf16_t>, dim3(n), dim3(256), 0, st, (bf16_t*)pool, geom, layer,
                           page_table_row, pos0, (bf16_t*)k, (bf16_t*)v, to_pool);
    else
        hipLaunchKernelGGL(kv_copy_kernel<float>, dim3(n), dim3(256), 0, st, (float*)pool, geom, layer, page_table_row,
                           pos0, (float*)k, (float*)v, to_pool);
    return hipGetLastError();
}

hipError_t set_i32(int32_t* p, int32_t v, hipStream_t st) {
    hipLaunchKernelGGL(set_i32_kernel, dim3(1), dim3(1), 0, st, p, v);
    return hipGetLastError();
}

hipError_t add_rows(int32_t* seq_len, const int32_t* req, int B, hipStream_t st) {
    hipLaunchKernelGGL(add_rows_kernel, dim3((B + 63) / 64), dim3(64), 0, st, seq_len, req, B);
    return hipGetLastError();
}

}  // namespace sv
