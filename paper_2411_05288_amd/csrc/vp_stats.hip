// Small bandwidth/latency-bound kernels around the GEMMs: softmax statistics, their folds
// (barrier C1 of Algorithm 1), and the D = softmax - G matrix of pass T from stored logits.
#include <type_traits>

#include "vp_internal.h"

namespace vp {

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    return v;
}
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Block-wide reductions over 256 threads with a fixed tree (deterministic).
__device__ __forceinline__ float block_max256(float v, float* sh) {
    v = wave_max(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    return fmaxf(fmaxf(sh[0], sh[1]), fmaxf(sh[2], sh[3]));
}
__device__ __forceinline__ float block_sum256(float v, float* sh) {
    v = wave_sum(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    return (sh[0] + sh[1]) + (sh[2] + sh[3]);
}

// fp32 path, pass S statistics of the shards from their stored logits: one workgroup per row and shard (blockIdx.y).  Bound by
// reading Y: rows of up to 1024 C values stay in registers (C chunks of four per thread) between the maximum and the sum, longer
// ones (C = 0) are read twice.  Rows start at any element (16-byte loads at 4-byte alignment).  N=1000, 8 shards of 4000 values,
// 131 MB: 55 us with two passes of 4-byte loads and the target logit fetched at the end -> 24 (5.5 TB/s); N=128, 2 of 4096:
// 7.8 -> 4.0; N=100, 2 of 30000: 50 -> 22.
template <int C>
__global__ __launch_bounds__(256) void row_stats_f32_kernel(ShardList l, const int64_t* __restrict__ labels, int N,
                                                            float* lmax, float* lsum, float* ltgt) {
    typedef float ua4 __attribute__((ext_vector_type(4), aligned(4)));
    __shared__ float sh[4];
    const int i = blockIdx.x, r = blockIdx.y, Vs = l.rows[r];
    const float* __restrict__ y = (const float*)l.Y[r] + (int64_t)i * l.ldy[r];
    const int64_t loc = labels[i] - l.offset[r];
    const float target = loc >= 0 && loc < Vs ? y[loc] : 0.f;
    auto chunk = [&](int q) {      // columns past the end: -inf, which adds nothing
        const int j = (q * 256 + (int)threadIdx.x) * 4;
        ua4 v = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
        if (j + 4 <= Vs) {
            v = *reinterpret_cast<const ua4*>(y + j);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (j + e < Vs) v[e] = y[j + e];
        }
        return v;
    };
    auto top = [](const ua4& v) { return fmaxf(fmaxf(v[0], v[1]), fmaxf(v[2], v[3])); };
    auto add = [](float s, const ua4& v, float m) {
#pragma unroll
        for (int e = 0; e < 4; ++e) s += expf(v[e] - m);
        return s;
    };
    float m = -INFINITY, s = 0.f;
    if constexpr (C > 0) {
        ua4 v[C];
#pragma unroll
        for (int q = 0; q < C; ++q) v[q] = chunk(q);
#pragma unroll
        for (int q = 0; q < C; ++q) m = fmaxf(m, top(v[q]));
        m = block_max256(m, sh);
#pragma unroll
        for (int q = 0; q < C; ++q) s = add(s, v[q], m);
    } else {
        const int chunks = (Vs + 1023) / 1024;
        for (int q = 0; q < chunks; ++q) m = fmaxf(m, top(chunk(q)));
        m = block_max256(m, sh);
        for (int q = 0; q < chunks; ++q) s = add(s, chunk(q), m);
    }
    s = block_sum256(s, sh);
    if (threadIdx.x == 0) {
        const size_t o = (size_t)r * N + i;
        lmax[o] = m;
        lsum[o] = s;
        ltgt[o] = target;
    }
}

hipError_t launch_row_stats_f32(const ShardList& l, const int64_t* labels, int N, float* lmax, float* lsum, float* ltgt,
                                hipStream_t st) {
    ProfScope prof(K_ROWSTATS_F32, st);
    int longest = 0;
    for (int r = 0; r < l.n; ++r) longest = l.rows[r] > longest ? l.rows[r] : longest;
#define VP_STATS(C) hipLaunchKernelGGL(row_stats_f32_kernel<C>, dim3(N, l.n), dim3(256), 0, st, l, labels, N, lmax, lsum, ltgt)
    if (longest <= 1024) VP_STATS(1);
    else if (longest <= 2048) VP_STATS(2);
    else if (longest <= 4096) VP_STATS(4);
    else if (longest <= 8192) VP_STATS(8);
    else VP_STATS(0);
#undef VP_STATS
    return hipGetLastError();
}

// Fold of the per-column-tile partial (max, sum-exp) pairs of one shard with the same online
// rescaling as the cross-shard fold.  A workgroup folds 64 token rows; wavefront g takes the
// tiles congruent to g mod 4 (independent loads, several in flight), and the four partial
// results meet in LDS in the fixed order g = 0..3.  blockIdx.y is the shard.
__global__ __launch_bounds__(256) void fold_partials_kernel(const float* __restrict__ pm, const float* __restrict__ ps,
                                                            const float* __restrict__ pt, ShardList l, int N,
                                                            const int64_t* __restrict__ labels,
                                                            float* lmax, float* lsum, float* ltgt) {
    const int sh = blockIdx.y;
    const int tiles = l.first[sh + 1] - l.first[sh], Vs = l.rows[sh];
    const int64_t off = l.offset[sh];
    pm += (size_t)l.first[sh] * N;
    ps += (size_t)l.first[sh] * N;
    pt += (size_t)sh * N;
    lmax += (size_t)sh * N;
    lsum += (size_t)sh * N;
    ltgt += (size_t)sh * N;
    __shared__ float xm[4][64], xs[4][64];
    const int g = threadIdx.x >> 6, r = threadIdx.x & 63;
    const int i = blockIdx.x * 64 + r;
    const int ic = i < N ? i : N - 1;
    float m = -INFINITY, s = 0.f;
    int t = g;
    for (; t + 12 < tiles; t += 16) {
        float a[4], b[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            a[u] = pm[(size_t)(t + 4 * u) * N + ic];
            b[u] = ps[(size_t)(t + 4 * u) * N + ic];
        }
        const float mn = fmaxf(fmaxf(fmaxf(a[0], a[1]), fmaxf(a[2], a[3])), m);
        s *= __expf(m - mn);          // m = -inf only while s = 0: exp(-inf) = 0
#pragma unroll
        for (int u = 0; u < 4; ++u) s += b[u] * __expf(a[u] - mn);
        m = mn;
    }
    for (; t < tiles; t += 4) {
        const float a = pm[(size_t)t * N + ic], b = ps[(size_t)t * N + ic];
        const float mn = fmaxf(a, m);
        s = s * __expf(m - mn) + b * __expf(a - mn);
        m = mn;
    }
    xm[g][r] = m;
    xs[g][r] = s;
    __syncthreads();
    if (g == 0 && i < N) {
        float mm = fmaxf(fmaxf(xm[0][r], xm[1][r]), fmaxf(xm[2][r], xm[3][r]));
        float ss = 0.f;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (xm[q][r] > -INFINITY) ss += xs[q][r] * __expf(xm[q][r] - mm);
        lmax[i] = mm;
        lsum[i] = ss;
        const int64_t loc = labels[i] - off;
        ltgt[i] = (loc >= 0 && loc < Vs) ? pt[i] : 0.f;
    }
}

hipError_t launch_fold_partials(const float* pm, const float* ps, const float* pt, const ShardList& l, int N,
                                const int64_t* labels, float* lmax, float* lsum, float* ltgt, hipStream_t st) {
    ProfScope prof(K_FOLD, st);
    hipLaunchKernelGGL(fold_partials_kernel, dim3((unsigned)ceil_div(N, 64), l.n), dim3(256), 0, st, pm, ps, pt, l, N, labels,
                       lmax, lsum, ltgt);
    return hipGetLastError();
}

// C_r (+)= the sum of the S partials of output r (blockIdx.y; elements V).  Bound by reading them.  A small matrix has few
// threads, so a long list of slices would be a serial chain of loads: G groups of 256 / G threads take an equal share of the
// slices each, in ascending order and four loads at a time, and the groups' sums are added in ascending order.  64 slices of
// 128 x 256: 16.8 us with one thread per element, 4.1 us with G = 4; with a thread for every lane of the chip (8 slices and
// more of 512 x 2048) G = 1 is the better one, 12.3 against 15.6 us.  One output alone (List = SumOne) needs no second read
// of the argument block at an address that hangs on blockIdx: 0.8 us of a step of N=128 h=256 V=8192.
struct SumOne {
    int64_t count;
    float* C;
};
template <typename V, int G, typename List>
__global__ __launch_bounds__(256) void sum_slices_kernel(const V* __restrict__ part, int S, int64_t stride, List list,
                                                         int accumulate) {
    constexpr int W = 256 / G;
    constexpr int E = sizeof(V) / sizeof(float);
    int64_t n;
    V* C;
    if constexpr (std::is_same<List, SumOne>::value) {
        n = list.count / E;
        C = (V*)list.C;
    } else {
        n = list.count[blockIdx.y] / E;
        C = (V*)list.C[blockIdx.y];
        part += list.first[blockIdx.y] / E;
    }
    stride /= E;
    const int g = threadIdx.x / W, l = threadIdx.x % W;
    const int64_t t = (int64_t)blockIdx.x * W + l;
    const int q = (S + G - 1) / G, z1 = min(S, (g + 1) * q);
    int z = min(S, g * q);
    V acc = {};
    if (t < n) {
        for (; z + 4 <= z1; z += 4) {
            V v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = part[(int64_t)(z + u) * stride + t];
#pragma unroll
            for (int u = 0; u < 4; ++u) acc += v[u];
        }
        for (; z < z1; ++z) acc += part[(int64_t)z * stride + t];
    }
    if constexpr (G > 1) {
        __shared__ V sh[G - 1][W];
        if (g > 0) sh[g - 1][l] = acc;
        __syncthreads();
        if (g > 0) return;
        for (int u = 0; u < G - 1; ++u) acc += sh[u][l];
    }
    if (t < n) C[t] = accumulate ? C[t] + acc : acc;
}

template <typename V, typename List>
static hipError_t launch_sum_slices_t(const float* part, int S, int64_t stride, const List& l, int n, int64_t longest,
                                      int64_t all, bool accumulate, hipStream_t st) {
    const int64_t E = sizeof(V) / sizeof(float);
    if (all / E >= 65536)
        hipLaunchKernelGGL((sum_slices_kernel<V, 1, List>), dim3((unsigned)ceil_div(longest / E, 256), n), dim3(256), 0, st,
                           (const V*)part, S, stride, l, accumulate ? 1 : 0);
    else
        hipLaunchKernelGGL((sum_slices_kernel<V, 4, List>), dim3((unsigned)ceil_div(longest / E, 64), n), dim3(256), 0, st,
                           (const V*)part, S, stride, l, accumulate ? 1 : 0);
    return hipGetLastError();
}

typedef float sum4 __attribute__((ext_vector_type(4)));

hipError_t launch_sum_slices(const float* part, int S, int64_t stride, const SumList& l, bool accumulate, hipStream_t st) {
    if (l.n == 1 && l.first[0] == 0 && l.count[0] == stride) return launch_sum_slices(part, S, stride, l.C[0], accumulate, st);
    bool vec = stride % 4 == 0 && ((uintptr_t)part & 15u) == 0;
    int64_t longest = 0, all = 0;
    for (int r = 0; r < l.n; ++r) {
        vec = vec && l.first[r] % 4 == 0 && l.count[r] % 4 == 0 && ((uintptr_t)l.C[r] & 15u) == 0;
        longest = l.count[r] > longest ? l.count[r] : longest;
        all += l.count[r];
    }
    return vec ? launch_sum_slices_t<sum4>(part, S, stride, l, l.n, longest, all, accumulate, st)
               : launch_sum_slices_t<float>(part, S, stride, l, l.n, longest, all, accumulate, st);
}

hipError_t launch_sum_slices(const float* part, int S, int64_t MN, float* C, bool accumulate, hipStream_t st) {
    const SumOne l{MN, C};
    return MN % 4 == 0 && ((((uintptr_t)part) | ((uintptr_t)C)) & 15u) == 0
               ? launch_sum_slices_t<sum4>(part, S, MN, l, 1, MN, MN, accumulate, st)
               : launch_sum_slices_t<float>(part, S, MN, l, 1, MN, MN, accumulate, st);
}

// Barrier C1 of one token row: global max, rescaled sum, loss.
__device__ __forceinline__ float combine_row(const float* __restrict__ lmax, const float* __restrict__ lsum,
                                             const float* __restrict__ ltgt, int p, int N, int i, float* gmax, float* gsum,
                                             float* loss_row) {
    float m = -INFINITY;
    for (int r = 0; r < p; ++r) m = fmaxf(m, lmax[(size_t)r * N + i]);
    float s = 0.f, t = 0.f;
    for (int r = 0; r < p; ++r) {
        s += lsum[(size_t)r * N + i] * expf(lmax[(size_t)r * N + i] - m);
        t += ltgt[(size_t)r * N + i];
    }
    gmax[i] = m;
    gsum[i] = s;
    const float loss = m + logf(s) - t;
    if (loss_row) loss_row[i] = loss;
    return loss;
}

// One thread per token row; the mean loss is reduced by a single-workgroup kernel with a fixed tree: a second launch, or
// this one where a workgroup holds all rows (N <= 1024: one launch less of a pass that is launches and latency).
__global__ __launch_bounds__(256) void combine_rows_kernel(const float* __restrict__ lmax, const float* __restrict__ lsum,
                                                           const float* __restrict__ ltgt, int p, int N, float* gmax,
                                                           float* gsum, float* loss_row) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= N) return;
    combine_row(lmax, lsum, ltgt, p, N, i, gmax, gsum, loss_row);
}

// Sum of the threads' values / N; 1024 threads
__device__ __forceinline__ void mean_of_block(float acc, int N, float* out) {
    __shared__ float sh[16];
    acc = wave_sum(acc);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        float s = 0.f;
        for (int w = 0; w < 16; ++w) s += sh[w];
        out[0] = s / (float)N;
    }
}

__global__ __launch_bounds__(1024) void combine_small_kernel(const float* __restrict__ lmax, const float* __restrict__ lsum,
                                                             const float* __restrict__ ltgt, int p, int N, float* gmax,
                                                             float* gsum, float* loss_row, float* out) {
    const int i = threadIdx.x;
    float acc = 0.f;
    if (i < N) acc += combine_row(lmax, lsum, ltgt, p, N, i, gmax, gsum, loss_row);
    mean_of_block(acc, N, out);
}

// Mean loss over the N rows by one workgroup: thread t sums rows t, t+1024, ... in order, then
// a fixed tree over the 1024 threads.  The per-row losses are read if the caller keeps them (N=4096, p=8: 11.5 us when
// every row is computed again from p targets), else computed again from the global statistics.
__global__ __launch_bounds__(1024) void mean_loss_kernel(const float* __restrict__ gmax, const float* __restrict__ gsum,
                                                         const float* __restrict__ ltgt, const float* __restrict__ loss_row,
                                                         int p, int N, float* out) {
    float acc = 0.f;
    if (loss_row) {
        for (int i = threadIdx.x; i < N; i += 1024) acc += loss_row[i];
    } else {
        for (int i = threadIdx.x; i < N; i += 1024) {
            float t = 0.f;
            for (int r = 0; r < p; ++r) t += ltgt[(size_t)r * N + i];
            acc += gmax[i] + logf(gsum[i]) - t;
        }
    }
    mean_of_block(acc, N, out);
}

hipError_t launch_combine(const float* lmax, const float* lsum, const float* ltgt, int p, int N, float* gmax,
                          float* gsum, float* loss_row, float* loss_mean, hipStream_t st) {
    ProfScope prof(K_COMBINE, st);
    if (N <= 1024) {
        hipLaunchKernelGGL(combine_small_kernel, dim3(1), dim3(1024), 0, st, lmax, lsum, ltgt, p, N, gmax, gsum, loss_row,
                           loss_mean);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(combine_rows_kernel, dim3((unsigned)ceil_div(N, 256)), dim3(256), 0, st, lmax, lsum, ltgt, p, N,
                       gmax, gsum, loss_row);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(mean_loss_kernel, dim3(1), dim3(1024), 0, st, gmax, gsum, ltgt, loss_row, p, N, loss_mean);
    return hipGetLastError();
}

// D = (exp(Y - m)/sum - G) * scale from stored logits (pass T of Algorithm 1 written with
// the rescale identity of section 4.3 folded in: softmax' * sum' e^{m'-m} / sum = e^{Y-m}/sum).
template <typename T>
__device__ __forceinline__ float ld_as_f32(const T* p);
template <>
__device__ __forceinline__ float ld_as_f32<float>(const float* p) { return *p; }
template <>
__device__ __forceinline__ float ld_as_f32<u16>(const u16* p) { return __uint_as_float((unsigned)(*p) << 16); }

__device__ __forceinline__ void st_from_f32(float* p, float v) { *p = v; }
__device__ __forceinline__ void st_from_f32(u16* p, float v) {
    __bf16 b = (__bf16)v;
    *p = __builtin_bit_cast(u16, b);
}

template <typename T, bool PRECISE>
__global__ __launch_bounds__(256) void dlogits_kernel(const T* Y, T* D,   // may alias (in place)
                                                      const int64_t* __restrict__ labels, int64_t off,
                                                      const float* __restrict__ gmax, const float* __restrict__ gsum,
                                                      float scale, int Vs, int64_t ldy, int64_t ldd) {
    const int i = blockIdx.y;
    const float m = gmax[i];
    const float inv = 1.0f / gsum[i];
    const int64_t loc = labels ? labels[i] - off : (int64_t)-1;
    const T* y = Y + (int64_t)i * ldy;
    T* d = D + (int64_t)i * ldd;
    for (int j = blockIdx.x * 256 + threadIdx.x; j < ldd; j += gridDim.x * 256) {
        if (j >= Vs) {   // padding of the row: zero, because the dH product multiplies it by zero
            st_from_f32(d + j, 0.f);
            continue;
        }
        const float v = ld_as_f32<T>(y + j) - m;
        float pr = (PRECISE ? expf(v) : __expf(v)) * inv;
        if ((int64_t)j == loc) pr -= 1.0f;
        st_from_f32(d + j, pr * scale);
    }
}

// Vector form: one thread per 16 bytes of a row (8 bf16 or 4 fp32); needs Vs % (16/sizeof(T)) == 0.
// Workgroup (x, y): row x, chunks 256 y .. 256 y + 255 of it: no division per thread, and the row's
// statistics and label are the same for the whole workgroup.
template <typename T, bool PRECISE>
__global__ __launch_bounds__(256) void dlogits_vec_kernel(const T* Y, T* D,   // may alias (in place)
                                                          const int64_t* __restrict__ labels, int64_t off,
                                                          const float* __restrict__ gmax, const float* __restrict__ gsum,
                                                          float scale, int chunks_per_row, int Vs, int64_t ldy,
                                                          int64_t ldd) {
    constexpr int E = 16 / (int)sizeof(T);
    const int i = blockIdx.x;
    const int c = blockIdx.y * 256 + threadIdx.x;      // chunk of the row of D: chunks_per_row = ldd / E
    if (c >= chunks_per_row) return;
    const int j0 = c * E;
    if (j0 >= Vs) {   // padding of the row: zero, because the dH product multiplies it by zero
        *reinterpret_cast<uint4*>(D + (int64_t)i * ldd + j0) = make_uint4(0u, 0u, 0u, 0u);
        return;
    }
    const float m = gmax[i];
    const float inv = 1.0f / gsum[i];
    // position of the label inside this chunk, if 0 <= loc < E
    const int64_t loc = labels ? labels[i] - off - j0 : (int64_t)-1;
    const uint4 raw = *reinterpret_cast<const uint4*>(Y + (int64_t)i * ldy + j0);
    const unsigned w[4] = {raw.x, raw.y, raw.z, raw.w};
    float v[E];
    if (sizeof(T) == 2) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            v[2 * e] = __uint_as_float(w[e] << 16);
            v[2 * e + 1] = __uint_as_float(w[e] & 0xFFFF0000u);
        }
    } else {
#pragma unroll
        for (int e = 0; e < E; ++e) v[e] = __uint_as_float(w[e]);
    }
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const float x = v[e] - m;
        float pr = (PRECISE ? expf(x) : __expf(x)) * inv;
        if (loc == (int64_t)e) pr -= 1.0f;
        v[e] = pr * scale;
    }
    uint4 o;
    if (sizeof(T) == 2) {
        unsigned q[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const __bf16 a = (__bf16)v[2 * e], b = (__bf16)v[2 * e + 1];
            q[e] = (unsigned)__builtin_bit_cast(u16, a) | ((unsigned)__builtin_bit_cast(u16, b) << 16);
        }
        o = make_uint4(q[0], q[1], q[2], q[3]);
    } else {
        o = make_uint4(__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[E > 2 ? 2 : 0]),
                       __float_as_uint(v[E > 3 ? 3 : 0]));
    }
    *reinterpret_cast<uint4*>(D + (int64_t)i * ldd + j0) = o;
}

// Zeroes columns rows .. ldd-1 of every row of the bf16 matrices D_r (recompute mode: the GEMM
// epilogue that writes D stops at the shard's last column).  blockIdx.y is the shard.
__global__ __launch_bounds__(256) void zero_pad_columns_kernel(ShardList l, int N) {
    const int sh = blockIdx.y, Vs = l.rows[sh];
    const int64_t ldd = l.ldd[sh];
    const int pad = (int)(ldd - Vs);
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (t >= (int64_t)N * pad) return;
    const int i = (int)(t / pad), j = (int)(t - (int64_t)i * pad);
    ((u16*)l.D[sh])[(int64_t)i * ldd + Vs + j] = 0;
}

hipError_t launch_zero_pad_columns(const ShardList& l, int N, hipStream_t st) {
    int64_t pad = 0;
    for (int r = 0; r < l.n; ++r) pad = l.ldd[r] - l.rows[r] > pad ? l.ldd[r] - l.rows[r] : pad;
    if (pad == 0) return hipSuccess;
    ProfScope prof(K_ZERO_PAD, st);
    hipLaunchKernelGGL(zero_pad_columns_kernel, dim3((unsigned)ceil_div((int64_t)N * pad, 256), l.n), dim3(256), 0, st, l, N);
    return hipGetLastError();
}

// bf16 D of all shards of a list, any number of rows per shard: a thread forms 8 elements of a row of D (16-byte aligned:
// ldd is a multiple of 64).  Rows of Y start 2 ldy[r] bytes apart, so their 16 bytes may begin at any element: the load
// is declared 2-byte aligned, which global memory takes on this hardware; the last chunk of a row is read by elements.
// Bound by memory (Y in, D out).  Workgroup (x, y, z): row x, chunks 256 y .. + 255, shard z.
__global__ __launch_bounds__(256) void dlogits_group_kernel(ShardList l, const int64_t* __restrict__ labels,
                                                            const float* __restrict__ gmax, const float* __restrict__ gsum,
                                                            int64_t shard_stats, float scale) {
    typedef unsigned ua4 __attribute__((ext_vector_type(4), aligned(2)));
    const int sh = blockIdx.z, Vs = l.rows[sh], i = blockIdx.x;
    const int64_t ldd = l.ldd[sh];
    const int j0 = (blockIdx.y * 256 + threadIdx.x) * 8;
    if (j0 >= ldd) return;
    const u16* y = (const u16*)l.Y[sh] + (int64_t)i * l.ldy[sh] + j0;
    u16* d = (u16*)l.D[sh] + (int64_t)i * ldd + j0;
    unsigned w[4] = {0u, 0u, 0u, 0u};
    if (j0 + 8 <= Vs) {
        const ua4 raw = *reinterpret_cast<const ua4*>(y);
#pragma unroll
        for (int e = 0; e < 4; ++e) w[e] = raw[e];
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e)
            if (j0 + e < Vs) w[e >> 1] |= (unsigned)y[e] << (16 * (e & 1));
    }
    const float m = gmax[sh * shard_stats + i];
    const float inv = 1.0f / gsum[sh * shard_stats + i];
    const int64_t loc = labels ? labels[i] - l.offset[sh] - j0 : (int64_t)-1;
    unsigned q[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        float v[2] = {__uint_as_float(w[e] << 16), __uint_as_float(w[e] & 0xFFFF0000u)};
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            float pr = __expf(v[u] - m) * inv;
            if (loc == (int64_t)(2 * e + u)) pr -= 1.0f;
            v[u] = j0 + 2 * e + u < Vs ? pr * scale : 0.f;    // padding: zero, the dH product multiplies it by zero
        }
        const __bf16 a = (__bf16)v[0], b = (__bf16)v[1];
        q[e] = (unsigned)__builtin_bit_cast(u16, a) | ((unsigned)__builtin_bit_cast(u16, b) << 16);
    }
    *reinterpret_cast<uint4*>(d) = make_uint4(q[0], q[1], q[2], q[3]);
}

// The same in fp32 (4 elements per thread, ldd a multiple of 4); D_r may be Y_r.
__global__ __launch_bounds__(256) void dlogits_group_f32_kernel(ShardList l, const int64_t* __restrict__ labels,
                                                                const float* __restrict__ gmax, const float* __restrict__ gsum,
                                                                int64_t shard_stats, float scale) {
    typedef float ua4 __attribute__((ext_vector_type(4), aligned(4)));
    const int sh = blockIdx.z, Vs = l.rows[sh], i = blockIdx.x;
    const int64_t ldd = l.ldd[sh];
    const int j0 = (blockIdx.y * 256 + threadIdx.x) * 4;
    if (j0 >= ldd) return;
    const float* y = (const float*)l.Y[sh] + (int64_t)i * l.ldy[sh] + j0;
    float v[4] = {0.f, 0.f, 0.f, 0.f};
    if (j0 + 4 <= Vs) {
        const ua4 raw = *reinterpret_cast<const ua4*>(y);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = raw[e];
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (j0 + e < Vs) v[e] = y[e];
    }
    const float m = gmax[sh * shard_stats + i];
    const float inv = 1.0f / gsum[sh * shard_stats + i];
    const int64_t loc = labels ? labels[i] - l.offset[sh] - j0 : (int64_t)-1;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        float pr = expf(v[e] - m) * inv;
        if (loc == (int64_t)e) pr -= 1.0f;
        v[e] = j0 + e < Vs ? pr * scale : 0.f;
    }
    *reinterpret_cast<float4*>((float*)l.D[sh] + (int64_t)i * ldd + j0) = make_float4(v[0], v[1], v[2], v[3]);
}

hipError_t launch_dlogits_group(const ShardList& l, int is_bf16, const int64_t* labels, const float* gmax, const float* gsum,
                                int64_t shard_stats, float scale, int N, hipStream_t st) {
    ProfScope prof(K_DLOGITS_EW, st);
    int64_t ldd = 0;
    for (int r = 0; r < l.n; ++r) ldd = l.ldd[r] > ldd ? l.ldd[r] : ldd;
    if (is_bf16)
        hipLaunchKernelGGL(dlogits_group_kernel, dim3((unsigned)N, (unsigned)ceil_div(ldd, 2048), l.n), dim3(256), 0, st, l,
                           labels, gmax, gsum, shard_stats, scale);
    else
        hipLaunchKernelGGL(dlogits_group_f32_kernel, dim3((unsigned)N, (unsigned)ceil_div(ldd, 1024), l.n), dim3(256), 0, st, l,
                           labels, gmax, gsum, shard_stats, scale);
    return hipGetLastError();
}

hipError_t launch_dlogits(const void* Y, int64_t ldy, void* D, int64_t ldd, int is_bf16, const int64_t* labels,
                          int64_t off, const float* gmax, const float* gsum, float scale, int N, int Vs,
                          hipStream_t st) {
    ProfScope prof(K_DLOGITS_EW, st);
    const int E = is_bf16 ? 8 : 4;
    if (Vs % E == 0 && ldd % E == 0 && ldy % E == 0 && ((((uintptr_t)Y) | ((uintptr_t)D)) & 15u) == 0) {
        const int cpr = (int)(ldd / E);
        const dim3 grid((unsigned)N, (unsigned)ceil_div(cpr, 256));     // rows in x: no 65535 limit on them
        if (is_bf16) {
            hipLaunchKernelGGL((dlogits_vec_kernel<u16, false>), grid, dim3(256), 0, st, (const u16*)Y, (u16*)D, labels,
                               off, gmax, gsum, scale, cpr, Vs, ldy, ldd);
        } else {
            hipLaunchKernelGGL((dlogits_vec_kernel<float, true>), grid, dim3(256), 0, st, (const float*)Y, (float*)D,
                               labels, off, gmax, gsum, scale, cpr, Vs, ldy, ldd);
        }
        return hipGetLastError();
    }
    unsigned gx = (unsigned)ceil_div(ldd, 256);
    if (gx > 64) gx = 64;
    // grid.y carries the row; rows beyond 65535 are covered by launching in slabs
    for (int r0 = 0; r0 < N; r0 += 65535) {
        const int rows = (N - r0 < 65535) ? (N - r0) : 65535;
        const int64_t* lab = labels ? labels + r0 : nullptr;
        if (is_bf16) {
            hipLaunchKernelGGL((dlogits_kernel<u16, false>), dim3(gx, rows), dim3(256), 0, st,
                               (const u16*)Y + (int64_t)r0 * ldy, (u16*)D + (int64_t)r0 * ldd, lab, off,
                               gmax + r0, gsum + r0, scale, Vs, ldy, ldd);
        } else {
            hipLaunchKernelGGL((dlogits_kernel<float, true>), dim3(gx, rows), dim3(256), 0, st,
                               (const float*)Y + (int64_t)r0 * ldy, (float*)D + (int64_t)r0 * ldd, lab, off,
                               gmax + r0, gsum + r0, scale, Vs, ldy, ldd);
        }
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// Input gradient of Algorithm 2 (section 4.4): dH += (A_r c_r - B_r) scale over the shards of the list in order
// (OVERWRITE: dH = ...), one thread per 4 columns.  Bound by memory: with a launch per shard dH was read and written once
// per shard; here it is written once (N=4096, h=4096, 8 shards: 8 launches of 28 us -> one of 184 us with 0.86 GB, 4.7 TB/s).
struct DxList {
    int n;
    const float* A[GEMM_GROUP_MAX];
    const void* B[GEMM_GROUP_MAX];
};

template <typename TB, bool OVERWRITE>
__global__ __launch_bounds__(256) void dx_alg2_kernel(DxList l, const float* __restrict__ lmax, const float* __restrict__ lsum,
                                                      const float* __restrict__ gmax, const float* __restrict__ gsum,
                                                      int N, int h, int64_t total, float scale, float* dH, int vec) {
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (t >= total) return;
    const int q = vec ? h / 4 : h;
    const int i = (int)(t / q);
    const float gm = gmax[i], gs = gsum[i];
    if (vec) {
        const int64_t e0 = (int64_t)i * h + (t - (int64_t)i * q) * 4;
        float4 d = OVERWRITE ? make_float4(0.f, 0.f, 0.f, 0.f) : *reinterpret_cast<const float4*>(dH + e0);
        for (int r = 0; r < l.n; ++r) {
            const float ml = lmax[(size_t)r * N + i];
            const float c = (ml > -INFINITY) ? lsum[(size_t)r * N + i] * expf(ml - gm) / gs : 0.f;
            const float4 a = *reinterpret_cast<const float4*>(l.A[r] + e0);
            float b[4];
            if (sizeof(TB) == 2) {
                const uint2 w = *reinterpret_cast<const uint2*>((const TB*)l.B[r] + e0);
                b[0] = __uint_as_float(w.x << 16); b[1] = __uint_as_float(w.x & 0xFFFF0000u);
                b[2] = __uint_as_float(w.y << 16); b[3] = __uint_as_float(w.y & 0xFFFF0000u);
            } else {
                const float4 w = *reinterpret_cast<const float4*>((const TB*)l.B[r] + e0);
                b[0] = w.x; b[1] = w.y; b[2] = w.z; b[3] = w.w;
            }
            d.x += (a.x * c - b[0]) * scale;
            d.y += (a.y * c - b[1]) * scale;
            d.z += (a.z * c - b[2]) * scale;
            d.w += (a.w * c - b[3]) * scale;
        }
        *reinterpret_cast<float4*>(dH + e0) = d;
    } else {
        float d = OVERWRITE ? 0.f : dH[t];
        for (int r = 0; r < l.n; ++r) {
            const float ml = lmax[(size_t)r * N + i];
            const float c = (ml > -INFINITY) ? lsum[(size_t)r * N + i] * expf(ml - gm) / gs : 0.f;
            d += (l.A[r][t] * c - ld_as_f32<TB>((const TB*)l.B[r] + t)) * scale;
        }
        dH[t] = d;
    }
}

template <typename TB>
static void launch_dx_alg2_t(const DxList& l, const float* lmax, const float* lsum, const float* gmax, const float* gsum, int N,
                             int h, float scale, bool overwrite, float* dH, hipStream_t st) {
    const int vec = (h % 4 == 0) ? 1 : 0;
    const int64_t total = vec ? (int64_t)N * (h / 4) : (int64_t)N * h;
    const unsigned blocks = (unsigned)ceil_div(total, 256);
    if (overwrite)
        hipLaunchKernelGGL((dx_alg2_kernel<TB, true>), dim3(blocks), dim3(256), 0, st, l, lmax, lsum, gmax, gsum, N, h, total,
                           scale, dH, vec);
    else
        hipLaunchKernelGGL((dx_alg2_kernel<TB, false>), dim3(blocks), dim3(256), 0, st, l, lmax, lsum, gmax, gsum, N, h, total,
                           scale, dH, vec);
}

hipError_t launch_dx_alg2(const float* const* A, const void* const* B, int p, int b_is_bf16, const float* lmax,
                          const float* lsum, const float* gmax, const float* gsum, int N, int h, float scale, bool overwrite,
                          float* dH, hipStream_t st) {
    ProfScope prof(K_DX_ALG2, st);
    for (int r0 = 0; r0 < p; r0 += GEMM_GROUP_MAX) {
        DxList l{};
        l.n = p - r0 < GEMM_GROUP_MAX ? p - r0 : GEMM_GROUP_MAX;
        for (int k = 0; k < l.n; ++k) {
            l.A[k] = A[r0 + k];
            l.B[k] = B[r0 + k];
        }
        const float *lm = lmax + (size_t)r0 * N, *ls = lsum + (size_t)r0 * N;
        const bool over = overwrite && r0 == 0;
        if (b_is_bf16) launch_dx_alg2_t<u16>(l, lm, ls, gmax, gsum, N, h, scale, over, dH, st);
        else launch_dx_alg2_t<float>(l, lm, ls, gmax, gsum, N, h, scale, over, dH, st);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// The same with the rows of B = G W taken from the shards themselves: of the p matrices B, which are zero but for one row per
// token, nothing is read.  A is [p, N, h], read once (non-temporal, four shards' values in flight).  Workgroup (x, y): token x,
// columns 1024 y on.  Bound by reading A: N=4096 h=4096, 8 shards, 0.64 GB: 180 us with the matrices B -> 110 us (5.8 TB/s).
struct DxGatherList {
    int n;
    int rows[GEMM_GROUP_MAX];
    int64_t offset[GEMM_GROUP_MAX];
    const void* W[GEMM_GROUP_MAX];
};

template <typename T, bool VEC>
__global__ __launch_bounds__(256) void dx_alg2_gather_kernel(DxGatherList l, const float* __restrict__ A,
                                                             const int64_t* __restrict__ labels,
                                                             const float* __restrict__ lmax, const float* __restrict__ lsum,
                                                             const float* __restrict__ gmax, const float* __restrict__ gsum,
                                                             int N, int h, float scale, bool overwrite, float* dH) {
    constexpr int E = VEC ? 4 : 1;
    typedef float V __attribute__((ext_vector_type(E)));
    const int i = blockIdx.x;
    const int j = (blockIdx.y * 256 + threadIdx.x) * E;
    if (j >= h) return;
    const int64_t e0 = (int64_t)i * h + j, plane = (int64_t)N * h;
    const float gm = gmax[i], gs = gsum[i];
    const int64_t label = labels[i];
    int owner = -1;
    for (int r = 0; r < l.n; ++r) owner = label >= l.offset[r] && label - l.offset[r] < l.rows[r] ? r : owner;
    V b = {};
    if (owner >= 0) {
        const T* w = (const T*)l.W[owner] + (label - l.offset[owner]) * h + j;
        if constexpr (VEC && sizeof(T) == 2) {
            const uint2 q = *reinterpret_cast<const uint2*>(w);
            b[0] = __uint_as_float(q.x << 16); b[1] = __uint_as_float(q.x & 0xFFFF0000u);
            b[2] = __uint_as_float(q.y << 16); b[3] = __uint_as_float(q.y & 0xFFFF0000u);
        } else if constexpr (VEC) {
            b = *reinterpret_cast<const V*>(w);
        } else {
            b[0] = ld_as_f32<T>(w);
        }
    }
    V d = {};
    if (!overwrite) d = *reinterpret_cast<const V*>(dH + e0);
    for (int r0 = 0; r0 < l.n; r0 += 4) {
        V a[4];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (r0 + u < l.n) a[u] = __builtin_nontemporal_load(reinterpret_cast<const V*>(A + (r0 + u) * plane + e0));
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int r = r0 + u;
            if (r < l.n) {
                const float ml = lmax[(size_t)r * N + i];
                const float c = (ml > -INFINITY) ? lsum[(size_t)r * N + i] * expf(ml - gm) / gs : 0.f;
#pragma unroll
                for (int e = 0; e < E; ++e) d[e] += (a[u][e] * c - (r == owner ? b[e] : 0.f)) * scale;
            }
        }
    }
    *reinterpret_cast<V*>(dH + e0) = d;
}

hipError_t launch_dx_alg2_gather(const float* A, const void* const* W, const int64_t* rows, const int64_t* offsets, int p,
                                 int is_bf16, const int64_t* labels, const float* lmax, const float* lsum, const float* gmax,
                                 const float* gsum, int N, int h, float scale, bool overwrite, float* dH, hipStream_t st) {
    if (p > GEMM_GROUP_MAX) return hipErrorInvalidValue;
    ProfScope prof(K_DX_ALG2, st);
    DxGatherList l{};
    l.n = p;
    for (int r = 0; r < p; ++r) {
        l.rows[r] = (int)rows[r];
        l.offset[r] = offsets[r];
        l.W[r] = W[r];
    }
    const bool vec = h % 4 == 0;
    const dim3 grid((unsigned)N, (unsigned)ceil_div(h, vec ? 1024 : 256));
#define VP_DX(T, V) hipLaunchKernelGGL((dx_alg2_gather_kernel<T, V>), grid, dim3(256), 0, st, l, A, labels, lmax, lsum, gmax, gsum, N, h, scale, overwrite, dH)
    if (is_bf16 && vec) VP_DX(u16, true);
    else if (is_bf16) VP_DX(u16, false);
    else if (vec) VP_DX(float, true);
    else VP_DX(float, false);
#undef VP_DX
    return hipGetLastError();
}

}  // namespace vp
