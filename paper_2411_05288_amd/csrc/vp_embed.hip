// Input (embedding) layer of the vocabulary shards one device holds (appendix C of the paper): the
// gather that builds every shard's full-size [N, h] output with zero rows for ids it does not own, and
// the scatter-add of the output gradient into the shards' fp32 table gradients.
//
// A launch serves up to EMBED_GROUP_MAX shards (shard s of the group owns rows [off + s Vs, off + (s+1) Vs)):
// the tokens are sorted once for all of them, and small shards fill the chip together.
//
// The scatter-add uses no atomics on the gradient.  Tokens are keyed by (row, token position), the keys
// are sorted (they are unique, so the order is total), and every run of equal rows is summed in
// increasing token position, starting from the value already in the table gradient.  The result does
// not depend on scheduling.
#include "vp_internal.h"

namespace vp {

typedef unsigned long long u64;
typedef unsigned uintx4 __attribute__((ext_vector_type(4)));

// (P = 1 or EMBED_GROUP_MAX: a launch of one shard carries one shard's arguments)
template <int P>
struct EmbedFwdGroup {
    const void* table[P];
    void* out[P];
};
template <int P>
struct EmbedBwdGroup {
    float* dtable[P];
};

// ------------------------------------------------------------------------- forward
// Bound by the stores: p full-size outputs leave, at most N table rows come in.  The output is written once and read much
// later (by the reduce over shards): streaming stores.  Two maps of threads to rows, both with the shard in blockIdx.y:
//  * a workgroup per row: its four wavefronts write neighbouring KB of one row at a time.  Workgroups are dealt to the 8 XCDs
//    round-robin and every XCD has its own L2, so each XCD takes a contiguous run of rows: a cache line that two rows share
//    is then completed in one L2.  Row i in workgroup i -> so, us in one launch: 34340 tokens, h = 728, bf16, 24 shards:
//    324 -> 231 (a launch per shard: 271), 20741, 1808, 16: 263 -> 218, 39694, 557, fp32, 8: 213 -> 163; rows of whole lines,
//    8192, 4096, bf16, 8: 95 -> 88, 65536, 2048, 8: 322 -> 337;
//  * a wavefront per row, rows_per_wg consecutive rows (about 32 KB) per workgroup: for short rows, of which one leaves most
//    lanes of a workgroup idle.
// Wavefront per row -> row i in workgroup i, us in one launch (V=32000): 65536 tokens, 8 shards, bf16, h = 128: 26 -> 114,
// 512: 101 -> 114, 640: 131 -> 123, 768: 157 -> 124, 1024: 202 -> 149, 2048: 394 -> 321; one shard, 640: 26 -> 28, 1024:
// 40 -> 38.  Rows that are not 16-byte aligned (4 shards, 30000 tokens): 261 bf16: 34 -> 36, 511: 62 -> 42, 1001: 120 -> 58;
// 131 fp32: 31 -> 33, 251: 51 -> 37.
constexpr int64_t FWD_WAVE_BYTES = 1280, FWD_WAVE_BYTES_UNALIGNED = 640;     // the longest row of a wavefront

template <typename V>
__device__ __forceinline__ void embed_row(V* o, const V* __restrict__ table, int64_t loc, int Vs, int row_vecs, int first, int step) {
    if (loc >= 0 && loc < Vs) {
        const V* __restrict__ t = table + (size_t)loc * row_vecs;
        for (int c = first; c < row_vecs; c += step) __builtin_nontemporal_store(t[c], o + c);
    } else {
        const V z = V(0);
        for (int c = first; c < row_vecs; c += step) __builtin_nontemporal_store(z, o + c);
    }
}

template <typename V, int P>
__global__ __launch_bounds__(256) void embed_fwd_wg_kernel(EmbedFwdGroup<P> g, const int64_t* __restrict__ ids, int row_vecs,
                                                           int Vs, int64_t off) {
    const int s = blockIdx.y, b = blockIdx.x, N = gridDim.x;
    const int x = b & 7, per = N >> 3, rem = N & 7;
    const int i = x * per + (x < rem ? x : rem) + (b >> 3);
    embed_row<V>((V*)g.out[s] + (size_t)i * row_vecs, (const V*)g.table[s], ids[i] - (off + (int64_t)s * Vs), Vs, row_vecs,
                 threadIdx.x, 256);
}

template <typename V, int P>
__global__ __launch_bounds__(256) void embed_fwd_wave_kernel(EmbedFwdGroup<P> g, const int64_t* __restrict__ ids, int N,
                                                             int row_vecs, int Vs, int64_t off, int rows_per_wg) {
    const int s = blockIdx.y;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const V* __restrict__ table = (const V*)g.table[s];
    V* __restrict__ out = (V*)g.out[s];
    const int64_t first = off + (int64_t)s * Vs;
    const int end = min(N, (int)(blockIdx.x + 1) * rows_per_wg);
    for (int i = blockIdx.x * rows_per_wg + wave; i < end; i += 4)
        embed_row<V>(out + (size_t)i * row_vecs, table, ids[i] - first, Vs, row_vecs, lane, 64);
}

template <typename V, int P>
static void launch_embed_fwd_p(const void* const* tables, void* const* outs, int n, const int64_t* ids, int N, int row_vecs, int Vs,
                               int64_t off, int rows, hipStream_t st) {
    EmbedFwdGroup<P> g{};
    for (int s = 0; s < n; ++s) {
        g.table[s] = tables[s];
        g.out[s] = outs[s];
    }
    if (rows == 0)
        hipLaunchKernelGGL((embed_fwd_wg_kernel<V, P>), dim3((unsigned)N, (unsigned)n), dim3(256), 0, st, g, ids, row_vecs, Vs, off);
    else
        hipLaunchKernelGGL((embed_fwd_wave_kernel<V, P>), dim3((unsigned)ceil_div(N, rows), (unsigned)n), dim3(256), 0, st, g, ids,
                           N, row_vecs, Vs, off, rows);
}
template <typename V>
static void launch_embed_fwd_t(const void* const* tables, void* const* outs, int n, const int64_t* ids, int N, int row_vecs, int Vs,
                               int64_t off, int rows, hipStream_t st) {
    if (n == 1) launch_embed_fwd_p<V, 1>(tables, outs, n, ids, N, row_vecs, Vs, off, rows, st);
    else launch_embed_fwd_p<V, EMBED_GROUP_MAX>(tables, outs, n, ids, N, row_vecs, Vs, off, rows, st);
}

hipError_t launch_embed_fwd(const void* const* tables, const int64_t* ids, int p, int N, int h, int Vs, int64_t off,
                            int elem_bytes, void* const* outs, hipStream_t st) {
    const int64_t row_bytes = (int64_t)h * elem_bytes;
    ProfScope prof(K_EMBED_FWD, st);
    const bool vec = row_bytes % 16 == 0;
    int rows = 0;              // of a workgroup with a wavefront per row; 0: a workgroup per row (N h < 2^31: below 2^23 rows)
    if (row_bytes <= (vec ? FWD_WAVE_BYTES : FWD_WAVE_BYTES_UNALIGNED)) {
        rows = (int)(32768 / row_bytes) / 4 * 4;
        if (rows > 64) rows = 64;
        // fewer rows per workgroup while the grid would leave compute units without one
        while (rows > 4 && ceil_div(N, rows) * p < 1024) rows -= 4;
    }
    for (int s0 = 0; s0 < p; s0 += EMBED_GROUP_MAX) {
        const int n = p - s0 < EMBED_GROUP_MAX ? p - s0 : EMBED_GROUP_MAX;
        const int64_t first = off + (int64_t)s0 * Vs;
        if (vec) launch_embed_fwd_t<uintx4>(tables + s0, outs + s0, n, ids, N, (int)(row_bytes / 16), Vs, first, rows, st);
        else if (elem_bytes == 4) launch_embed_fwd_t<unsigned>(tables + s0, outs + s0, n, ids, N, h, Vs, first, rows, st);
        else launch_embed_fwd_t<u16>(tables + s0, outs + s0, n, ids, N, h, Vs, first, rows, st);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// ------------------------------------------------------------------------- backward: common pieces
template <int VEC>
__device__ __forceinline__ void load_acc(float (&acc)[VEC], const float* d) {
    if (VEC == 2) {
        const float2 v = *reinterpret_cast<const float2*>(d);
        acc[0] = v.x; acc[1 % VEC] = v.y;
    } else {
        acc[0] = d[0];
    }
}
template <int VEC>
__device__ __forceinline__ void store_acc(float* d, const float (&acc)[VEC]) {
    if (VEC == 2) *reinterpret_cast<float2*>(d) = make_float2(acc[0], acc[1 % VEC]);
    else d[0] = acc[0];
}

// acc += gradient values; `on` false adds -0.0f instead, which leaves every float (either zero
// included) bit for bit unchanged.
__device__ __forceinline__ float gate(float x, bool on) { return on ? x : -0.0f; }
__device__ __forceinline__ void add_grad(float (&acc)[1], const u16& v, bool on) {
    acc[0] += gate(__uint_as_float((unsigned)v << 16), on);
}
__device__ __forceinline__ void add_grad(float (&acc)[1], const float& v, bool on) { acc[0] += gate(v, on); }
__device__ __forceinline__ void add_grad(float (&acc)[2], const unsigned& v, bool on) {
    acc[0] += gate(__uint_as_float(v << 16), on);
    acc[1] += gate(__uint_as_float(v & 0xFFFF0000u), on);
}
__device__ __forceinline__ void add_grad(float (&acc)[2], const float2& v, bool on) {
    acc[0] += gate(v.x, on); acc[1] += gate(v.y, on);
}

// The adds of those tokens in order; positions past cnt add -0.0f.
template <int D, int VEC, typename GV>
__device__ __forceinline__ void add_batch(float (&acc)[VEC], const GV (&v)[D], int u0, int cnt) {
#pragma unroll
    for (int u = 0; u < D; ++u) add_grad(acc, v[u], u0 + u < cnt);
}
// ------------------------------------------------------------------------- backward: one kernel for N <= 8192
// Up to FUSED_MAX_N tokens and FUSED_MAX_ROWS rows of all shards: one launch does everything.  EVERY workgroup (1024
// threads, one per compute unit) builds and sorts the keys in its own LDS - the same few microseconds in all of them,
// instead of a sort kernel, a round trip of the keys through memory and a second launch - numbers the runs of equal
// rows, and then takes its share of the sums: workgroup (slab, group) covers 64 * VEC columns; its 16 wavefronts take
// the runs group * 16 + w, + groups * 16, ... (sum_short_runs, sum_mid_run) but for the long ones, which the 16 share
// (sum_long_run).  Measured: 8192 Zipf tokens, h = 4096, bf16, 8 shards of 32000 rows: 81 us in one launch, 162 us in
// eight; N = 512, h = 1024, fp32: 12 us for 8 launches of 9 us.
constexpr int FUSED_MAX_N = 8192;
constexpr int TOKEN_BITS = 13;                       // a key: local row << 13 | token position
constexpr int FUSED_MAX_ROWS = (1 << (32 - TOKEN_BITS)) - 1;   // so that no key equals KEY32_NONE
constexpr unsigned KEY32_NONE = 0xFFFFFFFFu;
constexpr int FUSED_THREADS = 1024;
constexpr int FUSED_WAVES = FUSED_THREADS / 64;
constexpr int WAVE_KEYS = 512;                       // eight consecutive keys per lane

// n_rows: rows of all shards of the group
template <int TB>
__device__ __forceinline__ unsigned token_key32(const int64_t* __restrict__ ids, int i, int N, int n_rows, int64_t off,
                                                unsigned token) {
    if (i < N) {
        const int64_t loc = ids[i] - off;
        if (loc >= 0 && loc < n_rows) return ((unsigned)loc << TB) | token;
    }
    return KEY32_NONE;
}
__device__ __forceinline__ unsigned key_row(unsigned k) { return k >> TOKEN_BITS; }
__device__ __forceinline__ unsigned key_token(unsigned k) { return k & ((1u << TOKEN_BITS) - 1u); }

__device__ __forceinline__ void order(unsigned& x, unsigned& y, bool asc) {
    const unsigned lo = x < y ? x : y, hi = x < y ? y : x;
    x = asc ? lo : hi;
    y = asc ? hi : lo;
}

// The value lane ^ X holds.  X = 1, 2, 8: one DPP move (quad_perm [1,0,3,2], [2,3,0,1], row_ror:8); X = 4: row_shl:4
// for the lanes with bit 2 clear and row_shr:4 for the others (bank masks 0x5 / 0xA); across rows of 16: ds_bpermute.
template <int X>
__device__ __forceinline__ unsigned lane_xor(unsigned x) {
    const int v = (int)x;
    if (X == 1) return (unsigned)__builtin_amdgcn_update_dpp(v, v, 0xB1, 0xF, 0xF, false);
    if (X == 2) return (unsigned)__builtin_amdgcn_update_dpp(v, v, 0x4E, 0xF, 0xF, false);
    if (X == 4) {
        const int a = __builtin_amdgcn_update_dpp(v, v, 0x104, 0xF, 0x5, false);
        return (unsigned)__builtin_amdgcn_update_dpp(a, v, 0x114, 0xF, 0xA, false);
    }
    if (X == 8) return (unsigned)__builtin_amdgcn_update_dpp(v, v, 0x128, 0xF, 0xF, false);
    return (unsigned)__shfl_xor(v, X, 64);
}

// One pass of distance 8 X of stage k: the partner holds the same e in lane ^ X; k > 8 X >= 8, so the direction is
// the same for the whole lane.
template <int X>
__device__ __forceinline__ void exchange_pass(unsigned (&v)[8], int i0, int k) {
    const bool keep_min = ((i0 & (8 * X)) == 0) == ((i0 & k) == 0);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const unsigned o = lane_xor<X>(v[e]);
        const unsigned lo = v[e] < o ? v[e] : o, hi = v[e] < o ? o : v[e];
        v[e] = keep_min ? lo : hi;
    }
}

// Passes j_first, j_first / 2, ..., 1 (j_first <= 256) of stage k of the bitonic network on the 512 keys a wavefront
// holds, v[e] = key i0 + e with i0 a multiple of 8: distances of 8 and more exchange between lanes, 4, 2, 1 inside
// the lane.  No LDS traffic and no barrier.
__device__ __forceinline__ void bitonic_inwave(unsigned (&v)[8], int i0, int j_first, int k) {
    if (j_first >= 256) exchange_pass<32>(v, i0, k);
    if (j_first >= 128) exchange_pass<16>(v, i0, k);
    if (j_first >= 64) exchange_pass<8>(v, i0, k);
    if (j_first >= 32) exchange_pass<4>(v, i0, k);
    if (j_first >= 16) exchange_pass<2>(v, i0, k);
    if (j_first >= 8) exchange_pass<1>(v, i0, k);
    if (j_first >= 4) {
#pragma unroll
        for (int e = 0; e < 4; ++e) order(v[e], v[e + 4], ((i0 + e) & k) == 0);
    }
    if (j_first >= 2) {
#pragma unroll
        for (int e = 0; e < 8; ++e)
            if ((e & 2) == 0) order(v[e], v[e + 2], ((i0 + e) & k) == 0);
    }
#pragma unroll
    for (int e = 0; e < 8; e += 2) order(v[e], v[e + 1], ((i0 + e) & k) == 0);
}

// LEVELS consecutive passes (distances j, j / 2, ..., j >> (LEVELS - 1)) of stage k on LDS-resident keys, by the
// whole workgroup, in registers on groups of 2^LEVELS keys; ends with a barrier.
template <int LEVELS>
__device__ __forceinline__ void bitonic_levels_lds32(unsigned* sh, int m, int j, int k) {
    constexpr int G = 1 << LEVELS;
    const int low = j >> (LEVELS - 1);
    for (int t = threadIdx.x; t < m / G; t += FUSED_THREADS) {
        const int base = ((t & ~(low - 1)) << LEVELS) | (t & (low - 1));
        const bool asc = (base & k) == 0;
        unsigned v[G];
#pragma unroll
        for (int e = 0; e < G; ++e) v[e] = sh[base + e * low];
#pragma unroll
        for (int d = G >> 1; d > 0; d >>= 1)
#pragma unroll
            for (int e = 0; e < G; ++e)
                if ((e & d) == 0) order(v[e], v[e | d], asc);
#pragma unroll
        for (int e = 0; e < G; ++e) sh[base + e * low] = v[e];
    }
    __syncthreads();
}

__device__ __forceinline__ void load_keys8(unsigned (&v)[8], const unsigned* sh, int i0) {
    const uintx4 a = *reinterpret_cast<const uintx4*>(sh + i0), b = *reinterpret_cast<const uintx4*>(sh + i0 + 4);
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}
__device__ __forceinline__ void store_keys8(unsigned* sh, int i0, const unsigned (&v)[8]) {
    uintx4 a, b;
    a.x = v[0]; a.y = v[1]; a.z = v[2]; a.w = v[3]; b.x = v[4]; b.y = v[5]; b.z = v[6]; b.w = v[7];
    *reinterpret_cast<uintx4*>(sh + i0) = a;
    *reinterpret_cast<uintx4*>(sh + i0 + 4) = b;
}

// Ascending bitonic sort of sh[0 .. m), m a power of two between 512 and 8192, by a workgroup of 16 wavefronts.
// Wavefront w owns keys 512 w .. 512 w + 511: it sorts them alone (stages 2 .. 512, 45 passes, no barrier), and in
// each later stage k the workgroup does the passes of distance >= 512 on LDS (one round trip) and the wavefronts the
// remaining nine.  Barriers: 1 + 2 log2(m / 512).
__device__ __forceinline__ void bitonic_sort_lds32(unsigned* sh, int m, int lane, int wave) {
    const bool on = wave * WAVE_KEYS < m;
    const int i0 = wave * WAVE_KEYS + lane * 8;
    unsigned v[8];
    if (on) {
        load_keys8(v, sh, i0);
        for (int k = 2; k <= WAVE_KEYS; k <<= 1) bitonic_inwave(v, i0, k >> 1, k);
        store_keys8(sh, i0, v);
    }
    __syncthreads();
    for (int k = 2 * WAVE_KEYS; k <= m; k <<= 1) {
        switch (k / WAVE_KEYS) {       // passes k / 2 .. 512
            case 2: bitonic_levels_lds32<1>(sh, m, k >> 1, k); break;
            case 4: bitonic_levels_lds32<2>(sh, m, k >> 1, k); break;
            case 8: bitonic_levels_lds32<3>(sh, m, k >> 1, k); break;
            default: bitonic_levels_lds32<4>(sh, m, k >> 1, k); break;
        }
        if (on) {
            load_keys8(v, sh, i0);
            bitonic_inwave(v, i0, WAVE_KEYS >> 1, k);
            store_keys8(sh, i0, v);
        }
        __syncthreads();
    }
}

typedef unsigned uintx2 __attribute__((ext_vector_type(2)));
template <typename GV>
__device__ __forceinline__ GV buf_load(__amdgpu_buffer_rsrc_t rs, unsigned voff, unsigned soff);
template <> __device__ __forceinline__ unsigned buf_load<unsigned>(__amdgpu_buffer_rsrc_t rs, unsigned voff, unsigned soff) {
    return __builtin_amdgcn_raw_buffer_load_b32(rs, (int)voff, (int)soff, 0);
}
template <> __device__ __forceinline__ u16 buf_load<u16>(__amdgpu_buffer_rsrc_t rs, unsigned voff, unsigned soff) {
    return __builtin_amdgcn_raw_buffer_load_b16(rs, (int)voff, (int)soff, 0);
}
template <> __device__ __forceinline__ float2 buf_load<float2>(__amdgpu_buffer_rsrc_t rs, unsigned voff, unsigned soff) {
    const uintx2 v = __builtin_amdgcn_raw_buffer_load_b64(rs, (int)voff, (int)soff, 0);
    return make_float2(__uint_as_float(v.x), __uint_as_float(v.y));
}
template <> __device__ __forceinline__ float buf_load<float>(__amdgpu_buffer_rsrc_t rs, unsigned voff, unsigned soff) {
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, (int)voff, (int)soff, 0));
}

// B: tokens a wavefront fetches before it adds (data registers: 1024 threads leave 128 per lane)
template <typename T, int VEC> struct FusedVec;
template <> struct FusedVec<u16, 2> { typedef unsigned type; static constexpr int BATCH = 32; };
template <> struct FusedVec<u16, 1> { typedef u16 type; static constexpr int BATCH = 32; };
template <> struct FusedVec<float, 2> { typedef float2 type; static constexpr int BATCH = 16; };
template <> struct FusedVec<float, 1> { typedef float type; static constexpr int BATCH = 32; };

// Gradient rows through a raw buffer descriptor over the whole gradient matrix (below 4 GB: checked on the host):
// the lane's column offset is one loop-invariant VGPR, the token's row offset a scalar, so a load in flight
// costs its data registers only.
template <typename GV>
struct BufferRows {
    __amdgpu_buffer_rsrc_t rs;
    unsigned voff, row_bytes;
    __device__ __forceinline__ GV operator()(unsigned t) const { return buf_load<GV>(rs, voff, t * row_bytes); }
};
// The same through a 64-bit scalar base per row, for gradients of any size.
template <typename GV>
struct PointerRows {
    const char* base;
    unsigned voff;
    size_t row_bytes;
    __device__ __forceinline__ GV operator()(unsigned t) const {
        return *reinterpret_cast<const GV*>(base + (size_t)t * row_bytes + voff);
    }
};

// Positions past cnt re-read the last valid row; their adds are gated to -0.0f.  For readlane all 64 lanes must have
// taken part in forming `tok`, and the compiler may move that into a branch around the call: nothing here or above it
// may stand in a branch that only some lanes take.  Lanes whose columns lie past h load column 0 and store nothing.
template <int D, typename GV, typename Rows>
__device__ __forceinline__ void load_batch(GV (&v)[D], const Rows& rows, unsigned tok, int cnt) {
#pragma unroll
    for (int u = 0; u < D; ++u) {
        const int idx = u < cnt ? u : cnt - 1;
        v[u] = rows((unsigned)__builtin_amdgcn_readlane((int)tok, idx));
    }
}

constexpr int SHORT_Q = 4, SHORT_TINY = 4;      // runs of up to SHORT_TINY tokens go SHORT_Q at a time

// One wavefront, SHORT_Q runs of at most B tokens (len 0: none): lane u of tok[q] holds the u-th token of run q, d[q] is
// the lane's element of the run's row in the table gradient (any element of it if the lane is not active).  All loads of the
// runs of up to SHORT_TINY tokens, and of the first longer one, are in flight before the first add.
template <typename T, int VEC, typename Rows>
__device__ __forceinline__ void sum_short_runs(const int (&len)[SHORT_Q], const unsigned (&tok)[SHORT_Q],
                                               float* const (&d)[SHORT_Q], bool active, const Rows& rows) {
    typedef typename FusedVec<T, VEC>::type GV;
    constexpr int B = FusedVec<T, VEC>::BATCH, Q = SHORT_Q, TINY = SHORT_TINY;
    // the first run of 5 .. B tokens of this turn (seldom more than one) goes along with the small ones
    int mid = -1;
#pragma unroll
    for (int q = Q - 1; q >= 0; --q)
        if (len[q] > TINY) mid = q;
    unsigned tok_mid = 0;
    float* d_mid = nullptr;
    int len_mid = 0;
#pragma unroll
    for (int q = 0; q < Q; ++q)
        if (q == mid) { tok_mid = tok[q]; d_mid = d[q]; len_mid = len[q]; }
    float acc[Q][VEC], acc_mid[VEC];
    GV few[Q][TINY], v[B];
#pragma unroll
    for (int q = 0; q < Q; ++q)
        if (len[q] >= 1 && len[q] <= TINY) {
            load_acc<VEC>(acc[q], d[q]);
            load_batch<TINY>(few[q], rows, tok[q], len[q]);
        }
    if (mid >= 0) {
        load_acc<VEC>(acc_mid, d_mid);
        load_batch<B>(v, rows, tok_mid, len_mid);
    }
#pragma unroll
    for (int q = 0; q < Q; ++q)
        if (len[q] >= 1 && len[q] <= TINY) {
            add_batch<TINY, VEC>(acc[q], few[q], 0, len[q]);
            if (active) store_acc<VEC>(d[q], acc[q]);
        }
    if (mid >= 0) {
        add_batch<B, VEC>(acc_mid, v, 0, len_mid);
        if (active) store_acc<VEC>(d_mid, acc_mid);
    }
#pragma unroll
    for (int q = 1; q < Q; ++q)
        if (len[q] > TINY && q != mid) {
            load_acc<VEC>(acc_mid, d[q]);
            load_batch<B>(v, rows, tok[q], len[q]);
            add_batch<B, VEC>(acc_mid, v, 0, len[q]);
            if (active) store_acc<VEC>(d[q], acc_mid);
        }
}

// One wavefront, one run: batches of B tokens, the rows of the next batch in flight during the adds of this one.  For runs
// of B + 1 .. MID_BATCHES B tokens where there are many: a workgroup's chain (below) pays a few microseconds of latency per
// run whatever its length, which 16 wavefronts with a run each hide from one another.
constexpr int MID_BATCHES = 8;
constexpr int MID_PER_GROUP = 3;     // more of them per workgroup go to its wavefronts (embed_bwd_fused_kernel)
template <typename T, int VEC, typename Rows, typename TokenAt>
__device__ __forceinline__ void sum_mid_run(int len, float* d, bool active, int lane, const Rows& rows,
                                            const TokenAt& token_at) {
    typedef typename FusedVec<T, VEC>::type GV;
    constexpr int B = FusedVec<T, VEC>::BATCH;
    float acc[VEC];
    GV v0[B], v1[B];
    // 2 B <= 64 tokens at a time, fetched a round ahead
    unsigned tok = lane < 2 * B && lane < len ? token_at(lane) : 0u;
    load_acc<VEC>(acc, d);
    load_batch<B>(v0, rows, tok, len < B ? len : B);
#pragma unroll 1
    for (int j = 0; j < len; j += 2 * B) {
        const int at = j + 2 * B + lane;
        const unsigned tok_n = lane < 2 * B && at < len ? token_at(at) : 0u;
        const int cnt1 = len - j - B < 0 ? 0 : (len - j - B > B ? B : len - j - B);
        if (cnt1 > 0) load_batch<B>(v1, rows, (unsigned)__shfl((int)tok, (lane + B) & 63, 64), cnt1);
        add_batch<B, VEC>(acc, v0, 0, len - j);
        const int cnt2 = len - j - 2 * B;
        if (cnt2 > 0) load_batch<B>(v0, rows, tok_n, cnt2 > B ? B : cnt2);
        if (cnt1 > 0) add_batch<B, VEC>(acc, v1, 0, cnt1);
        tok = tok_n;
    }
    if (active) store_acc<VEC>(d, acc);
}

// Workgroup barrier that orders LDS accesses only: row loads stay in flight across it.
__device__ __forceinline__ void lds_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xC07F);          // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// A run of any length by the whole workgroup of NW (16) wavefronts: chunks of 16 B tokens, wavefront w has tokens
// B w .. B w + B - 1 of a chunk and turn w in the chain, the running sum passes from wavefront to wavefront through
// LDS, so the adds of a column happen in token order and the result equals the in-order loop bit for bit.
// Bound by the row loads at first (one compute unit alone draws little from memory) and by the chain after that: the
// rows of a chunk are requested by all wavefronts at once and while the previous chunk's chain runs, and every
// wavefront turns its rows into floats (-0.0f past cnt) before the chain starts, so that a turn is nothing but
// dependent adds.  token_at(j): token of position j of the run.
template <typename T, int VEC, int NW, typename Rows, typename TokenAt>
__device__ __forceinline__ void sum_long_run(int len, float* d, bool active, int lane, int wave, float* xchg,
                                             const Rows& rows, const TokenAt& token_at) {
    typedef typename FusedVec<T, VEC>::type GV;
    constexpr int B = FusedVec<T, VEC>::BATCH;
    float acc[VEC];
    GV v[B];
    float f[B][VEC];
    __syncthreads();                   // xchg is free again (previous long run)
    if (wave == 0) load_acc<VEC>(acc, d);
    int cnt = len - wave * B;
    cnt = cnt < 0 ? 0 : (cnt > B ? B : cnt);
    {
        const unsigned tok = lane < cnt ? token_at(wave * B + lane) : 0u;
        if (cnt > 0) load_batch<B>(v, rows, tok, cnt);
    }
    for (int c = 0; c < len; c += NW * B) {
        const int turns = len - c > NW * B ? NW : (len - c + B - 1) / B;
        const int first_n = c + NW * B + wave * B;
        const int cnt_n = len - first_n < 0 ? 0 : (len - first_n > B ? B : len - first_n);
        const unsigned tok_n = lane < cnt_n ? token_at(first_n + lane) : 0u;
        if (c == 0 && wave == 0) {
#pragma unroll
            for (int e = 0; e < VEC; ++e) xchg[e * 64 + lane] = acc[e];
        }
        if (cnt > 0) {
#pragma unroll
            for (int u = 0; u < B; ++u) {
#pragma unroll
                for (int e = 0; e < VEC; ++e) f[u][e] = -0.0f;
                add_grad(f[u], v[u], u < cnt);          // -0.0f + x = x for every x
#pragma unroll
                for (int e = 0; e < VEC; ++e) asm volatile("" : "+v"(f[u][e]));   // here, not inside the turn
            }
        }
        if (cnt_n > 0) load_batch<B>(v, rows, tok_n, cnt_n);
        cnt = cnt_n;
        lds_barrier();
#pragma unroll 1
        for (int p = 0; p < turns; ++p) {
            if (wave == p) {
#pragma unroll
                for (int e = 0; e < VEC; ++e) acc[e] = xchg[e * 64 + lane];
#pragma unroll
                for (int u = 0; u < B; ++u)
#pragma unroll
                    for (int e = 0; e < VEC; ++e) acc[e] += f[u][e];
#pragma unroll
                for (int e = 0; e < VEC; ++e) xchg[e * 64 + lane] = acc[e];
            }
            lds_barrier();
        }
    }
    if (wave == 0 && active) {
#pragma unroll
        for (int e = 0; e < VEC; ++e) acc[e] = xchg[e * 64 + lane];
        store_acc<VEC>(d, acc);
    }
}

// Row of the group -> row of its shard's table gradient.  One shard needs neither the division nor the read of the argument
// block that hangs on it, both in the chain of latencies that a turn of the short runs is: 6958 uniform tokens, h = 3664,
// bf16, one shard: 80.7 us with both, 77.0 without; 8192 Zipf-like tokens, h = 4096: 85.1 and 79.5.
template <int P>
__device__ __forceinline__ float* dtable_row(const EmbedBwdGroup<P>& g, unsigned row, unsigned Vs, int h) {
    if constexpr (P == 1) return g.dtable[0] + (size_t)row * h;
    const unsigned s = row / Vs;
    return g.dtable[s] + (size_t)(row - s * Vs) * h;
}

template <typename T, int VEC, int P>
__global__ __launch_bounds__(FUSED_THREADS) void embed_bwd_fused_kernel(EmbedBwdGroup<P> g, const int64_t* __restrict__ ids,
                                                                        int N, int Vs, int n_rows, int64_t off,
                                                                        const T* __restrict__ gout,
                                                                        unsigned grad_bytes, int h, int n_slabs,
                                                                        int n_groups) {
    typedef typename FusedVec<T, VEC>::type GV;
    constexpr int B = FusedVec<T, VEC>::BATCH, Q = SHORT_Q;
    __shared__ __align__(16) unsigned sh[FUSED_MAX_N];      // the keys
    __shared__ unsigned short run_start[FUSED_MAX_N + 2];   // position of the first key of run r; [n_runs] = owned
    __shared__ int wave_cnt[FUSED_MAX_N / 64];
    __shared__ float xchg[64 * VEC];
    __shared__ int s_owned, s_runs, s_mids;
    if (threadIdx.x == 0) { s_owned = 0; s_runs = 0; s_mids = 0; }
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const u64 below = (1ull << lane) - 1ull;

    // keys of the tokens these shards own (all ids requested before the first is used), packed into sh in any
    // order - they are unique and get sorted: one LDS atomic per wavefront
    constexpr int ROUNDS = FUSED_MAX_N / FUSED_THREADS;
    unsigned mine[ROUNDS];
    u64 have[ROUNDS];
#pragma unroll
    for (int q = 0; q < ROUNDS; ++q) {
        const int i = q * FUSED_THREADS + (int)threadIdx.x;
        mine[q] = token_key32<TOKEN_BITS>(ids, i, N, n_rows, off, (unsigned)i);
    }
    int total = 0;
#pragma unroll
    for (int q = 0; q < ROUNDS; ++q) {
        have[q] = __builtin_amdgcn_ballot_w64(mine[q] != KEY32_NONE);
        total += __builtin_popcountll(have[q]);
    }
    int at = 0;
    if (lane == 0 && total) at = atomicAdd(&s_owned, total);
    at = __builtin_amdgcn_readfirstlane(at);
#pragma unroll
    for (int q = 0; q < ROUNDS; ++q) {
        if (mine[q] != KEY32_NONE) sh[at + __builtin_popcountll(have[q] & below)] = mine[q];
        at += __builtin_popcountll(have[q]);
    }
    __syncthreads();
    const int owned = s_owned;
    if (owned == 0) return;
    int m = WAVE_KEYS;
    while (m < owned) m <<= 1;
    for (int t = owned + threadIdx.x; t < m; t += FUSED_THREADS) sh[t] = KEY32_NONE;
    __syncthreads();
    bitonic_sort_lds32(sh, m, lane, wave);

    // Runs of equal rows, numbered by position: every workgroup must arrive at the SAME numbering, because the
    // groups of a slab share the runs out by number.  Run number = how many runs start before the position:
    // ballot per wavefront and round, then an exclusive scan of the ROUNDS * 16 counts by wavefront 0.
    u64 starts[ROUNDS];
#pragma unroll
    for (int q = 0; q < ROUNDS; ++q) {
        const int t = q * FUSED_THREADS + (int)threadIdx.x;
        bool st = false;
        if (t < owned) st = t == 0 || key_row(sh[t - 1]) != key_row(sh[t]);
        starts[q] = __builtin_amdgcn_ballot_w64(st);
        if (lane == 0) wave_cnt[q * FUSED_WAVES + wave] = __builtin_popcountll(starts[q]);
    }
    __syncthreads();
    if (wave == 0) {
        static_assert(ROUNDS * FUSED_WAVES == 128, "two counts per lane");
        const int a = wave_cnt[2 * lane], b2 = wave_cnt[2 * lane + 1];
        int incl = a + b2;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int up = __shfl_up(incl, d, 64);
            if (lane >= d) incl += up;
        }
        wave_cnt[2 * lane] = incl - a - b2;
        wave_cnt[2 * lane + 1] = incl - b2;
        if (lane == 63) {
            s_runs = incl;
            run_start[incl] = (unsigned short)owned;
        }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < ROUNDS; ++q)
        if ((starts[q] >> lane) & 1ull)
            run_start[wave_cnt[q * FUSED_WAVES + wave] + __builtin_popcountll(starts[q] & below)] =
                (unsigned short)(q * FUSED_THREADS + (int)threadIdx.x);
    __syncthreads();
    const int n_runs = s_runs;

    // Runs of B + 1 .. MID_BATCHES B tokens: a wavefront each, or all 16 of a workgroup as the longer ones.  A wavefront alone
    // waits for memory once per batch, a workgroup once per 16 of them, so it is the quicker way until the workgroups of a
    // slab have several such runs each to take in turn.  us, a wavefront each -> a workgroup each (N tokens in V rows, h):
    //   runs per workgroup below 1:  1000, 10, 1024, bf16: 17.8 -> 12.5;  4000, 40, 256: 25.6 -> 19.0
    //   2.5: 8192, 40, 2048: 46.6 -> 37.7;  4 (two shards): 8192, 128, 1024: 35.4 -> 36.6;  6: 8192, 100, 2048: 38.1 -> 44.1
    // Runs of up to 2 B tokens always to a wavefront: 8192, 400, 2048: 37.6 -> 34.5, but 3203, 79, 152: 29.3 -> 32.8 and
    // 7000, 8000, 256 (four shards): 38.7 -> 42.5, because the long runs then start later.
    // (owned - n_runs) / B bounds their number, so that they are seldom counted.
    int mid_max = B;
    if ((owned - n_runs) / B > MID_PER_GROUP * n_groups) {
        int mids = 0;
        for (int r0 = 0; r0 < n_runs; r0 += FUSED_THREADS) {
            const int r = r0 + (int)threadIdx.x;
            bool is_mid = false;
            if (r < n_runs) {
                const int len = (int)run_start[r + 1] - (int)run_start[r];
                is_mid = len > B && len <= MID_BATCHES * B;
            }
            mids += __builtin_popcountll(__builtin_amdgcn_ballot_w64(is_mid));
        }
        if (lane == 0 && mids) atomicAdd(&s_mids, mids);
        __syncthreads();
        if (s_mids > MID_PER_GROUP * n_groups) mid_max = MID_BATCHES * B;
    }

    const int slab = blockIdx.x % n_slabs, group = blockIdx.x / n_slabs;
    const bool active = (slab * 64 + lane) * VEC < h;
    const int c0 = active ? (slab * 64 + lane) * VEC : 0;
    const unsigned row_bytes = (unsigned)h * (unsigned)sizeof(T);
    const unsigned voff = (unsigned)c0 * (unsigned)sizeof(T);
    const BufferRows<GV> rows{__builtin_amdgcn_make_buffer_rsrc((void*)gout, 0, (int)grad_bytes, 0x00020000), voff, row_bytes};

    // short runs: one wavefront each, Q of them per turn
    const int stride = n_groups * FUSED_WAVES;
    for (int r0 = group * FUSED_WAVES + wave; r0 < n_runs; r0 += Q * stride) {
        int len[Q];
        unsigned tok[Q], row[Q];
        float* d[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int r = r0 + q * stride;
            int s = 0;
            len[q] = 0;
            if (r < n_runs) {
                s = run_start[r];
                len[q] = (int)run_start[r + 1] - s;
            }
            s = __builtin_amdgcn_readfirstlane(s);
            len[q] = __builtin_amdgcn_readfirstlane(len[q]);
            if (len[q] > B) len[q] = 0;
            tok[q] = lane < len[q] ? key_token(sh[s + lane]) : 0u;
            row[q] = __builtin_amdgcn_readfirstlane(key_row(sh[s]));
        }
#pragma unroll
        for (int q = 0; q < Q; ++q) d[q] = dtable_row(g, row[q], (unsigned)Vs, h) + c0;
        sum_short_runs<T, VEC>(len, tok, d, active, rows);
    }
    // mid runs: the wavefront looks through its run numbers 64 at a time (a loop of its own: kept over the one above, the
    // positions of mid runs cost it registers)
    if (mid_max > B)
        for (int base = group * FUSED_WAVES + wave; base < n_runs; base += 64 * stride) {
            const int cand = base + lane * stride;
            bool is_mid = false;
            if (cand < n_runs) {
                const int len = (int)run_start[cand + 1] - (int)run_start[cand];
                is_mid = len > B && len <= mid_max;
            }
            u64 todo = __builtin_amdgcn_ballot_w64(is_mid);
            while (todo) {
                const int r = base + __builtin_ctzll(todo) * stride;
                todo &= todo - 1;
                const int s = __builtin_amdgcn_readfirstlane((int)run_start[r]);
                const int len = __builtin_amdgcn_readfirstlane((int)run_start[r + 1]) - s;
                float* const d = dtable_row(g, __builtin_amdgcn_readfirstlane(key_row(sh[s])), (unsigned)Vs, h) + c0;
                sum_mid_run<T, VEC>(len, d, active, lane, rows, [&](int j) { return key_token(sh[s + j]); });
            }
        }
    // long runs: run r belongs to group r % n_groups, all 16 wavefronts of it.  Each wavefront looks through that
    // group's run numbers 64 at a time; LDS holds the same in all of them, so they agree on which runs are long
    // and meet at the same barriers.
    for (int base = 0; base < n_runs; base += 64 * n_groups) {
        const int cand = base + lane * n_groups + group;
        bool is_long = false;
        if (cand < n_runs) is_long = (int)run_start[cand + 1] - (int)run_start[cand] > mid_max;
        u64 todo = __builtin_amdgcn_ballot_w64(is_long);
        while (todo) {
            const int r = base + __builtin_ctzll(todo) * n_groups + group;
            todo &= todo - 1;
            const int s = __builtin_amdgcn_readfirstlane((int)run_start[r]);
            const int len = __builtin_amdgcn_readfirstlane((int)run_start[r + 1]) - s;
            float* const d = dtable_row(g, __builtin_amdgcn_readfirstlane(key_row(sh[s])), (unsigned)Vs, h) + c0;
            sum_long_run<T, VEC, FUSED_WAVES>(len, d, active, lane, wave, xchg, rows,
                                 [&](int j) { return key_token(sh[s + j]); });
        }
    }
}

// ------------------------------------------------------------------------- backward: few tokens
// Up to FEW_MAX_N tokens (and FEW_MAX_WAVES tokens times slabs) nothing is sorted: a wavefront per token and slab of 64 * VEC
// columns looks its row up among all tokens' rows (in LDS, 64 per ballot), has nothing to do if an earlier token has it, and
// else sums the row's tokens in order; rows of many tokens are summed by all wavefronts of its workgroup.  What bounds it is a
// launch, the ids and one round of rows; the sort and the numbering of the runs above take 7 us at any N.  us, the kernel above
// -> this one: 16 tokens, h=1024, fp32, 8 shards 9.5 -> 2.9; 128: 11.4 -> 3.7; 512: 12.2 -> 5.5; 512, h=1001: 11.2 -> 8.3; Zipf, h=4096, bf16,
// 2 shards: 128 tokens 11.8 -> 4.9, 256: 11.6 -> 8.9, 384: 13.5 -> 12.5, 512: 15.0 -> 16.8; every token in one row, h=4096, fp32: 256:
// 13.3 -> 9.5; three rows, h=8192, bf16: 128 tokens 11.7 -> 7.7, 256: 10.4 -> 11.3, 512: 11.6 -> 19.8 (every slab looks through all
// tokens: hence the limit on their product).
constexpr int FEW_MAX_N = 512, FEW_MAX_WAVES = 8192;
constexpr int FEW_WAVES = 8;

template <typename T, int VEC, int P>
__global__ __launch_bounds__(64 * FEW_WAVES) void embed_bwd_few_kernel(EmbedBwdGroup<P> g, const int64_t* __restrict__ ids, int N,
                                                                       int Vs, int n_rows, int64_t off,
                                                                       const T* __restrict__ gout, unsigned grad_bytes, int h) {
    typedef typename FusedVec<T, VEC>::type GV;
    __shared__ int rows_of[FEW_MAX_N];                          // row of token t among those of the launch's shards, or -1
    __shared__ unsigned short list[FEW_WAVES][FEW_MAX_N];       // of each wavefront: the tokens of its row
    __shared__ int long_len[FEW_WAVES], long_row[FEW_WAVES];
    __shared__ float xchg[64 * VEC];
    for (int t = threadIdx.x; t < N; t += 64 * FEW_WAVES) {
        const int64_t loc = ids[t] - off;
        rows_of[t] = loc >= 0 && loc < n_rows ? (int)loc : -1;
    }
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // early tokens, among which the long runs start, in different workgroups, and those of different slabs on different XCDs
    const int i = wave * gridDim.x + (blockIdx.x + blockIdx.y) % gridDim.x;
    const int row = i < N ? __builtin_amdgcn_readfirstlane(rows_of[i]) : -1;
    bool head = row >= 0;
    for (int t0 = 0; head && t0 < i; t0 += 64) {
        const int t = t0 + lane;
        head = !__builtin_amdgcn_ballot_w64(t < i && rows_of[t] == row);
    }
    int len = 0;
    for (int t0 = i & ~63; head && t0 < N; t0 += 64) {
        const int t = t0 + lane;
        const bool mine = t >= i && t < N && rows_of[t] == row;
        const u64 m = __builtin_amdgcn_ballot_w64(mine);
        if (mine) list[wave][len + __builtin_popcountll(m & ((1ull << lane) - 1ull))] = (unsigned short)t;
        len += __builtin_popcountll(m);
    }
    // a wavefront's LDS accesses are executed in order: what its lanes wrote is there for all of them
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const int slab = blockIdx.y;
    const bool active = (slab * 64 + lane) * VEC < h;
    const int c0 = active ? (slab * 64 + lane) * VEC : 0;
    const BufferRows<GV> rows{__builtin_amdgcn_make_buffer_rsrc((void*)gout, 0, (int)grad_bytes, 0x00020000),
                              (unsigned)c0 * (unsigned)sizeof(T), (unsigned)h * (unsigned)sizeof(T)};
    constexpr int LONG = 2 * FusedVec<T, VEC>::BATCH;
    if (lane == 0) {
        long_len[wave] = len > LONG ? len : 0;
        long_row[wave] = row;
    }
    if (len > 0 && len <= LONG) {
        float* const d = dtable_row(g, (unsigned)row, (unsigned)Vs, h) + c0;
        if (len <= SHORT_TINY) {
            const unsigned tok = lane < len ? list[wave][lane] : 0u;
            float acc[VEC];
            GV v[SHORT_TINY];
            load_acc<VEC>(acc, d);
            load_batch<SHORT_TINY>(v, rows, tok, len);
            add_batch<SHORT_TINY, VEC>(acc, v, 0, len);
            if (active) store_acc<VEC>(d, acc);
        } else {
            sum_mid_run<T, VEC>(len, d, active, lane, rows, [&](int j) { return (unsigned)list[wave][j]; });
        }
    }
    // longer runs by all wavefronts of the workgroup: one alone draws too little from memory
    __syncthreads();
    for (int w = 0; w < FEW_WAVES; ++w) {
        const int n = __builtin_amdgcn_readfirstlane(long_len[w]);
        if (n > 0)
            sum_long_run<T, VEC, FEW_WAVES>(n, dtable_row(g, (unsigned)__builtin_amdgcn_readfirstlane(long_row[w]), (unsigned)Vs, h) + c0,
                                            active, lane, wave, xchg, rows, [&](int j) { return (unsigned)list[w][j]; });
    }
}

// ------------------------------------------------------------------------- backward: any number of tokens
// Keys, sort, runs and sums as kernels of their own:
//   1. embed_sort_chunks: chunks of SORT_CHUNK tokens, each sorted by one workgroup as above (32-bit keys: row and
//      position in the chunk), written out as 64-bit keys row << 32 | token; a token of no shard has row NO_ROW.
//   2. embed_merge_ranks: MERGE_WAYS sorted runs of the array become one: the final position of a key is the number of
//      smaller keys in each of them, one binary search per run, all in step (a search is a chain of dependent loads;
//      MERGE_WAYS of them cost the time of one).  One pass up to 32768 tokens, two up to 2^19, ...
//   3. embed_find_runs: where runs of equal rows start, in three lists: up to `batch` tokens, up to MID_BATCHES times
//      that, and above (with the length).
//   4. embed_bwd_accum: the sums; the workgroups of a column slab share the runs of the lists out, the long ones first.
// Bound by gradient and table rows in step 4; steps 1 to 3 are latency.  Measured for 32768 Zipf tokens, h = 4096, bf16,
// 8 shards of 16032 rows: 9 + 19 + 7 + 144 us (0.5 GB).  A sort and an accumulation per shard (16384-key bitonic chunks,
// one workgroup per long run) took 8 x 213 us.
constexpr int SORT_CHUNK = 2048, CHUNK_BITS = 11, MERGE_WAYS = 16;
constexpr int MAX_GROUP_ROWS = (1 << (32 - CHUNK_BITS)) - 1;      // rows of a group: no key equals KEY32_NONE
constexpr unsigned NO_ROW = 0xFFFFFFFFu;
constexpr unsigned MAX_SHORT = 16;                                // short runs of a wavefront in one share

struct RunLists {
    u64* longs;           // length << 32 | start position
    unsigned* shorts;     // start positions
    unsigned* mids;       // start positions
    unsigned* count;      // [3]: shorts, mids, longs
    unsigned* next;       // [3 * n_slabs]: what has been drawn of the short, mid, long runs beyond the first shares, per slab
};

__global__ __launch_bounds__(FUSED_THREADS) void embed_sort_chunks_kernel(const int64_t* __restrict__ ids, int N, int n_rows,
                                                                          int64_t off, u64* __restrict__ keys,
                                                                          unsigned* __restrict__ counters, int n_counters) {
    __shared__ __align__(16) unsigned sh[SORT_CHUNK];
    if (blockIdx.x == 0)
        for (int t = threadIdx.x; t < n_counters; t += FUSED_THREADS) counters[t] = 0u;
    const int base = blockIdx.x * SORT_CHUNK;
    for (int t = threadIdx.x; t < SORT_CHUNK; t += FUSED_THREADS)
        sh[t] = token_key32<CHUNK_BITS>(ids, base + t, N, n_rows, off, (unsigned)t);
    __syncthreads();
    bitonic_sort_lds32(sh, SORT_CHUNK, threadIdx.x & 63, __builtin_amdgcn_readfirstlane(threadIdx.x >> 6));
    for (int t = threadIdx.x; t < SORT_CHUNK; t += FUSED_THREADS) {
        const unsigned k = sh[t];
        // keys stay unique: a key of no shard is told apart by its position
        keys[base + t] = k == KEY32_NONE ? ((u64)NO_ROW << 32) | (unsigned)(base + t)
                                         : ((u64)(k >> CHUNK_BITS) << 32) | (unsigned)(base + (int)(k & (SORT_CHUNK - 1)));
    }
}

// run_len: a power of two times SORT_CHUNK; the last run of the array, and the last group of runs, may be short.
// Bound by the divergent loads of the searches (32768 keys, 16 runs: 38 us with every step in memory), so the first
// steps search 128 samples of each run in LDS, which leaves log2(run_len / 128) steps, most of them in one cache line.
constexpr int MERGE_SAMPLES = 128, MERGE_THREADS = 128;
__global__ __launch_bounds__(MERGE_THREADS) void embed_merge_ranks_kernel(const u64* __restrict__ in, u64* __restrict__ out,
                                                                          int n, int64_t run_len) {
    __shared__ u64 sample[MERGE_WAYS][MERGE_SAMPLES];
    const int e = blockIdx.x * MERGE_THREADS + threadIdx.x;      // n is a multiple of MERGE_THREADS
    const u64 x = in[e];
    const int64_t stride = run_len / MERGE_SAMPLES;
    const int64_t first = (int64_t)e / (run_len * MERGE_WAYS) * (run_len * MERGE_WAYS);     // the same for the workgroup
#pragma unroll
    for (int u = 0; u < MERGE_WAYS; ++u) {
        const int64_t at = first + u * run_len + (threadIdx.x + 1) * stride - 1;
        sample[u][threadIdx.x] = at < n ? in[at] : ~0ull;
    }
    __syncthreads();
    int lo[MERGE_WAYS];                       // keys of run u known to be smaller
#pragma unroll
    for (int u = 0; u < MERGE_WAYS; ++u) lo[u] = 0;
#pragma unroll
    for (int step = MERGE_SAMPLES / 2; step > 0; step >>= 1)
#pragma unroll
        for (int u = 0; u < MERGE_WAYS; ++u)
            if (sample[u][lo[u] + step - 1] < x) lo[u] += step;
#pragma unroll
    for (int u = 0; u < MERGE_WAYS; ++u) {
        lo[u] += sample[u][lo[u]] < x ? 1 : 0;
        lo[u] = (int)(lo[u] * stride);        // run_len: all of them are smaller
    }
    for (int64_t step = stride >> 1; step > 0; step >>= 1) {
#pragma unroll
        for (int u = 0; u < MERGE_WAYS; ++u) {
            const int64_t at = first + u * run_len + lo[u] + step - 1;
            if (lo[u] < run_len && at < n && in[at] < x) lo[u] += (int)step;
        }
    }
    int64_t rank = first;
#pragma unroll
    for (int u = 0; u < MERGE_WAYS; ++u) {
        const int64_t at = first + u * run_len + lo[u];
        rank += lo[u] + (lo[u] < run_len && at < n && in[at] < x ? 1 : 0);
    }
    out[rank] = x;
}

// Appends s to a list for the lanes with `yes`: one atomic per wavefront.
__device__ __forceinline__ void append(unsigned* list, unsigned* count, bool yes, int s, int lane) {
    const u64 m = __builtin_amdgcn_ballot_w64(yes);
    unsigned at = 0;
    if (lane == 0 && m) at = atomicAdd(count, (unsigned)__builtin_popcountll(m));
    at = __builtin_amdgcn_readfirstlane(at);
    if (yes) list[at + __builtin_popcountll(m & ((1ull << lane) - 1ull))] = (unsigned)s;
}

__global__ __launch_bounds__(256) void embed_find_runs_kernel(const u64* __restrict__ keys, int n, int batch, RunLists runs) {
    const int s = blockIdx.x * 256 + threadIdx.x;            // n is a multiple of 256
    const int lane = threadIdx.x & 63;
    const int mid_max = batch * MID_BATCHES;
    const unsigned row = (unsigned)(keys[s] >> 32);
    const unsigned before = s > 0 ? (unsigned)(keys[s - 1] >> 32) : ~row;
    const unsigned after_short = s + batch < n ? (unsigned)(keys[s + batch] >> 32) : NO_ROW;
    const unsigned after_mid = s + mid_max < n ? (unsigned)(keys[s + mid_max] >> 32) : NO_ROW;
    const bool start = row != NO_ROW && before != row;
    const bool is_long = start && after_mid == row;
    const bool is_mid = start && !is_long && after_short == row;
    append(runs.shorts, runs.count, start && !is_mid && !is_long, s, lane);
    append(runs.mids, runs.count + 1, is_mid, s, lane);
    // the length of a long run: its keys are a prefix of keys[s ..], found by the wavefront in steps of 1/64
    u64 lm = __builtin_amdgcn_ballot_w64(is_long);
    while (lm) {
        const int l = __builtin_ctzll(lm);
        lm &= lm - 1;
        const int s0 = __builtin_amdgcn_readlane(s, l);
        const unsigned r0 = (unsigned)__builtin_amdgcn_readlane((int)row, l);
        int lo = s0, width = n - s0, step;             // keys[lo] is of the run, keys[lo + width] is not (or the end)
        do {
            step = (width + 63) / 64;
            const int64_t p = (int64_t)lo + (int64_t)lane * step;
            const bool same = p < n && (unsigned)(keys[p] >> 32) == r0;
            const int c = __builtin_popcountll(__builtin_amdgcn_ballot_w64(same));
            lo += (c - 1) * step;
            width = step;
        } while (step > 1);
        if (lane == 0) runs.longs[atomicAdd(runs.count + 2, 1u)] = ((u64)(unsigned)(lo + 1 - s0) << 32) | (unsigned)s0;
    }
}

// Workgroup (slab, group): 64 * VEC columns.  A draw from a counter that all XCDs add to takes about 50 ns of that counter's
// time, so that a draw per wavefront and list took longer than the sums where a row is few slabs and a slab many
// workgroups.  So a workgroup draws for its 16 wavefronts, its first share of every list is fixed, and without long runs
// (which are what makes workgroups late) all shares are.  us of this kernel, a draw per wavefront -> so: 12000 uniform tokens,
// h = 512, V = 50000, bf16: 150 -> 16; 60000, 1024, 32000: 257 -> 76; 8193 skewed tokens, h = 256: 127 -> 18; 16384 of which
// the shard owns 2048, h = 1024: 101 -> 9.6; 32768 Zipf tokens, h = 4096, 8 shards: 196 -> 144.
template <typename T, int VEC, int P>
__global__ __launch_bounds__(FUSED_THREADS) void embed_bwd_accum_kernel(EmbedBwdGroup<P> g, const u64* __restrict__ keys, int n,
                                                                        RunLists runs, const T* __restrict__ gout, int h,
                                                                        int Vs, int n_slabs) {
    typedef typename FusedVec<T, VEC>::type GV;
    constexpr int B = FusedVec<T, VEC>::BATCH, Q = SHORT_Q;
    __shared__ float xchg[64 * VEC];
    __shared__ unsigned s_next;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int slab = blockIdx.x % n_slabs, group = blockIdx.x / n_slabs;
    const unsigned n_groups = gridDim.x / n_slabs;
    const bool active = (slab * 64 + lane) * VEC < h;
    const int c0 = active ? (slab * 64 + lane) * VEC : 0;
    const PointerRows<GV> rows{(const char*)gout, (unsigned)c0 * (unsigned)sizeof(T), (size_t)h * sizeof(T)};
    const unsigned n_short = runs.count[0], n_mid = runs.count[1], n_long = runs.count[2];

    // Thread 0 draws for the workgroup (start_draw; the others do nothing), all learn the result (end_draw).  (The address is
    // one that the compiler takes for a different one per lane: it would otherwise wait for the result on the spot.)
    auto start_draw = [&](unsigned* counter, unsigned n) {
        asm volatile("" : "+v"(counter));
        return threadIdx.x == 0 ? atomicAdd(counter, n) : 0u;
    };
    auto end_draw = [&](unsigned drawn) {
        __syncthreads();
        if (threadIdx.x == 0) s_next = drawn;
        __syncthreads();
        return (unsigned)__builtin_amdgcn_readfirstlane(s_next);
    };

    for (unsigned r = group; r < n_long;) {
        const u64 run = runs.longs[r];
        const int s = __builtin_amdgcn_readfirstlane((int)(unsigned)run);
        const int len = __builtin_amdgcn_readfirstlane((int)(run >> 32));
        const unsigned row = __builtin_amdgcn_readfirstlane((unsigned)(keys[s] >> 32));
        float* const d = dtable_row(g, row, (unsigned)Vs, h) + c0;
        sum_long_run<T, VEC, FUSED_WAVES>(len, d, active, lane, wave, xchg, rows,
                             [&](int j) { return (unsigned)keys[s + j]; });
        if (n_long <= n_groups) break;
        r = n_groups + end_draw(start_draw(runs.next + 2 * n_slabs + slab, 1u));
    }

    // Workgroup `worker` begins with share `worker` of the mid and of the short runs.  Those that have just had a long run are
    // left out, if they are less than half.  No long runs: the shares that follow are fixed as well; else they are drawn.
    const unsigned busy = 2 * n_long < n_groups ? n_long : 0u, workers = n_groups - busy;
    const bool fixed = n_long == 0;
    auto shares = [&](unsigned n, unsigned share, unsigned* counter, const auto& sum_share) {
        const unsigned drawn_from = workers * share;         // what is beyond the first shares
        const bool draws = !fixed && drawn_from < n;
        unsigned at = (unsigned)group >= busy ? (group - busy) * share
                                              : draws ? drawn_from + end_draw(start_draw(counter, share)) : n;
        while (at < n) {
            const unsigned drawn = draws ? start_draw(counter, share) : 0u;     // (under way while this share is summed)
            sum_share(at);
            at = fixed ? at + drawn_from : draws ? drawn_from + end_draw(drawn) : n;
        }
    };

    shares(n_mid, FUSED_WAVES, runs.next + n_slabs + slab, [&](unsigned at) {
        if (at + wave >= n_mid) return;
        const int s = __builtin_amdgcn_readfirstlane((int)runs.mids[at + wave]);
        const unsigned row = __builtin_amdgcn_readfirstlane((unsigned)(keys[s] >> 32));
        int len = 0;
        for (;;) {
            const int p = s + len + lane;
            const u64 m = __builtin_amdgcn_ballot_w64(p < n && (unsigned)(keys[p] >> 32) == row);
            const int c = m == ~0ull ? 64 : __builtin_ctzll(~m);
            len += c;
            if (c < 64) break;
        }
        sum_mid_run<T, VEC>(len, dtable_row(g, row, (unsigned)Vs, h) + c0, active, lane, rows,
                            [&](int j) { return (unsigned)keys[s + j]; });
    });

    // short runs per wavefront and share: all of them in one share each if that is no more than MAX_SHORT
    unsigned per_wave = (n_short + workers * FUSED_WAVES - 1) / (workers * FUSED_WAVES);
    per_wave = per_wave > MAX_SHORT ? MAX_SHORT : (per_wave + Q - 1) / Q * Q;
    per_wave = per_wave < Q ? Q : per_wave;
    shares(n_short, per_wave * FUSED_WAVES, runs.next + slab, [&](unsigned at) {
        const unsigned first = at + wave * per_wave;
        const unsigned starts = lane < (int)per_wave && first + lane < n_short ? runs.shorts[first + lane] : 0u;
#pragma unroll 1
        for (unsigned q0 = 0; q0 < per_wave && first + q0 < n_short; q0 += Q) {
            u64 key[Q];
            int len[Q];
            unsigned tok[Q], row[Q];
            float* d[Q];
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const int s = __builtin_amdgcn_readlane((int)starts, (int)q0 + q);
                key[q] = s + lane < n && lane <= B ? keys[s + lane] : ~0ull;
            }
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                row[q] = __builtin_amdgcn_readfirstlane((unsigned)(key[q] >> 32));
                const u64 m = __builtin_amdgcn_ballot_w64((unsigned)(key[q] >> 32) == row[q]);
                tok[q] = (unsigned)key[q];
                len[q] = first + q0 + q < n_short ? __builtin_ctzll(~m) : 0;
            }
#pragma unroll
            for (int q = 0; q < Q; ++q) d[q] = dtable_row(g, row[q], (unsigned)Vs, h) + c0;
            sum_short_runs<T, VEC>(len, tok, d, active, rows);
        }
    });
}

static int compute_units() {
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n > 0)
        return n;
    return 256;
}

// The one-kernel path: 32-bit keys, gradient matrix addressable with 32-bit byte offsets.
static bool fused_ok(int64_t N, int64_t h, int64_t Vs, int elem_bytes) {
    return N <= FUSED_MAX_N && Vs <= FUSED_MAX_ROWS && (uint64_t)N * (uint64_t)h * (unsigned)elem_bytes < ((uint64_t)1 << 32);
}

static int64_t padded_tokens(int64_t N) { return ceil_div(N, SORT_CHUNK) * SORT_CHUNK; }

// Workspace of the general path: two key arrays, the run lists, the counters.  (Mid and long runs have more than 16 tokens.)
size_t embed_bwd_workspace(int64_t N, int64_t h, int64_t Vs, int elem_bytes) {
    if (fused_ok(N, h, Vs, elem_bytes)) {      // needs none; the size callers have been told since the first version
        int64_t pow2 = 2;
        while (pow2 < N) pow2 <<= 1;
        return (size_t)pow2 * 12 + 256;
    }
    const size_t n = (size_t)padded_tokens(N);
    return n * (8 + 8 + 4) + n / 16 * (8 + 4) + (3 + 3 * (size_t)ceil_div(h, 64)) * 4;
}

template <typename T, int VEC, int P>
static hipError_t launch_fused(const EmbedBwdGroup<P>& g, const int64_t* ids, int N, int Vs, int n_rows, int64_t off, const T* gout,
                               int h, hipStream_t st) {
    ProfScope prof(K_EMBED_ACCUM, st);
    const int n_slabs = (int)ceil_div(h, 64 * VEC);
    if (N <= FEW_MAX_N && (int64_t)N * n_slabs <= FEW_MAX_WAVES) {
        hipLaunchKernelGGL((embed_bwd_few_kernel<T, VEC, P>), dim3((unsigned)ceil_div(N, FEW_WAVES), (unsigned)n_slabs),
                           dim3(64 * FEW_WAVES), 0, st, g, ids, N, Vs, n_rows, off, gout, (unsigned)((size_t)N * h * sizeof(T)), h);
        return hipGetLastError();
    }
    int n_groups = compute_units() / n_slabs;
    const int want = (int)ceil_div(N, 64);          // no more groups than there could be work for
    if (n_groups > want) n_groups = want;
    if (n_groups < 1) n_groups = 1;
    const unsigned grad_bytes = (unsigned)((size_t)N * h * sizeof(T));
    hipLaunchKernelGGL((embed_bwd_fused_kernel<T, VEC, P>), dim3((unsigned)(n_slabs * n_groups)), dim3(FUSED_THREADS), 0, st, g, ids,
                       N, Vs, n_rows, off, gout, grad_bytes, h, n_slabs, n_groups);
    return hipGetLastError();
}

template <typename T, int VEC, int P>
static hipError_t launch_general(const EmbedBwdGroup<P>& g, const int64_t* ids, int N, int Vs, int n_rows, int64_t off,
                                 const T* gout, int h, void* ws, hipStream_t st) {
    const int n = (int)padded_tokens(N);
    const int n_slabs = (int)ceil_div(h, 64 * VEC);
    u64* a = (u64*)ws;
    u64* b = a + n;
    RunLists runs;
    runs.longs = b + n;
    runs.shorts = (unsigned*)(runs.longs + n / 16);
    runs.mids = runs.shorts + n;
    runs.count = runs.mids + n / 16;
    runs.next = runs.count + 3;
    hipError_t e;
    {
        ProfScope prof(K_EMBED_SORT, st);
        hipLaunchKernelGGL(embed_sort_chunks_kernel, dim3((unsigned)(n / SORT_CHUNK)), dim3(FUSED_THREADS), 0, st, ids, N,
                           n_rows, off, a, runs.count, 3 + 3 * n_slabs);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        for (int64_t len = SORT_CHUNK; len < n; len *= MERGE_WAYS) {
            hipLaunchKernelGGL(embed_merge_ranks_kernel, dim3((unsigned)(n / MERGE_THREADS)), dim3(MERGE_THREADS), 0, st, a, b, n, len);
            if ((e = hipGetLastError()) != hipSuccess) return e;
            u64* t = a; a = b; b = t;
        }
        hipLaunchKernelGGL(embed_find_runs_kernel, dim3((unsigned)(n / 256)), dim3(256), 0, st, a, n,
                           FusedVec<T, VEC>::BATCH, runs);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    ProfScope prof(K_EMBED_ACCUM, st);
    int n_groups = compute_units() / n_slabs;
    const int want = (int)ceil_div(N, 64);
    if (n_groups > want) n_groups = want;
    if (n_groups < 1) n_groups = 1;
    hipLaunchKernelGGL((embed_bwd_accum_kernel<T, VEC, P>), dim3((unsigned)(n_slabs * n_groups)), dim3(FUSED_THREADS), 0, st, g, a,
                       n, runs, gout, h, Vs, n_slabs);
    return hipGetLastError();
}

template <typename T, int VEC, int P>
static hipError_t launch_bwd_part(float* const* dtables, const int64_t* ids, int n, int N, int Vs, int64_t off, const T* gout, int h,
                                  bool fused, void* ws, hipStream_t st) {
    EmbedBwdGroup<P> g{};
    for (int s = 0; s < n; ++s) g.dtable[s] = dtables[s];
    return fused ? launch_fused<T, VEC, P>(g, ids, N, Vs, n * Vs, off, gout, h, st)
                 : launch_general<T, VEC, P>(g, ids, N, Vs, n * Vs, off, gout, h, ws, st);
}

template <typename T, int VEC>
static hipError_t launch_bwd_group(float* const* dtables, const int64_t* ids, int p, int N, int Vs, int64_t off, const T* gout,
                                   int h, void* ws, hipStream_t st) {
    const bool fused = fused_ok(N, h, Vs, (int)sizeof(T));
    // shards per launch: as many as the key width and the argument block hold
    int per = (fused ? FUSED_MAX_ROWS : MAX_GROUP_ROWS) / Vs;
    if (per > EMBED_GROUP_MAX) per = EMBED_GROUP_MAX;
    for (int s0 = 0; s0 < p; s0 += per) {
        const int n = p - s0 < per ? p - s0 : per;
        const int64_t first = off + (int64_t)s0 * Vs;
        const hipError_t e =
            n == 1 ? launch_bwd_part<T, VEC, 1>(dtables + s0, ids, n, N, Vs, first, gout, h, fused, ws, st)
                   : launch_bwd_part<T, VEC, EMBED_GROUP_MAX>(dtables + s0, ids, n, N, Vs, first, gout, h, fused, ws, st);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_embed_bwd(const void* gout, const int64_t* ids, int p, int N, int h, int Vs, int64_t off, int is_bf16,
                            float* const* dtables, void* ws, hipStream_t st) {
    if (is_bf16) return h % 2 == 0 ? launch_bwd_group<u16, 2>(dtables, ids, p, N, Vs, off, (const u16*)gout, h, ws, st)
                                   : launch_bwd_group<u16, 1>(dtables, ids, p, N, Vs, off, (const u16*)gout, h, ws, st);
    return h % 2 == 0 ? launch_bwd_group<float, 2>(dtables, ids, p, N, Vs, off, (const float*)gout, h, ws, st)
                      : launch_bwd_group<float, 1>(dtables, ids, p, N, Vs, off, (const float*)gout, h, ws, st);
}

}  // namespace vp
