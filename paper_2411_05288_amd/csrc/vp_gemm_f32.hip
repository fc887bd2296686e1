// fp32 path of the output layer: fp32 products on the matrix cores (v_mfma_f32_32x32x2_f32: fp32
// operands, fp32 products and accumulation) with arbitrary operand layouts.  It serves the three
// products of section 4.2 for fp32 storage:  Y = X W^T,  dX += D W,  dW = D^T X.
//
// C[m, n] (+)= sum_k A(m, k) * B(n, k), each operand stored K-contiguous ([rows][K]) or K-strided
// ([K][rows]).
//
// What bounds it: the fp32 matrix rate (157 TFLOP/s dense; one MFMA keeps a SIMD's matrix core busy
// for 64 cycles and needs one operand register per side, so LDS and load traffic are light).  A
// vector-ALU version of this kernel (64 x 64 tiles, no double buffering) took 411 us per product of
// N=1000, h=1024, Vs=4000 (20 TFLOP/s); this one takes 88 us on the outputs of 256 tiles of 128 x 128
// (one workgroup per compute unit, 94 TFLOP/s) and 120 us on the 1000 x 1024 output.
//
// Workgroup: 4 wavefronts (2 x 2) on a TM x TN tile, TM = TN = 128 (64 x 64 per wavefront) or 64.
// K advances 32 at a time through two LDS stages; the global loads of step k + 1 are in flight in
// registers while step k is multiplied (4096 cycles at 128 x 128), one barrier per step; two
// workgroups share a compute unit and fill each other's barriers.
//
// LDS: K-contiguous tile [rows][32 + 4]: one ds_read_b128 gives four k of one row, and lanes 32-63
// take the next four, so MFMA step j of a group multiplies k = j and k = 4 + j (the order of the k
// does not matter as long as both operands use it).  K-strided tile [32][rows + 8]: one ds_read_b32
// per step; 4 * (rows + 8) words are 32 banks apart, so both lane halves fall into different banks.
//
// Small outputs with a long K (dX of the tiny configuration: 128 x 256 outputs, K = 4096) would
// occupy a handful of compute units.  With scratch memory the K range is cut into S slices
// (grid.y); every slice writes its partial tile to scratch[z], and a second kernel adds the S
// partials in a fixed order (results repeat bit for bit).
#include <climits>

#include "vp_internal.h"

namespace vp {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef unsigned uintx4 __attribute__((ext_vector_type(4)));

constexpr int FK = 32;             // K step
constexpr int F_THREADS = 256;
constexpr unsigned F_OOB = 0x80000000u;   // beyond every buffer descriptor below (each covers at most 2^29 bytes)

struct GemmF32Params {
    const float* A;
    const float* B;
    float* C;
    int64_t lda, ldb, ldc;
    int M, N, K;
    int a_vec, b_vec;              // not 0: 16-byte loads allowed (rows 16-byte aligned, and if K-contiguous K % 4 == 0
                                   // or zeros behind the row's last element up to a multiple of 4)
    int accumulate;
    int k_per_slice, slices;       // of one shard
    int64_t slice_stride;          // floats between the partial outputs of consecutive slices
    // shards: n of them; along N or M `first` is the first tile column / row of each (INT_MAX from n on) and `total` all of
    // them, along K a slice belongs to one shard (slice z to shard z / slices)
    int n, total;
    int first[GEMM_GROUP_MAX];
    GemmF32Shard sh[GEMM_GROUP_MAX];
};

template <bool KC, int ROWS>
struct F32Tile {
    static constexpr int RS = KC ? FK + 4 : ROWS + 8;                // row stride in floats
    static constexpr int FLOATS = KC ? ROWS * RS : FK * RS;
    static constexpr int CHUNKS = ROWS * FK / 4 / F_THREADS;         // 16-byte chunks per thread
};

template <bool KC, int ROWS>
using F32Chunks = uintx4[F32Tile<KC, ROWS>::CHUNKS];

// Global -> registers for one ROWS x FK operand tile.  Out-of-range elements come back as zeros: the
// descriptor covers exactly the rows of this tile that exist (K-contiguous) or the k-rows that exist
// (K-strided), and elements past the end of a K-contiguous row get an offset beyond it.  (Rows past the
// end of a K-strided operand read the neighbouring k-row: finite values for outputs never stored.)
template <bool KC, int ROWS>
__device__ __forceinline__ void f32_load(F32Chunks<KC, ROWS>& r, const float* p, int64_t ld, int r0,
                                         int k0, int rows, int k_end, int vec, int tid) {
    constexpr int CPR = KC ? FK / 4 : ROWS / 4;     // chunks per stored row of the tile
    const float* base = KC ? p + (int64_t)r0 * ld + k0 : p + (int64_t)k0 * ld + r0;
    const int left = KC ? rows - r0 : k_end - k0;   // stored rows that exist from here on
    const int have = left < 0 ? 0 : (left < (KC ? ROWS : FK) ? left : (KC ? ROWS : FK));
    // bytes from `base` to the end of the last existing stored row
    const int64_t in_row = KC ? (int64_t)k_end - k0 : (int64_t)rows - r0;
    const int64_t bytes = have > 0 && in_row > 0 ? (((int64_t)have - 1) * ld + in_row) * 4 : 0;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, (int)bytes, 0x00020000);
#pragma unroll
    for (int i = 0; i < F32Tile<KC, ROWS>::CHUNKS; ++i) {
        const int q = tid + F_THREADS * i;
        const int row = q / CPR, c = (q % CPR) * 4;
        const unsigned off = ((unsigned)row * (unsigned)ld + (unsigned)c) * 4u;
        if (vec) {
            r[i] = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)(KC && k0 + c >= k_end ? F_OOB : off), 0, 0);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                r[i][e] = __builtin_amdgcn_raw_buffer_load_b32(
                    rs, (int)(KC && k0 + c + e >= k_end ? F_OOB : off + 4u * e), 0, 0);
        }
    }
}

template <bool KC, int ROWS>
__device__ __forceinline__ void f32_store(const F32Chunks<KC, ROWS>& r, float* s, int tid) {
    constexpr int CPR = KC ? FK / 4 : ROWS / 4;
#pragma unroll
    for (int i = 0; i < F32Tile<KC, ROWS>::CHUNKS; ++i) {
        const int q = tid + F_THREADS * i;
        *reinterpret_cast<uintx4*>(s + (q / CPR) * F32Tile<KC, ROWS>::RS + (q % CPR) * 4) = r[i];
    }
}

// The four k values (8q + 4 hf .. + 3) of tile row `row`
template <bool KC, int ROWS>
__device__ __forceinline__ floatx4 f32_frag(const float* s, int row, int q, int hf) {
    constexpr int RS = F32Tile<KC, ROWS>::RS;
    if (KC) return *reinterpret_cast<const floatx4*>(s + row * RS + 8 * q + 4 * hf);
    floatx4 v;
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = s[(8 * q + 4 * hf + j) * RS + row];
    return v;
}

template <bool A_KC, bool B_KC, int TM, int TN>
__global__ __launch_bounds__(F_THREADS, TM == 128 ? 2 : 4) void gemm_f32_kernel(GemmF32Params g) {
    constexpr int MT = TM / 64, NT = TN / 64;            // 32 x 32 MFMA tiles per wavefront and direction
    typedef F32Tile<A_KC, TM> TA;
    typedef F32Tile<B_KC, TN> TB;
    __shared__ __attribute__((aligned(16))) float sA[2][TA::FLOATS];
    __shared__ __attribute__((aligned(16))) float sB[2][TB::FLOATS];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1, l32 = lane & 31, hf = lane >> 5;

    // Tiles in panels of 8 tile rows, column by column; workgroups are dealt to the 8 XCDs round-robin, so
    // every XCD takes a contiguous run of tiles and shares the operand panels of its run in its L2.
    constexpr bool CAT_N = A_KC && B_KC, CAT_M = !A_KC && !B_KC, CAT_K = A_KC && !B_KC;
    const int tiles_m = CAT_M ? g.total : (g.M + TM - 1) / TM, tiles_n = CAT_N ? g.total : (g.N + TN - 1) / TN;
    const int total = tiles_m * tiles_n, b = blockIdx.x;
    const int x = b & 7, per = total >> 3, rem = total & 7;
    const int t = x * per + (x < rem ? x : rem) + (b >> 3);
    const int panel = t / (8 * tiles_n), in_panel = t - panel * 8 * tiles_n;
    const int prows = min(8, tiles_m - panel * 8);
    int tile_m = panel * 8 + in_panel % prows, tile_n = in_panel / prows;

    // the shard of this tile (or slice), its operands and its part of the output
    int shard = CAT_K ? blockIdx.y / g.slices : 0;
    const int slice = CAT_K ? blockIdx.y - shard * g.slices : blockIdx.y;
    if (!CAT_K) {
        const int tc = CAT_N ? tile_n : tile_m;
#pragma unroll
        for (int i = 1; i < GEMM_GROUP_MAX; ++i) shard += tc >= g.first[i] ? 1 : 0;
        if (CAT_N) tile_n -= g.first[shard];
        else tile_m -= g.first[shard];
    }
    const GemmF32Shard& s = g.sh[shard];
    const float* A = CAT_N ? g.A : s.A;
    const float* B = CAT_M ? g.B : s.B;
    const int64_t lda = CAT_N ? g.lda : s.ld, ldc = CAT_N ? s.ld : g.ldc;
    const int M = CAT_M ? s.rows : g.M, N = CAT_N ? s.rows : g.N, K = CAT_K ? s.rows : g.K;
    const int m0 = tile_m * TM, n0 = tile_n * TN;
    // slice of the K range; with one slice this is all of K and C is the real output (a short shard's last slices are empty)
    const int k_begin = min(K, slice * g.k_per_slice);
    const int k_end = min(K, k_begin + g.k_per_slice);
    float* C = (CAT_K ? g.C : s.C) + (int64_t)blockIdx.y * g.slice_stride;

    floatx16 acc[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    uintx4 ra[TA::CHUNKS], rb[TB::CHUNKS];
    f32_load<A_KC, TM>(ra, A, lda, m0, k_begin, M, k_end, g.a_vec, tid);
    f32_load<B_KC, TN>(rb, B, g.ldb, n0, k_begin, N, k_end, g.b_vec, tid);
    f32_store<A_KC, TM>(ra, sA[0], tid);
    f32_store<B_KC, TN>(rb, sB[0], tid);
    __syncthreads();
    int cur = 0;
    for (int k0 = k_begin; k0 < k_end; k0 += FK, cur ^= 1) {
        const bool more = k0 + FK < k_end;
        if (more) {
            f32_load<A_KC, TM>(ra, A, lda, m0, k0 + FK, M, k_end, g.a_vec, tid);
            f32_load<B_KC, TN>(rb, B, g.ldb, n0, k0 + FK, N, k_end, g.b_vec, tid);
        }
#pragma unroll
        for (int q = 0; q < FK / 8; ++q) {
            floatx4 a[MT], bb[NT];
#pragma unroll
            for (int i = 0; i < MT; ++i) a[i] = f32_frag<A_KC, TM>(sA[cur], (wm * MT + i) * 32 + l32, q, hf);
#pragma unroll
            for (int j = 0; j < NT; ++j) bb[j] = f32_frag<B_KC, TN>(sB[cur], (wn * NT + j) * 32 + l32, q, hf);
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int i = 0; i < MT; ++i)
#pragma unroll
                    for (int j = 0; j < NT; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i][e], bb[j][e], acc[i][j], 0, 0, 0);
        }
        if (more) {     // the other stage was last read before the previous barrier
            f32_store<A_KC, TM>(ra, sA[cur ^ 1], tid);
            f32_store<B_KC, TN>(rb, sB[cur ^ 1], tid);
        }
        __syncthreads();
    }

    // register r of lane l of a tile holds C[8 (r/4) + 4 (l/32) + r%4][l%32]: 128 contiguous bytes per row and store
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            const int col = n0 + (wn * NT + j) * 32 + l32;
            const int row0 = m0 + (wm * MT + i) * 32 + 4 * hf;
            if (col >= N) continue;
            float* c = C + (int64_t)row0 * ldc + col;
            if (g.accumulate) {
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int dr = 8 * (r >> 2) + (r & 3);
                    if (row0 + dr < M) acc[i][j][r] += c[(int64_t)dr * ldc];
                }
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int dr = 8 * (r >> 2) + (r & 3);
                if (row0 + dr < M) c[(int64_t)dr * ldc] = acc[i][j][r];
            }
        }
}

// K slices for an output of this many 64 x 64 tiles: enough workgroups to cover the chip, slices of at least min_k.
static int slices_for(int64_t tiles, int64_t K, int64_t min_k) {
    int64_t S = 256 / tiles;
    if (S > 32) S = 32;
    if (S > K / min_k) S = K / min_k;
    return S < 2 ? 1 : (int)S;
}
static int splitk_slices(int64_t M, int64_t N, int64_t K) { return slices_for(ceil_div(M, 64) * ceil_div(N, 64), K, 64); }
// Logits and dW of a group.  A K step of 32 takes 0.55 us where a workgroup has a compute unit to itself; the sum of the
// slices is another launch, 3 us of host time in passes that the host bounds.  So slices of at least 256, from K = 1024 on.
// 32 tiles, product and forward pass, us, in one chain -> in slices: K = 512: 19.3 -> 15.4 and 28.0 -> 31.2; 640: 22.4 ->
// 17.2 and 27.8 -> 30.6; 800: 26.5 -> 16.5 and 30.6 -> 31.0; 1024: 32.4 -> 15.9 and 36.9 -> 30.5; 2048: 58 -> 17 and 63 -> 30.
int gemm_f32_group_slices(int64_t tiles, int64_t K) { return K < 1024 ? 1 : slices_for(tiles, K, 256); }
// A product cut in S slices advances in steps of FK.
static int slice_length(int64_t K, int S) { return S > 1 ? (int)(ceil_div(ceil_div(K, S), FK) * FK) : (int)K; }

size_t gemm_f32_scratch_floats(int64_t M, int64_t N, int64_t K) {
    const int S = splitk_slices(M, N, K);
    return S > 1 ? (size_t)S * (size_t)M * (size_t)N : 0;
}

template <bool A_KC, bool B_KC>
static void launch_f32_t(GemmF32Params& g, int tile, hipStream_t st) {
    int64_t tm = ceil_div(g.M, tile), tn = ceil_div(g.N, tile), cat = 0;
    for (int r = 0; r < GEMM_GROUP_MAX; ++r) {
        g.first[r] = r < g.n ? (int)cat : INT_MAX;
        if (r < g.n) cat += ceil_div(g.sh[r].rows, tile);
    }
    g.total = (int)cat;
    int z = g.slices;
    if (A_KC && B_KC) tn = cat;
    else if (!A_KC) tm = cat;
    else z *= g.n;
    const dim3 grid((unsigned)(tm * tn), (unsigned)z);
    if (tile == 128)
        hipLaunchKernelGGL((gemm_f32_kernel<A_KC, B_KC, 128, 128>), grid, dim3(F_THREADS), 0, st, g);
    else
        hipLaunchKernelGGL((gemm_f32_kernel<A_KC, B_KC, 64, 64>), grid, dim3(F_THREADS), 0, st, g);
}

// Launches the product; C is [M, N] with row stride ldc where the shards share the output (dH).  With more than one K slice
// (dH: of all shards together) the partial outputs go through scratch, every slice laid out like the output, or like the
// outputs of the shards one behind the other.
static hipError_t launch_f32(GemmF32Params g, bool a_kc, bool b_kc, float* C, int64_t ldc, bool accumulate, float* scratch,
                             hipStream_t st) {
    const bool cat_n = a_kc && b_kc, cat_k = a_kc && !b_kc;
    const int parts = g.slices * (cat_k ? g.n : 1);
    // workgroups of 128 x 128 tiles; these (half the LDS and load traffic per flop) once every compute unit gets one
    int64_t wg = 0;
    for (int r = 0; r < g.n; ++r) {
        if (cat_n) wg += ceil_div(g.M, 128) * ceil_div(g.sh[r].rows, 128);
        else if (cat_k) wg += ceil_div(g.M, 128) * ceil_div(g.N, 128);
        else wg += ceil_div(g.sh[r].rows, 128) * ceil_div(g.N, 128);
    }
    // (slices of logits and dW are counted in 64 x 64 tiles: gemm_f32_group_slices)
    const int tile = wg * g.slices >= 256 && (cat_k || g.slices == 1) ? 128 : 64;
    g.C = C;
    if (!cat_n) g.ldc = ldc;
    g.accumulate = accumulate ? 1 : 0;
    SumList l{};
    if (parts > 1) {
        l.n = cat_k ? 1 : g.n;
        for (int r = 0; r < l.n; ++r) {
            GemmF32Shard& s = g.sh[r];
            l.first[r] = g.slice_stride;
            l.count[r] = cat_n ? (int64_t)g.M * s.ld : cat_k ? (int64_t)g.M * ldc : (int64_t)s.rows * ldc;
            l.C[r] = cat_k ? C : s.C;
            if (!cat_k) s.C = scratch + l.first[r];
            g.slice_stride += l.n == 1 ? l.count[r] : (l.count[r] + 3) / 4 * 4;
        }
        g.C = scratch;
        g.accumulate = 0;
    }
    if (cat_n) launch_f32_t<true, true>(g, tile, st);
    else if (cat_k) launch_f32_t<true, false>(g, tile, st);
    else if (!b_kc) launch_f32_t<false, false>(g, tile, st);
    else return hipErrorInvalidValue;
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || parts == 1) return e;
    return launch_sum_slices(scratch, parts, g.slice_stride, l, accumulate, st);
}

hipError_t launch_gemm_f32(const float* A, int64_t sam, int64_t sak, const float* B, int64_t sbn, int64_t sbk,
                           float* C, int64_t ldc, int M, int N, int K, bool accumulate, float* scratch,
                           hipStream_t st) {
    if (M <= 0 || N <= 0 || K <= 0) return hipErrorInvalidValue;
    if ((sam != 1 && sak != 1) || (sbn != 1 && sbk != 1)) return hipErrorInvalidValue;
    ProfScope prof(K_GEMM_F32, st);
    // (a matrix of one column, or one row, is K-contiguous and K-strided at once: B is then taken as A is, because a
    // K-strided A with a K-contiguous B is the one pair that is not instantiated - dW of hidden size 1)
    const bool a_kc = sak == 1, b_kc = sbk == 1 && (a_kc || sbn != 1);
    GemmF32Params g{};
    g.A = A; g.B = B;
    g.lda = a_kc ? sam : sak; g.ldb = b_kc ? sbn : sbk;
    g.M = M; g.N = N; g.K = K;
    g.k_per_slice = slice_length(K, scratch ? splitk_slices(M, N, K) : 1);
    g.slices = (int)ceil_div(K, g.k_per_slice);
    g.a_vec = g.lda % 4 == 0 && ((uintptr_t)A & 15u) == 0 && (!a_kc || K % 4 == 0);
    g.b_vec = g.ldb % 4 == 0 && ((uintptr_t)B & 15u) == 0 && (!b_kc || K % 4 == 0);
    g.n = 1;
    GemmF32Shard& s = g.sh[0];
    s.A = A; s.B = B; s.C = C;
    s.rows = a_kc && b_kc ? N : a_kc ? K : M;
    s.ld = (int)(a_kc && b_kc ? ldc : g.lda);
    return launch_f32(g, a_kc, b_kc, C, ldc, accumulate, scratch, st);
}

// The three products over n shards (see GemmBf16Group for how they are laid end to end; here a K slice never crosses a
// shard, so a sum runs over at most one shard's K before it meets the others in ascending order, as with one call per
// shard).  D_r has rows of ld elements, zero behind the shard's columns, a multiple of four: 16-byte loads for any row count.
// Logits and dW are cut into K slices where the tiles of all shards leave compute units idle, as in a call per shard.  One
// launch for all shards with a single chain over K, and with slices: forward pass of N=16 h=2048 V=2000 p=2: 62 -> 31 us,
// N=64 h=2048 V=1024 p=2: 62 -> 31, backward pass of N=2048 h=64 V=2000 p=16: 93 -> 56.
hipError_t launch_gemm_f32_logits(const float* H, int64_t N, int64_t h, const GemmF32Shard* sh, int n, int slices, float* scratch,
                                  hipStream_t st) {
    ProfScope prof(K_GEMM_F32, st);
    GemmF32Params g{};
    g.A = H;
    g.lda = g.ldb = h;
    g.M = (int)N; g.K = (int)h;
    g.a_vec = g.b_vec = h % 4 == 0 ? 1 : 0;
    g.k_per_slice = slice_length(h, slices);
    g.slices = (int)ceil_div(h, g.k_per_slice);
    g.n = n;
    for (int r = 0; r < n; ++r) g.sh[r] = sh[r];
    return launch_f32(g, true, true, nullptr, 0, false, scratch, st);
}

hipError_t launch_gemm_f32_dh(int64_t N, int64_t h, const GemmF32Shard* sh, int n, int slices, float* dH, bool accumulate,
                              float* scratch, hipStream_t st) {
    ProfScope prof(K_GEMM_F32, st);
    GemmF32Params g{};
    g.ldb = h;
    g.M = (int)N; g.N = (int)h;
    int rows = 0;
    for (int r = 0; r < n; ++r) {
        g.sh[r] = sh[r];
        rows = sh[r].rows > rows ? sh[r].rows : rows;
    }
    g.a_vec = 1;
    g.b_vec = h % 4 == 0 ? 1 : 0;
    g.slices = slices;
    g.k_per_slice = (int)(ceil_div(ceil_div(rows, slices), FK) * FK);
    g.n = n;
    return launch_f32(g, true, false, dH, h, accumulate, scratch, st);
}

hipError_t launch_gemm_f32_dw(const float* H, int64_t N, int64_t h, const GemmF32Shard* sh, int n, int slices, float* scratch,
                              hipStream_t st) {
    ProfScope prof(K_GEMM_F32, st);
    GemmF32Params g{};
    g.B = H;
    g.ldb = h;
    g.N = (int)h; g.K = (int)N;
    g.a_vec = 1;
    g.b_vec = h % 4 == 0 ? 1 : 0;
    g.k_per_slice = slice_length(N, slices);
    g.slices = (int)ceil_div(N, g.k_per_slice);
    g.n = n;
    for (int r = 0; r < n; ++r) g.sh[r] = sh[r];
    return launch_f32(g, false, false, nullptr, h, false, scratch, st);
}

// K slices per shard of a grouped dH product: one if 128 x 128 tiles of all shards fill the chip; else slices of at least
// 512 k that make them do so; else 64 x 64 tiles, up to two workgroups per compute unit, slices of at least 64.
int gemm_f32_dh_slices(int64_t N, int64_t h, int64_t rows, int n) {
    const int64_t big = ceil_div(N, 128) * ceil_div(h, 128) * n, small = ceil_div(N, 64) * ceil_div(h, 64) * n;
    const int64_t S = ceil_div(256, big);
    if (rows / S >= 512 || S == 1) return (int)S;
    int64_t S64 = 512 / small;
    if (S64 > rows / 64) S64 = rows / 64;
    if (S64 > 32) S64 = 32;
    return S64 < 1 ? 1 : (int)S64;
}

}  // namespace vp
