// fp32 path of the output layer: fp32 products on the bf16 matrix cores, with arbitrary operand layouts.  It serves the three
// products of section 4.2 for fp32 storage:  Y = X W^T,  dX += D W,  dW = D^T X.
//
// C[m, n] (+)= sum_k A(m, k) * B(n, k), each operand stored K-contiguous ([rows][K]) or K-strided ([K][rows]).
//
// What bounds it: the matrix cores.  v_mfma_f32_32x32x2_f32 gives 157 TFLOP/s, the bf16 instruction sixteen times as much, so
// every operand is split exactly into three bf16 parts, x = x0 + x1 + x2 (8 significant bits each, 24 together), and of
// the nine products of parts the six largest are summed in fp32 accumulators: x0 y0, x0 y1, x1 y0, x1 y1 (at most 2^-16 of the
// whole), x0 y2, x2 y0 (2^-17).  What is left out is at most 2^-24 of a product (both operands just above a power of two; 2^-27 in
// the root mean square); and one bf16 MFMA adds 16 products at once, so that a sum is rounded six times per 16 k instead of
// eight.  Sums of at most four products, in which what is left out would show (one product: 3.9e-8 instead of 2.5e-8), are formed
// with the fp32 instruction; from five on both the 2-norm of the error and the largest of 630000 are smaller than its own (K = 5: 4.3e-8
// -> 3.2e-8, 16: 7.4e-8 -> 3.4e-8, 256: 2.9e-7 -> 1.7e-7).  Error of the results against float64 (2-norm, relative; fp32 MFMA -> this kernel): N=1000 h=1024 V=32000 p=8: logits 5.7e-7 -> 4.9e-7, dH 1.1e-6 -> 5.0e-7, dW
// 5.7e-7 -> 3.6e-7; N=128 h=256 V=8192: 2.9e-7 -> 2.4e-7, 2.1e-7 -> 1.9e-7, 2.0e-7 -> 1.4e-7; N=2000 h=2048 V=8000: 8.1e-7 ->
// 7.0e-7, 1.1e-6 -> 5.0e-7, 8.0e-7 -> 5.1e-7.  Time of a product at the first of these sizes: 520-560 us -> 330-350 us
// (200 TFLOP/s of fp32 work, 1.2 PFLOP/s of the matrix cores'); whole step 1700 -> 1040 us.
//
// Workgroup: 4 wavefronts (2 x 2) on tiles of 256 x 128 (dW: vocabulary rows first) or 128 x 256 (tokens first), 128 x 128 or
// 64 x 64.  Operands go global -> registers (fp32) -> split -> LDS (three bf16 planes), K advances 16 (small tiles: 32) at a
// time through two LDS stages with one barrier each: while stage q is multiplied, stage q + 1 is split between its products
// (6.5 vector instructions per value, one of them the scaling, which issue while the matrix cores work; left to the compiler they
// came in one block, 363 instead of 328 us; the two values of a pair converted apart from one another, 10.5 instructions, 1082
// instead of 1047 us for the whole step of the first size above) and stage q + 2 is on its way into the freed registers.  Two workgroups of the large
// tiles (three of the others) share a compute unit and fill each other's barriers.  The split happens once per workgroup and
// value: with every wavefront splitting what it loads, without LDS, small launches took as long and large ones 1.3 times.
//
// LDS planes: K-contiguous tile [rows][16 or 32 k], one ds_read_b128 per MFMA operand; K-strided tile [k][rows], two
// transposing reads (ds_read_b64_tr_b16) per operand.
//
// Small outputs with a long K (dX of the tiny configuration: 128 x 256 outputs, K = 4096) would
// occupy a handful of compute units.  With scratch memory the K range is cut into S slices
// (grid.y); every slice writes its partial tile to scratch[z], and a second kernel adds the S
// partials in a fixed order (results repeat bit for bit).
#include <climits>

#include "vp_internal.h"

namespace vp {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short short4v __attribute__((ext_vector_type(4)));
typedef unsigned uintx4 __attribute__((ext_vector_type(4)));

// Operands are scaled by this before they are split, and the sums by the square of its inverse (all exact): the last bit of the
// smallest fp32 number is then a normal bf16 number, so that the three parts hold every finite operand exactly.  (Scaled operands
// from 2^128 on and sums from 2^80 on are not finite and are computed again: f32_again.)
constexpr float IN_SCALE = 0x1p24f;

__device__ __forceinline__ unsigned pack_bf16(float lo, float hi) {      // round to nearest even, one instruction
    typedef float floatx2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(unsigned, __builtin_convertvector((floatx2{lo, hi}), bf16x2));
}

constexpr int F_THREADS = 256;
constexpr int F_FEW = 5;                  // sums of fewer products than this: the fp32 instruction
constexpr unsigned F_OOB = 0x80000000u;   // beyond every buffer descriptor below (each covers at most 2^30 bytes)

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

// One operand's part of a tile: ROWS rows by SK of the K dimension, fetched by THREADS threads.
template <bool KC, int ROWS, int SK, int THREADS = F_THREADS>
struct F32Tile {
    static constexpr int RB = KC ? 2 * SK : 2 * ROWS;                // bytes per stored row of a plane
    static constexpr int PLANE = 2 * ROWS * SK;                      // bytes per bf16 plane; three planes
    static constexpr int CHUNKS = ROWS * SK / 4 / THREADS;           // 16-byte chunks of fp32 per thread
    static constexpr int CPR = KC ? SK / 4 : ROWS / 4;               // chunks per stored row

    // K-contiguous: position of the 16-byte chunk c (eight k) of row r within its row of SK * 2 bytes, so that the 16 rows
    // that a pass of ds_read_b128 serves fall into different banks
    static __device__ __forceinline__ int chunk_at(int r, int c) { return SK == 16 ? c ^ ((r >> 3) & 1) : SK == 32 ? c ^ ((r >> 2) & 3) : c ^ ((r >> 1) & 7); }
    // K-strided: position of the 32-byte segment s (16 rows) of k-row k, so that the four k-rows by two segments that a
    // pass of the transposing read serves fall into different banks
    static __device__ __forceinline__ int seg_at(int k, int s) {
        return ROWS == 64 ? s ^ (k & 2) : s ^ ((k & 3) ^ ((k & 1) << 2));
    }
};

// Global -> registers for chunk i of this thread of one operand's ROWS x SK.  Out-of-range elements come back as zeros: the
// descriptor covers exactly the rows of this tile that exist (K-contiguous) or the k-rows that exist
// (K-strided), and elements past the end of a K-contiguous row get an offset beyond it.  (Rows past the
// end of a K-strided operand read the neighbouring k-row: values for outputs never stored.)
template <bool KC, int ROWS, int SK, bool VEC, int THREADS = F_THREADS>
__device__ __forceinline__ uintx4 f32_load(const float* p, int64_t ld, int r0, int k0, int rows, int k_end, int tid, int i) {
    typedef F32Tile<KC, ROWS, SK, THREADS> T;
    const float* base = KC ? p + (int64_t)r0 * ld + k0 : p + (int64_t)k0 * ld + r0;
    const int left = KC ? rows - r0 : k_end - k0;   // stored rows that exist from here on
    const int have = left < 0 ? 0 : (left < (KC ? ROWS : SK) ? left : (KC ? ROWS : SK));
    // bytes from `base` to the end of the last existing stored row
    const int64_t in_row = KC ? (int64_t)k_end - k0 : (int64_t)rows - r0;
    const int64_t bytes = have > 0 && in_row > 0 ? (((int64_t)have - 1) * ld + in_row) * 4 : 0;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, (int)bytes, 0x00020000);
    const int q = tid + THREADS * i;
    const int row = q / T::CPR, c = (q % T::CPR) * 4;
    const unsigned off = ((unsigned)row * (unsigned)ld + (unsigned)c) * 4u;
    uintx4 r;
    if (VEC) {
        r = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)(KC && k0 + c >= k_end ? F_OOB : off), 0, 0);
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            r[e] = __builtin_amdgcn_raw_buffer_load_b32(rs, (int)(KC && k0 + c + e >= k_end ? F_OOB : off + 4u * e), 0, 0);
    }
    return r;
}

// x = p0 + p1 + p2 with bf16 p (round to nearest: |x - p0| <= 2^-8 |x|, |x - p0 - p1| <= 2^-17 |x|, and the third holds
// what is left exactly).  Two values at a time, packed.
__device__ __forceinline__ void split2(float x0, float x1, unsigned& p0, unsigned& p1, unsigned& p2) {
    p0 = pack_bf16(x0, x1);
    x0 -= __builtin_bit_cast(float, p0 << 16);
    x1 -= __builtin_bit_cast(float, p0 & 0xFFFF0000u);
    p1 = pack_bf16(x0, x1);
    x0 -= __builtin_bit_cast(float, p1 << 16);
    x1 -= __builtin_bit_cast(float, p1 & 0xFFFF0000u);
    p2 = pack_bf16(x0, x1);
}

// Byte offset of chunk i of this thread in a plane
template <bool KC, int ROWS, int SK>
__device__ __forceinline__ int f32_chunk_at(int tid, int i) {
    typedef F32Tile<KC, ROWS, SK> T;
    const int q = tid + F_THREADS * i;
    const int row = q / T::CPR, c = q % T::CPR;
    return KC ? row * T::RB + T::chunk_at(row, c >> 1) * 16 + (c & 1) * 8
              : row * T::RB + T::seg_at(row, c >> 2) * 32 + (c & 3) * 8;
}

// This lane's MFMA operand from a plane: tile t of the wavefront's ROWS / 2 rows, sub-step kk of 16 k.
template <bool KC, int ROWS, int SK>
__device__ __forceinline__ bf16x8 f32_frag(const char* plane, int wt, int t, int kk, int lane) {
    typedef F32Tile<KC, ROWS, SK> T;
    if (KC) {
        const int l32 = lane & 31, hf = lane >> 5;
        return *reinterpret_cast<const bf16x8*>(plane + (wt * (ROWS / 2) + t * 32 + l32) * T::RB +
                                                T::chunk_at(l32, 2 * kk + hf) * 16);
    }
    // lane s of a group of 16 points at k-row kb + s / 4, rows 4 (s % 4) .. + 3 and receives row s of four k-rows
    const int b = lane >> 4, s = lane & 15;
    const char* p = plane + (16 * kk + 8 * (b >> 1) + (s >> 2)) * T::RB +
                    T::seg_at(s >> 2, wt * (ROWS / 32) + t * 2 + (b & 1)) * 32 + 8 * (s & 3);
    union { short4v h[2]; bf16x8 v; } u;
    u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) short4v*)(p));
    u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) short4v*)(p + 4 * T::RB));
    return u.v;
}

// The work of one workgroup: its tile of TM x TN, the shard it belongs to and the range of K.
struct F32Work {
    const float* A;
    const float* B;
    float* C;
    int64_t lda, ldb, ldc;
    int M, N, m0, n0, k_begin, k_end;
};

template <bool A_KC, bool B_KC, int TM, int TN>
__device__ __forceinline__ F32Work f32_work(const GemmF32Params& g, int bx, int by) {
    constexpr bool CAT_N = A_KC && B_KC, CAT_M = !A_KC && !B_KC, CAT_K = A_KC && !B_KC;
    // Tiles in panels of 8 tile rows, column by column; workgroups are dealt to the 8 XCDs round-robin, so
    // every XCD takes a contiguous run of tiles and shares the operand panels of its run in its L2.
    const int tiles_m = CAT_M ? g.total : (g.M + TM - 1) / TM, tiles_n = CAT_N ? g.total : (g.N + TN - 1) / TN;
    const int total = tiles_m * tiles_n, b = bx;
    const int x = b & 7, per = total >> 3, rem = total & 7;
    const int t = x * per + (x < rem ? x : rem) + (b >> 3);
    const int panel = t / (8 * tiles_n), in_panel = t - panel * 8 * tiles_n;
    const int prows = min(8, tiles_m - panel * 8);
    int tile_m = panel * 8 + in_panel % prows, tile_n = in_panel / prows;

    // the shard of this tile (or slice), its operands and its part of the output
    int shard = CAT_K ? by / g.slices : 0;
    const int slice = CAT_K ? by - shard * g.slices : by;
    if (!CAT_K) {
        const int tc = CAT_N ? tile_n : tile_m;
#pragma unroll
        for (int i = 1; i < GEMM_GROUP_MAX; ++i) shard += tc >= g.first[i] ? 1 : 0;
        if (CAT_N) tile_n -= g.first[shard];
        else tile_m -= g.first[shard];
    }
    const GemmF32Shard& s = g.sh[shard];
    F32Work w;
    w.A = CAT_N ? g.A : s.A;
    w.B = CAT_M ? g.B : s.B;
    w.lda = CAT_N ? g.lda : s.ld;
    w.ldb = g.ldb;
    w.ldc = CAT_N ? s.ld : g.ldc;
    w.M = CAT_M ? s.rows : g.M;
    w.N = CAT_N ? s.rows : g.N;
    w.m0 = tile_m * TM;
    w.n0 = tile_n * TN;
    // slice of the K range; with one slice this is all of K and C is the real output (a short shard's last slices are empty)
    const int K = CAT_K ? s.rows : g.K;
    w.k_begin = min(K, slice * g.k_per_slice);
    w.k_end = min(K, w.k_begin + g.k_per_slice);
    w.C = (CAT_K ? g.C : s.C) + (int64_t)by * g.slice_stride;
    return w;
}

// Two stages of three planes of both operands.
template <int MT, int NT, int SK>
constexpr int f32_lds_bytes() { return 2 * 3 * 2 * SK * 64 * (MT + NT); }

// Stores the elements `which` (bit r: register r) of the 32 x 32 block at (row0, col0): register r of lane l holds
// C[8 (r/4) + 4 (l/32) + r%4][l%32], 128 contiguous bytes per row and store.
__device__ __forceinline__ void f32_store(floatx16 v, unsigned which, const F32Work& w, int row0, int col0, bool accumulate, int lane) {
    const int l32 = lane & 31, hf = lane >> 5;
    const int col = col0 + l32, row = row0 + 4 * hf;
    if (col >= w.N) return;
    float* c = w.C + (int64_t)row * w.ldc + col;
    if (accumulate) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int dr = 8 * (r >> 2) + (r & 3);
            if (row + dr < w.M && (which >> r & 1)) v[r] += c[(int64_t)dr * w.ldc];
        }
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int dr = 8 * (r >> 2) + (r & 3);
        if (row + dr < w.M && (which >> r & 1)) c[(int64_t)dr * w.ldc] = v[r];
    }
}

// Elements `again` (bit r: register r of block i, j) of the wavefront's blocks with the fp32 instruction from the operands as they
// are: global -> registers -> this wavefront's part of the LDS (one stage; K-contiguous rows SK + 4 floats apart, K-strided ones
// an odd multiple of 32, so that the two k of a read fall into different banks) -> MFMA, every stage's loads on their way while the one before it is multiplied.  No barrier: the
// wavefronts whose elements are all finite are done.  Bound by that instruction.  Step of N=1000 h=1024 V=32000 p=8 (finite: 1.05 ms)
// with a NaN in one token / in all / an infinity in W, ms: 4.51 / 8.42 / 5.13 with every block's operands read from global
// memory, 4 bytes a lane -> 2.47 / 2.42 / 2.16 (before the split into parts 1.70 in every case).
template <bool A_KC, bool B_KC, int MT, int NT, int SK, bool VEC>
__device__ __forceinline__ void f32_again(const F32Work& w, const unsigned (&again)[MT][NT], bool accumulate, char* lds, int wave, int lane) {
    constexpr int RA = 32 * MT, RB = 32 * NT;
    typedef F32Tile<A_KC, RA, SK, 64> TA;
    typedef F32Tile<B_KC, RB, SK, 64> TB;
    // floats from stored row to stored row
    constexpr int LA = A_KC ? SK + 4 : RA + (RA % 64 ? 0 : 32), LB = B_KC ? SK + 4 : RB + (RB % 64 ? 0 : 32);
    constexpr int A_FLOATS = (A_KC ? RA : SK) * LA, B_FLOATS = (B_KC ? RB : SK) * LB;
    static_assert(4 * (A_FLOATS + B_FLOATS) * 4 <= f32_lds_bytes<MT, NT, SK>(), "one stage in fp32 for each wavefront");
    asm volatile("" : "+v"(lane));      // addresses are formed here, not held through the products of parts
    float* const la = reinterpret_cast<float*>(lds) + wave * (A_FLOATS + B_FLOATS);
    float* const lb = la + A_FLOATS;
    const int l32 = lane & 31, hf = lane >> 5;
    const int m0 = w.m0 + (wave >> 1) * RA, n0 = w.n0 + (wave & 1) * RB;
    auto in_order = []() {      // a wavefront's LDS accesses are executed in order
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    floatx16 acc[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    uintx4 raw[TA::CHUNKS + TB::CHUNKS];
    auto load = [&](int k0) {
#pragma unroll
        for (int c = 0; c < TA::CHUNKS; ++c) raw[c] = f32_load<A_KC, RA, SK, VEC, 64>(w.A, w.lda, m0, k0, w.M, w.k_end, lane, c);
#pragma unroll
        for (int c = 0; c < TB::CHUNKS; ++c)
            raw[TA::CHUNKS + c] = f32_load<B_KC, RB, SK, VEC, 64>(w.B, w.ldb, n0, k0, w.N, w.k_end, lane, c);
    };
    load(w.k_begin);
    for (int k0 = w.k_begin; k0 < w.k_end; k0 += SK) {
        in_order();
#pragma unroll
        for (int c = 0; c < TA::CHUNKS; ++c) {
            const int q = lane + 64 * c;
            *reinterpret_cast<uintx4*>(la + (q / TA::CPR) * LA + (q % TA::CPR) * 4) = raw[c];
        }
#pragma unroll
        for (int c = 0; c < TB::CHUNKS; ++c) {
            const int q = lane + 64 * c;
            *reinterpret_cast<uintx4*>(lb + (q / TB::CPR) * LB + (q % TB::CPR) * 4) = raw[TA::CHUNKS + c];
        }
        load(k0 + SK);
        in_order();
#pragma unroll 2
        for (int k = 0; k < SK; k += 2) {      // elements past the end of K are zeros in both operands
            float a[MT], b[NT];
#pragma unroll
            for (int i = 0; i < MT; ++i) a[i] = A_KC ? la[(i * 32 + l32) * LA + k + hf] : la[(k + hf) * LA + i * 32 + l32];
#pragma unroll
            for (int j = 0; j < NT; ++j) b[j] = B_KC ? lb[(j * 32 + l32) * LB + k + hf] : lb[(k + hf) * LB + j * 32 + l32];
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int j = 0; j < NT; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], b[j], acc[i][j], 0, 0, 0);
        }
    }
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) f32_store(acc[i][j], again[i][j], w, m0 + i * 32, n0 + j * 32, accumulate, lane);
}

// Workgroup (bx, by) of a product: MT x NT MFMA tiles of 32 x 32 per wavefront, SK of K per LDS stage, PD stages of global loads
// in flight in registers.
template <bool A_KC, bool B_KC, int MT, int NT, int SK, int PD, bool VEC>
__device__ __forceinline__ void gemm_f32_tile(const GemmF32Params& g, char* lds, int bx, int by) {
    constexpr int TM = 64 * MT, TN = 64 * NT;
    typedef F32Tile<A_KC, TM, SK> TA;
    typedef F32Tile<B_KC, TN, SK> TB;
    constexpr int STAGE = 3 * (TA::PLANE + TB::PLANE);
    static_assert(2 * STAGE == f32_lds_bytes<MT, NT, SK>(), "two stages");
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const F32Work w = f32_work<A_KC, B_KC, TM, TN>(g, bx, by);
    constexpr int KS = SK / 16;
    static_assert(MT * NT == 8 || MT * NT == 4 ? KS == 1 : MT * NT == 1 && KS == 2, "tile");
    floatx16 acc[KS][MT][NT];
#pragma unroll
    for (int kk = 0; kk < KS; ++kk)
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[kk][i][j][r] = 0.f;

    // Stage q waits in registers from its request until it is split into LDS buffer q & 1 while stage q - 1 is multiplied;
    // stages past the end of K are zeros that nothing multiplies.
    constexpr int CA = TA::CHUNKS, CB = TB::CHUNKS;
    uintx4 raw[PD][CA + CB];
    auto load = [&](int u, int c, int q) {
        const int k0 = w.k_begin + q * SK;
        raw[u][c] = c < CA ? f32_load<A_KC, TM, SK, VEC>(w.A, w.lda, w.m0, k0, w.M, w.k_end, tid, c)
                           : f32_load<B_KC, TN, SK, VEC>(w.B, w.ldb, w.n0, k0, w.N, w.k_end, tid, c - CA);
    };
    // Splits two of the values of chunk c (first: the lower two); with the upper two the chunk's parts go to LDS.
    uint2 parts[3];
    auto split = [&](int u, int c, bool first, char* stage) {
        float x0 = __builtin_bit_cast(float, (unsigned)raw[u][c][first ? 0 : 2]);
        float x1 = __builtin_bit_cast(float, (unsigned)raw[u][c][first ? 1 : 3]);
        x0 *= IN_SCALE;
        x1 *= IN_SCALE;
        if (first) {
            split2(x0, x1, parts[0].x, parts[1].x, parts[2].x);
            return;
        }
        split2(x0, x1, parts[0].y, parts[1].y, parts[2].y);
        char* at = c < CA ? stage + f32_chunk_at<A_KC, TM, SK>(tid, c)
                          : stage + 3 * TA::PLANE + f32_chunk_at<B_KC, TN, SK>(tid, c - CA);
#pragma unroll
        for (int l = 0; l < 3; ++l) *reinterpret_cast<uint2*>(at + l * (c < CA ? TA::PLANE : TB::PLANE)) = parts[l];
    };
    const int stages = (w.k_end - w.k_begin + SK - 1) / SK;
#pragma unroll
    for (int u = 0; u < PD; ++u)
#pragma unroll
        for (int c = 0; c < CA + CB; ++c) load(u, c, u);
#pragma unroll
    for (int c = 0; c < CA + CB; ++c) {
        split(0, c, true, lds);
        split(0, c, false, lds);
        load(0, c, PD);
    }
    __syncthreads();
    for (int q0 = 0; q0 < stages; q0 += PD) {
#pragma unroll
        for (int u = 0; u < PD; ++u) {
            const int q = q0 + u;
            if (q >= stages) break;
            const char* sa = lds + (q & 1) * STAGE;
            const char* sb = sa + 3 * TA::PLANE;
            char* next = lds + ((q + 1) & 1) * STAGE;      // last read before the previous barrier
            // MFMAs that follow one another are independent (one waits for the sum it adds to): four tiles, of the 2 x 4 or
            // 4 x 2 ones those of one column / row at a time, or where a wavefront has a single tile two sums over k.
            constexpr int PASSES = MT * NT == 8 ? 2 : 1;
            bf16x8 a[KS][3][MT], b[KS][3][NT];
#pragma unroll
            for (int f = 0; f < 3; ++f) {      // in the order of their first use
                const int la = (f + 2) % 3, lb = (3 - f) % 3;
#pragma unroll
                for (int kk = 0; kk < KS; ++kk) {
#pragma unroll
                    for (int i = 0; i < (NT > MT ? MT / PASSES : MT); ++i)
                        a[kk][la][i] = f32_frag<A_KC, TM, SK>(sa + la * TA::PLANE, wm, i, kk, lane);
#pragma unroll
                    for (int j = 0; j < (NT > MT ? NT : NT / PASSES); ++j)
                        b[kk][lb][j] = f32_frag<B_KC, TN, SK>(sb + lb * TB::PLANE, wn, j, kk, lane);
                }
            }
#pragma unroll
            for (int o = 0; o < PASSES; ++o) {
                // the six largest products of parts, the small ones first; after each of them a share of the next
                // stage's split, whose vector instructions issue while the matrix cores work
                constexpr int LA[6] = {2, 0, 1, 1, 0, 0}, LB[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
                for (int e = 0; e < 6; ++e) {
                    if (e == 3 && o + 1 < PASSES) {
#pragma unroll
                        for (int l = 0; l < 3; ++l) {
                            if (NT > MT) a[0][l][1] = f32_frag<A_KC, TM, SK>(sa + l * TA::PLANE, wm, 1, 0, lane);
                            else b[0][l][1] = f32_frag<B_KC, TN, SK>(sb + l * TB::PLANE, wn, 1, 0, lane);
                        }
                    }
                    constexpr int INNER = PASSES == 2 ? 4 : KS * MT * NT;
#pragma unroll
                    for (int xx = 0; xx < INNER; ++xx) {
                        const int y = (e & 1) ? INNER - 1 - xx : xx;
                        const int kk = KS == 2 ? y : 0;
                        const int i = PASSES == 2 ? (NT > MT ? o : y) : KS == 2 ? 0 : y >> 1;
                        const int j = PASSES == 2 ? (NT > MT ? y : o) : KS == 2 ? 0 : (y ^ (y >> 1)) & 1;
                        acc[kk][i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[kk][LA[e]][i], b[kk][LB[e]][j], acc[kk][i][j], 0, 0, 0);
                    }
                    constexpr int PAIRS = 2 * (CA + CB), PER = (PAIRS + 6 * PASSES - 1) / (6 * PASSES);
#pragma unroll
                    for (int z = 0; z < PER; ++z) {
                        const int pair = (o * 6 + e) * PER + z;
                        if (pair < PAIRS) {
                            split((u + 1) % PD, pair >> 1, (pair & 1) == 0, next);
                            if (pair & 1) load((u + 1) % PD, pair >> 1, q + 1 + PD);
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            __syncthreads();
        }
    }

    // A non-finite operand (or one that rounds to a bf16 infinity, or an overflow) makes the parts of the split cancel to NaN.
    // Elements that are not finite are computed again from the operands as they are, in fp32; and so are sums of fewer than five
    // products, in which what the split leaves out shows (a single product would be off by its last bit).
    const bool few = w.k_end - w.k_begin < F_FEW;
    const int lid = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));      // the lane, not held through the loop
    bool any = few;
    unsigned again[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            floatx16 v = acc[0][i][j];
            if constexpr (KS == 2) {
#pragma unroll
                for (int r = 0; r < 16; ++r) v[r] += acc[1][i][j][r];
            }
            float nf = 0.f;
#pragma unroll
            for (int r = 0; r < 16; ++r) nf = fmaf(v[r], 0.f, nf);
#pragma unroll
            for (int r = 0; r < 16; ++r) v[r] *= 1.f / (IN_SCALE * IN_SCALE);
            again[i][j] = few ? 0xFFFFu : 0u;
            if (__builtin_amdgcn_ballot_w64(!(nf == 0.f)) != 0) {
                any = true;
#pragma unroll
                for (int r = 0; r < 16; ++r) again[i][j] |= fabsf(v[r]) < INFINITY ? 0u : 1u << r;
            }
            f32_store(v, ~again[i][j], w, w.m0 + (wm * MT + i) * 32, w.n0 + (wn * NT + j) * 32, g.accumulate != 0, lid);
        }
    // (every wavefront is done with the stages in LDS)
    if (any) f32_again<A_KC, B_KC, MT, NT, SK, VEC>(w, again, g.accumulate != 0, lds, wave, lid);
}

// WPC workgroups per compute unit.
template <bool A_KC, bool B_KC, int MT, int NT, int SK, int PD, int WPC, bool VEC>
__global__ __launch_bounds__(F_THREADS, WPC) void gemm_f32_kernel(GemmF32Params g) {
    __shared__ __attribute__((aligned(16))) char lds[f32_lds_bytes<MT, NT, SK>()];
    gemm_f32_tile<A_KC, B_KC, MT, NT, SK, PD, VEC>(g, lds, blockIdx.x, blockIdx.y);
}

// dH and dW in one launch: the first `nh` workgroups are dH's, hx in a row of its grid.  Neither needs the other, and where one
// alone does not fill the chip, its workgroups wait (for loads, LDS and barriers) more than they multiply: N=128 h=256 V=8192
// p=2: 12.8 + 11.3 us -> 15.3 to 17.6, the step 48.3 -> 40.7.
template <int MT, int NT, int SK, int PD, int WPC>
__global__ __launch_bounds__(F_THREADS, WPC) void gemm_f32_dh_dw_kernel(GemmF32Params h, GemmF32Params w, int nh, int hx) {
    __shared__ __attribute__((aligned(16))) char lds[f32_lds_bytes<MT, NT, SK>()];
    const int b = blockIdx.x;
    if (b < nh) gemm_f32_tile<true, false, MT, NT, SK, PD, true>(h, lds, b % hx, b / hx);
    else gemm_f32_tile<false, false, MT, NT, SK, PD, true>(w, lds, b - nh, 0);
}

// Estimated time of `wg` workgroups over k steps of K each.  A workgroup alone on a compute unit takes `alone` us per 16 k
// (a chain of load, split, LDS and products); several share the unit at `each` us (K = 1024: 256 tiles of 64 x 64 28 us, 1024 of
// them 88; 64 tiles of 128 x 128 61; 512 of the largest 170).  A larger tile's start and end take longer (K = 64: 7.5 us, 11).
static double product_us(int tile, int64_t wg, int64_t k) {
    const double alone = tile == 64 ? 0.42 : tile == 128 ? 0.95 : 1.6, each = tile == 64 ? 0.34 : tile == 128 ? 0.72 : 1.28;
    const double n = (double)ceil_div(wg, 256) * each;
    return (double)ceil_div(k, 16) * (n > alone ? n : alone) + (tile == 64 ? 0.0 : tile == 128 ? 3.0 : 6.0);
}

// K slices for an output of this many 64 x 64 tiles: enough workgroups to cover the chip, slices of at least min_k.
static int slices_for(int64_t tiles, int64_t K, int64_t min_k) {
    int64_t S = 256 / tiles;
    if (S > 32) S = 32;
    if (S > K / min_k) S = K / min_k;
    return S < 2 ? 1 : (int)S;
}
static int splitk_slices(int64_t M, int64_t N, int64_t K) { return slices_for(ceil_div(M, 64) * ceil_div(N, 64), K, 64); }
// Logits and dW of a group.  A K step of 32 takes 0.55-0.85 us where a workgroup has a compute unit to itself; the sum of the
// slices is another launch, 3 us of host time in passes that the host bounds.  So slices of at least 256, from K = 1024 on.
// 32 tiles, product and forward pass, us, in one chain -> in slices: K = 512: 19.3 -> 15.4 and 28.0 -> 31.2; 640: 22.4 ->
// 17.2 and 27.8 -> 30.6; 800: 26.5 -> 16.5 and 30.6 -> 31.0; 1024: 32.4 -> 15.9 and 36.9 -> 30.5; 2048: 58 -> 17 and 63 -> 30.
int gemm_f32_group_slices(int64_t tiles, int64_t K) { return K < 1024 ? 1 : slices_for(tiles, K, 256); }
// Slices are multiples of 32 k long, the step of the small tiles.
static int slice_length(int64_t K, int S) { return S > 1 ? (int)(ceil_div(ceil_div(K, S), 32) * 32) : (int)K; }

// Fills first and total for this tile and returns the grid.
template <bool A_KC, bool B_KC>
static dim3 f32_grid(GemmF32Params& g, int tile) {
    constexpr bool DW = !A_KC;
    const int tile_m = tile == 256 && !DW ? 128 : tile, tile_n = tile == 256 && DW ? 128 : tile;
    int64_t tm = ceil_div(g.M, tile_m), tn = ceil_div(g.N, tile_n), cat = 0;
    for (int r = 0; r < GEMM_GROUP_MAX; ++r) {
        g.first[r] = r < g.n ? (int)cat : INT_MAX;
        if (r < g.n) cat += ceil_div(g.sh[r].rows, A_KC ? tile_n : tile_m);
    }
    g.total = (int)cat;
    int z = g.slices;
    if (A_KC && B_KC) tn = cat;
    else if (!A_KC) tm = cat;
    else z *= g.n;
    return dim3((unsigned)(tm * tn), (unsigned)z);
}

template <bool A_KC, bool B_KC>
static void launch_f32_t(GemmF32Params& g, int tile, hipStream_t st) {
    constexpr bool DW = !A_KC;
    const dim3 grid = f32_grid<A_KC, B_KC>(g, tile);
    const bool vec = g.a_vec && g.b_vec;
#define VP_LAUNCH(...) hipLaunchKernelGGL((gemm_f32_kernel<A_KC, B_KC, __VA_ARGS__>), grid, dim3(F_THREADS), 0, st, g)
    if (tile == 256) VP_LAUNCH((DW ? 4 : 2), (DW ? 2 : 4), 16, 1, 2, true);
    else if (tile == 128 && vec) VP_LAUNCH(2, 2, 16, 2, 3, true);
    else if (tile == 128) VP_LAUNCH(2, 2, 16, 2, 2, false);
    else if (vec) VP_LAUNCH(1, 1, 32, 1, 3, true);
    else VP_LAUNCH(1, 1, 32, 1, 3, false);
#undef VP_LAUNCH
}

// Tile of the least estimated time.
static int tile_for(const GemmF32Params& g, bool a_kc, bool b_kc) {
    const bool cat_n = a_kc && b_kc, cat_k = a_kc && !b_kc;
    if (!cat_k && g.slices > 1) return 64;      // (slices of logits and dW are counted in 64 x 64 tiles: gemm_f32_group_slices)
    int tile = 64;
    double best = 0;
    for (int t : {64, 128, 256}) {
        if (t == 256 && !(g.a_vec && g.b_vec)) continue;
        const int tm = t == 256 && a_kc ? 128 : t, tn = t == 256 && !a_kc ? 128 : t;
        int64_t wg = 0;
        for (int r = 0; r < g.n; ++r)
            wg += cat_n ? ceil_div(g.M, tm) * ceil_div(g.sh[r].rows, tn)
                        : ceil_div(cat_k ? g.M : g.sh[r].rows, tm) * ceil_div(g.N, tn);
        const double us = product_us(t, wg * g.slices, g.k_per_slice);
        if (t == 64 || us < best) {
            best = us;
            tile = t;
        }
    }
    return tile;
}

// A product ready to be launched; C is [M, N] with row stride ldc where the shards share the output (dH).  With more than one K
// slice (dH: of all shards together) the partial outputs go through scratch, every slice laid out like the output, or like
// the outputs of the shards one behind the other.
struct F32Launch {
    GemmF32Params g;
    bool a_kc, b_kc, accumulate;
    int tile, parts;
    float* scratch;
    SumList l;
};

static F32Launch prepare_f32(const GemmF32Params& g0, bool a_kc, bool b_kc, float* C, int64_t ldc, bool accumulate, float* scratch) {
    F32Launch f{g0, a_kc, b_kc, accumulate, tile_for(g0, a_kc, b_kc), 0, scratch, {}};
    GemmF32Params& g = f.g;
    const bool cat_n = a_kc && b_kc, cat_k = a_kc && !b_kc;
    f.parts = g.slices * (cat_k ? g.n : 1);
    g.C = C;
    if (!cat_n) g.ldc = ldc;
    g.accumulate = accumulate ? 1 : 0;
    if (f.parts > 1) {
        SumList& l = f.l;
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
    return f;
}

static hipError_t launch_f32(F32Launch& f, hipStream_t st) {
    if (f.a_kc && f.b_kc) launch_f32_t<true, true>(f.g, f.tile, st);
    else if (f.a_kc) launch_f32_t<true, false>(f.g, f.tile, st);
    else if (!f.b_kc) launch_f32_t<false, false>(f.g, f.tile, st);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

static hipError_t sum_f32(const F32Launch& f, hipStream_t st) {
    return f.parts == 1 ? hipSuccess : launch_sum_slices(f.scratch, f.parts, f.g.slice_stride, f.l, f.accumulate, st);
}

static hipError_t launch_and_sum_f32(F32Launch f, hipStream_t st) {
    const hipError_t e = launch_f32(f, st);
    return e == hipSuccess ? sum_f32(f, st) : e;
}

// K slices of one shard's product: the launch cuts K into at most as many as the scratch is sized for.
static int single_slices(F32Product kind, int64_t M, int64_t N, int64_t K) {
    return kind == F32Product::DH ? gemm_f32_dh_slices(M, N, K, 1) : splitk_slices(M, N, K);
}

size_t gemm_f32_scratch_floats(F32Product kind, int64_t M, int64_t N, int64_t K) {
    const int S = single_slices(kind, M, N, K);
    return S > 1 ? (size_t)S * (size_t)M * (size_t)N : 0;
}

// One shard's product.  Its layouts and K slices follow from which product it is, never from the strides: a matrix of one column,
// or of one row, is K-contiguous and K-strided at once.
static GemmF32Params single_params(F32Product kind, const float* A, int64_t lda, const float* B, int64_t ldb, float* C, int M, int N,
                                   int K) {
    const bool a_kc = kind != F32Product::DW, b_kc = kind == F32Product::Logits;
    GemmF32Params g{};
    g.A = A; g.B = B;
    g.lda = lda; g.ldb = ldb;
    g.M = M; g.N = N; g.K = K;
    g.k_per_slice = slice_length(K, single_slices(kind, M, N, K));
    g.slices = (int)ceil_div(K, g.k_per_slice);
    g.a_vec = lda % 4 == 0 && ((uintptr_t)A & 15u) == 0 && (!a_kc || K % 4 == 0);
    g.b_vec = ldb % 4 == 0 && ((uintptr_t)B & 15u) == 0 && (!b_kc || K % 4 == 0);
    g.n = 1;
    GemmF32Shard& s = g.sh[0];
    s.A = A; s.B = B; s.C = C;
    s.rows = b_kc ? N : a_kc ? K : M;
    s.ld = b_kc ? N : (int)lda;
    return g;
}

hipError_t launch_gemm_f32(F32Product kind, const float* A, int64_t lda, const float* B, int64_t ldb, float* C, int M, int N, int K,
                           bool accumulate, float* scratch, hipStream_t st) {
    if (M <= 0 || N <= 0 || K <= 0) return hipErrorInvalidValue;
    ProfScope prof(K_GEMM_F32, st);
    const GemmF32Params g = single_params(kind, A, lda, B, ldb, C, M, N, K);
    if (g.slices > 1 && !scratch) return hipErrorInvalidValue;
    return launch_and_sum_f32(prepare_f32(g, kind != F32Product::DW, kind == F32Product::Logits, C, N, accumulate, scratch), st);
}

// What prepare_f32 lays out for this product: every float that its launches write outside the output.
size_t gemm_f32_written_floats(F32Product kind, int64_t M, int64_t N, int64_t K) {
    const F32Launch f = prepare_f32(single_params(kind, nullptr, 0, nullptr, 0, nullptr, (int)M, (int)N, (int)K),
                                    kind != F32Product::DW, kind == F32Product::Logits, nullptr, N, false, nullptr);
    return f.parts > 1 ? (size_t)f.parts * (size_t)f.g.slice_stride : 0;
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
    return launch_and_sum_f32(prepare_f32(g, true, true, nullptr, 0, false, scratch), st);
}

static GemmF32Params dh_params(int64_t N, int64_t h, const GemmF32Shard* sh, int n, int slices) {
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
    g.k_per_slice = (int)(ceil_div(ceil_div(rows, slices), 32) * 32);
    g.n = n;
    return g;
}

hipError_t launch_gemm_f32_dh(int64_t N, int64_t h, const GemmF32Shard* sh, int n, int slices, float* dH, bool accumulate,
                              float* scratch, hipStream_t st) {
    ProfScope prof(K_GEMM_F32, st);
    return launch_and_sum_f32(prepare_f32(dh_params(N, h, sh, n, slices), true, false, dH, h, accumulate, scratch), st);
}

static GemmF32Params dw_params(const float* H, int64_t N, int64_t h, const GemmF32Shard* sh, int n, int slices) {
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
    return g;
}

hipError_t launch_gemm_f32_dw(const float* H, int64_t N, int64_t h, const GemmF32Shard* sh, int n, int slices, float* scratch,
                              hipStream_t st) {
    ProfScope prof(K_GEMM_F32, st);
    return launch_and_sum_f32(prepare_f32(dw_params(H, N, h, sh, n, slices), false, false, nullptr, h, false, scratch), st);
}

// Both products of pass T.  One launch where both take the same tiles and together have at most four workgroups per compute
// unit (three fit): 840 of them (N=300 h=1000 V=5001 p=3) 117 -> 115 us a step, 1024 (N=400 h=512 V=16000 p=4) 219 -> 211, 1050 (N=781
// h=704 V=6252 p=16) 227 -> 229.  dW in slices needs the scratch that dH's slices are in, so it comes after their sum.
hipError_t launch_gemm_f32_dh_dw(const float* H, int64_t N, int64_t h, const GemmF32Shard* sh, int n, int dh_slices, int dw_slices,
                                 float* dH, bool accumulate, float* scratch, hipStream_t st) {
    F32Launch a = prepare_f32(dh_params(N, h, sh, n, dh_slices), true, false, dH, h, accumulate, scratch);
    F32Launch b = prepare_f32(dw_params(H, N, h, sh, n, dw_slices), false, false, nullptr, h, false, scratch);
    if (a.tile == b.tile && a.tile <= 128 && b.parts == 1 && a.g.b_vec && b.g.b_vec) {
        const dim3 ga = f32_grid<true, false>(a.g, a.tile), gb = f32_grid<false, false>(b.g, b.tile);
        const int na = (int)(ga.x * ga.y), nb = (int)gb.x;
        if (na + nb <= 1024) {
            ProfScope prof(K_GEMM_F32, st);
            if (a.tile == 64)
                hipLaunchKernelGGL((gemm_f32_dh_dw_kernel<1, 1, 32, 1, 3>), dim3(na + nb), dim3(F_THREADS), 0, st, a.g, b.g, na, (int)ga.x);
            else
                hipLaunchKernelGGL((gemm_f32_dh_dw_kernel<2, 2, 16, 2, 3>), dim3(na + nb), dim3(F_THREADS), 0, st, a.g, b.g, na, (int)ga.x);
            const hipError_t e = hipGetLastError();
            return e == hipSuccess ? sum_f32(a, st) : e;
        }
    }
    const hipError_t e = launch_gemm_f32_dh(N, h, sh, n, dh_slices, dH, accumulate, scratch, st);
    return e == hipSuccess ? launch_gemm_f32_dw(H, N, h, sh, n, dw_slices, scratch, st) : e;
}

hipError_t launch_gemm_f32_each(int64_t N, int64_t h, const GemmF32Shard* sh, int n, int slices, float* out, float* scratch,
                                hipStream_t st) {
    ProfScope prof(K_GEMM_F32, st);
    GemmF32Params g = dh_params(N, h, sh, n, slices);
    g.C = slices > 1 ? scratch : out;
    g.ldc = h;
    g.slice_stride = N * h;
    launch_f32_t<true, false>(g, tile_for(g, true, false), st);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || slices == 1) return e;
    SumList l{};
    l.n = n;
    for (int r = 0; r < n; ++r) {
        l.first[r] = (int64_t)r * slices * N * h;
        l.count[r] = N * h;
        l.C[r] = out + (int64_t)r * N * h;
    }
    return launch_sum_slices(scratch, slices, N * h, l, false, st);
}

// K slices per shard of the dH product of n shards with at most `rows` rows each: the least estimated time; the partial
// outputs are written and read once (4 TB/s), by another launch (one: they are summed even with one slice per shard).
static int dh_slices(int64_t N, int64_t h, int64_t rows, int n, bool one) {
    int best = 1;
    double best_us = 0;
    for (int64_t S = 1; S <= 64 && (S == 1 || (rows >= 64 * S && n * S * N * h <= (int64_t)1 << 26)); ++S) {
        const double sum = (one ? n * S : S) > 1 ? (double)(n * S) * (double)(N * h) * 8.0 / 4e6 + 4.0 : 0.0;
        for (int t : {64, 128, 256}) {
            const double us = sum + product_us(t, ceil_div(N, t == 256 ? 128 : t) * ceil_div(h, t) * n * S, ceil_div(rows, S));
            if ((S == 1 && t == 64) || us < best_us) {
                best = (int)S;
                best_us = us;
            }
        }
    }
    return best;
}
int gemm_f32_dh_slices(int64_t N, int64_t h, int64_t rows, int n) { return dh_slices(N, h, rows, n, true); }
int gemm_f32_each_slices(int64_t N, int64_t h, int64_t rows, int n) { return dh_slices(N, h, rows, n, false); }

}  // namespace vp
