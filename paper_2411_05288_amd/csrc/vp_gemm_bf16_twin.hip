// dW with two workgroups per compute unit, for few tokens.
#include "vp_gemm_bf16_fast.h"

namespace vp {

// dW = D^T H for few tokens (few k tiles per output tile): two workgroups per compute unit, so that one multiplies while
// the other stores.  With one workgroup of 256 x 256 per compute unit the 256 KB of a finished tile leave in 8-10 us (all
// compute units together: the rate of the memory) during which its matrix cores idle, and the memory idles while it
// multiplies; at K = 512 both take about as long, and the launch took their sum.
//
// Tile 256 x 128 (per wavefront 128 x 64: 128 accumulators, so that two wavefronts fit a SIMD), three LDS slots of 32 k
// (A half as above, 16 KB, then B: [32 k][128 rows], 256-byte k-rows, the same 32-byte segment swizzle, 8 KB): 72 KB per
// workgroup.  Slot i is multiplied while i + 1 and i + 2 are on their way; one barrier per slot.  Twice the LDS reads of B
// per flop of the tile above: where the stores are a small part, the large tile is the better one (see launch_dw).
constexpr int TWIN_BN = 128;
constexpr int TWIN_SLOT_BYTES = HALF_OP_BYTES + HALF_OP_BYTES / 2;
static __shared__ __attribute__((aligned(1024))) char g_twin0[TWIN_SLOT_BYTES];
static __shared__ __attribute__((aligned(1024))) char g_twin1[TWIN_SLOT_BYTES];
static __shared__ __attribute__((aligned(1024))) char g_twin2[TWIN_SLOT_BYTES];
static_assert(2 * StageF32<64>::BYTES <= TWIN_SLOT_BYTES, "epilogue staging of two wavefronts exceeds a slot");

template <int S>
__device__ __forceinline__ char* twin_slot() {
    if constexpr (S == 0) return g_twin0;
    else if constexpr (S == 1) return g_twin1;
    else return g_twin2;
}

// The 6 wave-wide loads of this wavefront's share of slot i: 4 pieces of A, 2 of B (k advance as in issue_operand_loads).
template <int S>
__device__ __forceinline__ void twin_loads(const void* A, unsigned a_bytes, unsigned a_adv, const unsigned (&avoff)[4],
                                           const void* B, unsigned b_bytes, unsigned b_adv, const unsigned (&bvoff)[2], int wave) {
    const unsigned aa = a_adv < a_bytes ? a_adv : a_bytes, ba = b_adv < b_bytes ? b_adv : b_bytes;
    const __amdgpu_buffer_rsrc_t ra =
        __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)A + aa), 0, (int)(a_bytes - aa), 0x00020000);
    const __amdgpu_buffer_rsrc_t rb =
        __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)B + ba), 0, (int)(b_bytes - ba), 0x00020000);
#pragma unroll
    for (int jj = 0; jj < 4; ++jj)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (lds_ptr)(twin_slot<S>() + (wave * 4 + jj) * 1024), 16, (int)avoff[jj], 0, 0, 0);
#pragma unroll
    for (int jj = 0; jj < 2; ++jj)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rb, (lds_ptr)(twin_slot<S>() + HALF_OP_BYTES + (wave * 2 + jj) * 1024), 16,
                                                 (int)bvoff[jj], 0, 0, 0);
}

__device__ __forceinline__ bf16x8 twin_read_b(const char* half, int base, int kk) {
    union { short4v h[2]; bf16x8 v; } u;
    const char* p = half + base + kk * 4096;
    u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) short4v*)(p));
    u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) short4v*)(p + 1024));
    return u.v;
}

__global__ __launch_bounds__(NT, 2) void gemm_bf16_dw_twin_kernel(GemmBf16Group gg) {
    const GemmBf16Params& g = gg.base;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int tiles_m = gg.total, tiles_n = (g.N + TWIN_BN - 1) / TWIN_BN;
    const int total_tiles = tiles_m * tiles_n;

    int abase[4], bbase[2];
    frag_offsets<false>(abase, wm, lane);
    {
        const int b = lane >> 4, s = lane & 15;
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int seg = (wn * 4 + t * 2 + (b & 1)) ^ seg_swizzle(s >> 2);
            bbase[t] = (8 * (b >> 1) + (s >> 2)) * 256 + seg * 32 + 8 * (s & 3);
        }
    }
    for (int v = blockIdx.x; v < total_tiles; v += gridDim.x) {
        int tile_m, tile_n;
        tile_of_block(v, gridDim.x, total_tiles, tiles_m, tiles_n, tile_m, tile_n);
        int shard = shard_of(gg, tile_m);
        tile_m -= gg.first[shard];
        const GemmBf16Shard& s = gg.sh[shard];
        const void *A = s.A, *B = g.B;
        const unsigned a_bytes = (unsigned)g.K * (unsigned)s.ld * 2u, b_bytes = (unsigned)g.K * (unsigned)g.ldb * 2u;
        const unsigned a_step = 64u * (unsigned)s.ld, b_step = 64u * (unsigned)g.ldb;      // 32 k-rows
        unsigned avoff[4], bvoff[2];
        half_voffsets<false>(avoff, tile_m * BM, s.ld, wave, lane);
#pragma unroll
        for (int jj = 0; jj < 2; ++jj) {      // a piece of B is 4 k-rows of 16 chunks of 16 bytes
            const int krow = (wave * 2 + jj) * 4 + (lane >> 4), cpos = lane & 15;
            const int c = ((cpos >> 1) ^ seg_swizzle(krow & 3)) * 2 + (cpos & 1);
            bvoff[jj] = ((unsigned)krow * (unsigned)g.ldb + (unsigned)(tile_n * TWIN_BN + c * 8)) * 2u;
        }
        const int n_slots = (g.K + 31) / 32;

#define VP_TWIN_LOADS(I, S) twin_loads<S>(A, a_bytes, (unsigned)(I) * a_step, avoff, B, b_bytes, (unsigned)(I) * b_step, bvoff, wave)
        VP_TWIN_LOADS(0, 0);
        VP_TWIN_LOADS(1, 1);
        floatx16 acc[4][2];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

        // slot i: it has landed (all but the 6 loads of slot i + 1), every wavefront is done with slot i - 1, whose place the
        // loads of slot i + 2 take (past the end of K: empty descriptors)
#define VP_TWIN_STEP(I, S)                                                                              \
        {                                                                                               \
            __builtin_amdgcn_s_waitcnt(0x0076);       /* vmcnt(6) lgkmcnt(0) */                         \
            asm volatile("" ::: "memory");                                                              \
            __builtin_amdgcn_s_barrier();                                                               \
            asm volatile("" ::: "memory");                                                              \
            VP_TWIN_LOADS((I) + 2, ((S) + 2) % 3);                                                      \
            _Pragma("unroll") for (int kk = 0; kk < 2; ++kk) {                                          \
                bf16x8 af[4], bf[2];                                                                    \
                _Pragma("unroll") for (int t = 0; t < 4; ++t) af[t] = read_operand<false>(twin_slot<S>(), abase, t, kk); \
                _Pragma("unroll") for (int t = 0; t < 2; ++t) bf[t] = twin_read_b(twin_slot<S>() + HALF_OP_BYTES, bbase[t], kk); \
                _Pragma("unroll") for (int j = 0; j < 2; ++j)                                           \
                    _Pragma("unroll") for (int ii = 0; ii < 4; ++ii) {                                  \
                        const int i = (j & 1) ? 3 - ii : ii;                                            \
                        mfma_tile<Epi::StoreF32>(acc[i][j], af[i], bf[j]);                              \
                    }                                                                                   \
            }                                                                                           \
        }
        int i0 = 0;
        for (; i0 + 3 <= n_slots; i0 += 3) {
            VP_TWIN_STEP(i0, 0)
            VP_TWIN_STEP(i0 + 1, 1)
            VP_TWIN_STEP(i0 + 2, 2)
        }
        if (i0 < n_slots) {
            VP_TWIN_STEP(i0, 0)
            if (i0 + 1 < n_slots) VP_TWIN_STEP(i0 + 1, 1)
        }
#undef VP_TWIN_STEP
#undef VP_TWIN_LOADS
        __builtin_amdgcn_s_waitcnt(0x0070);      // vmcnt(0) lgkmcnt(0): no load into a slot is in flight
        __syncthreads();                         // and every wavefront is done with them before the epilogue uses them
        asm volatile("" : "+s"(tile_m), "+s"(tile_n), "+s"(shard));
        GemmBf16Params e = g;
        e.M = gg.sh[shard].rows;
        e.C = (float*)gg.sh[shard].out;
        gemm_epilogue_f32<Epi::StoreF32, 2, 2, true, 4>(acc, e, tile_m, tile_n,
                                                     (wave < 2 ? g_twin0 : g_twin1) + (wave & 1) * StageF32<64>::BYTES);
        __syncthreads();   // the staging blocks are read before the next tile streams in
    }
}

hipError_t launch_gemm_bf16_dw_twin(const GemmBf16Group& g, hipStream_t st) {
    const int tiles = (int)(g.total * ceil_div(g.base.N, TWIN_BN)), room = 2 * compute_unit_count();
    hipLaunchKernelGGL(gemm_bf16_dw_twin_kernel, dim3(tiles > room ? room : tiles), dim3(NT), 0, st, g);
    return hipGetLastError();
}

}  // namespace vp
