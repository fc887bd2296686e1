// Fast path of the bf16 MFMA GEMM (gfx950): operands go from global memory straight into LDS
// (buffer loads with the LDS bit, 16 bytes per lane) through a ring of five half-k-tile slots,
// MFMA operands are prefetched one 16-wide k sub-step ahead, two workgroup barriers per 64-wide
// k tile.  The loads of a k tile are in flight for a whole tile period before anything waits for
// them: with one wavefront per SIMD nothing else hides the load latency (about 0.9 us under load,
// longer than the matrix cores need for a tile at any clock this part sustains).
//
// Preconditions (checked by gemm_bf16_fast_ok on the host; anything else takes the generic
// kernel): rows of both operands 16-byte aligned, operands smaller than 4 GB with slack for
// the offsets of the zero-filled tile overhang.
//
// Out-of-range handling relies on the buffer descriptor: every operand is described by a raw
// buffer of exactly its size, so a lane whose 16 bytes start at or beyond the end of the
// matrix receives zeros.  Rows past the end of a K-contiguous operand and k-rows past the
// end of a K-strided operand are therefore zero.  What is NOT zero is the overhang inside
// the matrix (the k tail of a K-contiguous row runs into the next row, the column tail of a
// K-strided row runs into the next k-row): that data either meets zeros of the other operand
// (k tails: D's rows are padded with zeros to a multiple of 64) or lands in output rows / columns
// that the epilogue never stores.  Where no operand is K-strided and K is no multiple of 64, an
// instantiation of its own (KTAIL) gives the lanes past the end of K in the last k tile an offset
// beyond every buffer, in both operands.
//
// LDS layouts (a slot holds 32 of a k tile's 64 k for both operands, 16 KB each, written by 16
// wave-wide loads of 1 KB per operand; a load writes lane i's 16 bytes at byte 16*i of its 1 KB
// piece, so the swizzles below are applied to the global address each lane fetches):
//   K-contiguous half  [256 rows][32 k]: 64 B rows; 16-byte chunk c of row r sits at chunk
//       position c ^ ((r >> 2) & 3).  One ds_read_b128 per MFMA operand; the 16 consecutive rows a
//       pass of that read serves fall into 16 different bank groups (counter: no bank conflicts).
//   K-strided half [32 k][256 rows]: 512 B k-rows of 16 segments of 32 B (16 rows); segment s of
//       k-row k sits at segment position s ^ f(k & 3), f = {0,5,2,7}.  MFMA operands are read
//       with the transposing LDS load (ds_read_b64_tr_b16): in a group of 16 lanes, lane s
//       points at k-row kb + s/4, rows nb + 4*(s%4)..+3, and lane i receives rows nb + i for
//       the four k-rows kb..kb+3.  f makes the 4 k-rows of a group, and the 8 of two groups,
//       fall into different banks.
#pragma once

#include "vp_gemm_bf16_common.h"

namespace vp {

typedef short short4v __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void* lds_ptr;

constexpr int HALF_OP_BYTES = 16384;          // one operand, 32 of the 64 k of a k tile: 256 x 32 bf16
constexpr int SLOT_BYTES = 2 * HALF_OP_BYTES; // A half then B half
constexpr int N_SLOTS = 5;

// Five LDS slots of half a k tile each (all 160 KB of the compute unit).  K tile T occupies the slots
// (2T) % 5 and (2T + 1) % 5, so that next to the two tiles being multiplied and landing there is one
// spare slot: together with the first half of the running tile, which is free after its first two
// sub-steps, it takes the two halves of tile T + 2 from the MIDDLE of tile T on.  The global loads of
// a tile are thus a whole tile period in flight before they are waited for (with two full-tile stages
// it was half a period: the main loop then ran at "load latency + issue time" per tile, one third
// below the matrix cores' own time, at any clock).
//
// Separate arrays: the compiler orders an LDS read after the direct-to-LDS loads it may alias with by
// a wait on the memory counter, and tells the arrays apart by their identity - reads of one slot do
// not wait for loads still in flight to another.  (This also means every LDS access of the main loop
// must name its slot at compile time: the loop is unrolled over the period of five tiles.)
static __shared__ __attribute__((aligned(1024))) char g_slot0[SLOT_BYTES];
static __shared__ __attribute__((aligned(1024))) char g_slot1[SLOT_BYTES];
static __shared__ __attribute__((aligned(1024))) char g_slot2[SLOT_BYTES];
static __shared__ __attribute__((aligned(1024))) char g_slot3[SLOT_BYTES];
static __shared__ __attribute__((aligned(1024))) char g_slot4[SLOT_BYTES];
static_assert(EPI_XCHG_BYTES + StageF32<128>::BYTES <= SLOT_BYTES, "epilogue staging exceeds an LDS slot");
static_assert(StageBf16<128>::BYTES <= StageF32<128>::BYTES, "bf16 staging block larger than the fp32 one");

template <int S>
__device__ __forceinline__ char* lds_slot() {
    static_assert(S >= 0 && S < N_SLOTS, "slot");
    if constexpr (S == 0) return g_slot0;
    else if constexpr (S == 1) return g_slot1;
    else if constexpr (S == 2) return g_slot2;
    else if constexpr (S == 3) return g_slot3;
    else return g_slot4;
}

__device__ __forceinline__ int seg_swizzle(int k_low2) { return k_low2 ^ ((k_low2 & 1) << 2); }

// Byte offsets (within the operand's buffer, before the k advance) of the P chunks this lane fetches
// for one operand half tile of 64 P rows: wave w fills 1 KB pieces P w .. P w + P - 1 of the half.  The same offsets serve
// both halves of a k tile (the half is selected by the descriptor's base).
template <bool KC, int P = 4>
__device__ __forceinline__ void half_voffsets(unsigned (&voff)[P], int r0, int ld, int wave, int lane) {
#pragma unroll
    for (int jj = 0; jj < P; ++jj) {
        const int piece = wave * P + jj;
        if (KC) {
            const int row = piece * 16 + (lane >> 2);
            const int c = (lane & 3) ^ ((row >> 2) & 3);
            voff[jj] = ((unsigned)(r0 + row) * (unsigned)ld + (unsigned)(c * 8)) * 2u;
        } else {
            const int krow = piece * 2 + (lane >> 5);
            const int cpos = lane & 31;
            const int seg = (cpos >> 1) ^ seg_swizzle(krow & 3);
            const int c = seg * 2 + (cpos & 1);
            voff[jj] = ((unsigned)krow * (unsigned)ld + (unsigned)(r0 + c * 8)) * 2u;
        }
    }
}

// The 8 wave-wide loads that bring this wavefront's share of one operand of k tile `kadv / kstep` in:
// 4 pieces, each as a pair (first half -> slot S0, second half -> slot S1) issued back to back, so that
// the two 64-byte halves of a 128-byte line of a K-contiguous operand meet in the vector cache.  The k
// advance is applied to the descriptors (base += advance, size -= advance, clamped to the operand size:
// a tile past the end of K yields empty descriptors, every lane reads zero and no access is made), so
// the per-lane offsets are loop invariant and the range check still sees the true distance to the end.
template <bool IS_B, int S0, int S1, bool KTAIL, int P>
__device__ __forceinline__ void issue_operand_loads(const void* base, unsigned bytes, unsigned kadv, unsigned half_adv,
                                                    const unsigned (&voff)[P], int wave, unsigned tail0, unsigned tail1) {
    const unsigned adv0 = kadv < bytes ? kadv : bytes;
    const unsigned adv1 = kadv + half_adv < bytes ? kadv + half_adv : bytes;
    const __amdgpu_buffer_rsrc_t rs0 = __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)base + adv0), 0,
                                                                         (int)(bytes - adv0), 0x00020000);
    const __amdgpu_buffer_rsrc_t rs1 = __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)base + adv1), 0,
                                                                         (int)(bytes - adv1), 0x00020000);
#pragma unroll
    for (int jj = 0; jj < P; ++jj) {
        const int off = (IS_B ? HALF_OP_BYTES : 0) + (wave * P + jj) * 1024;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rs0, (lds_ptr)(lds_slot<S0>() + off), 16, (int)(KTAIL ? voff[jj] | tail0 : voff[jj]), 0, 0, 0);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rs1, (lds_ptr)(lds_slot<S1>() + off), 16, (int)(KTAIL ? voff[jj] | tail1 : voff[jj]), 0, 0, 0);
    }
}

// Per-lane LDS byte offsets for operand reads of the wavefront's 128 rows (4 MFMA tiles) in a half.
//  KC: 64-byte rows, 16-byte chunk c of row r at chunk position c ^ ((r >> 2) & 3) (16 consecutive rows
//      with the same chunk then fall into 16 different bank groups).  base[kk] = address of
//      (row = wt*128 + l32, chunk 2kk + hf); tile t adds t*2048.  base[2], base[3] unused.
//  KS: base[t]  = address of (k = 8*(b>>1) + s/4, segment of tile t and lane group b, 8*(s&3));
//                 sub-step kk / half rd adds (16kk + 4rd) * 512
template <bool KC, int MI = 4>
__device__ __forceinline__ void frag_offsets(int (&base)[4], int wt, int lane) {
    if (KC) {
        const int l32 = lane & 31, hf = lane >> 5;
#pragma unroll
        for (int kk = 0; kk < 2; ++kk)
            base[kk] = (wt * (32 * MI) + l32) * 64 + ((((kk << 1) | hf) ^ ((l32 >> 2) & 3)) << 4);
        base[2] = base[3] = 0;
    } else {
        const int b = lane >> 4, s = lane & 15;
        const int f = seg_swizzle(s >> 2);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int seg = (wt * (2 * MI) + t * 2 + (b & 1)) ^ f;
            base[t] = (8 * (b >> 1) + (s >> 2)) * 512 + seg * 32 + 8 * (s & 3);
        }
    }
}

template <bool KC>
__device__ __forceinline__ void opaque_offsets(int (&base)[4]) {
    if (KC) asm volatile("" : "+v"(base[0]), "+v"(base[1]));
    else asm volatile("" : "+v"(base[0]), "+v"(base[1]), "+v"(base[2]), "+v"(base[3]));
}

// kk: sub-step within the half (0 or 1)
template <bool KC>
__device__ __forceinline__ bf16x8 read_operand(const char* half, const int (&base)[4], int t, int kk) {
    if (KC) {
        return *reinterpret_cast<const bf16x8*>(half + base[kk] + t * 2048);
    } else {
        union { short4v h[2]; bf16x8 v; } u;
        const char* p = half + base[t] + kk * 8192;
        u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) short4v*)(p));
        u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) short4v*)(p + 2048));
        return u.v;
    }
}

// MI: row blocks of 32 of a wavefront.
template <bool A_KC, bool B_KC, int MI>
__device__ __forceinline__ void read_frags(bf16x8 (&af)[MI], bf16x8 (&bf)[4], const char* slot, const int (&abase)[4],
                                           const int (&bbase)[4], int kk) {
#pragma unroll
    for (int t = 0; t < MI; ++t) af[t] = read_operand<A_KC>(slot, abase, t, kk);
#pragma unroll
    for (int t = 0; t < 4; ++t) bf[t] = read_operand<B_KC>(slot + HALF_OP_BYTES, bbase, t, kk);
}

template <Epi EPI, int MI>
__device__ __forceinline__ void mfma_step(floatx16 (&acc)[MI][4], const bf16x8 (&af)[MI], const bf16x8 (&bf)[4]) {
    // Column by column in a snake, so that only one of the two operands changes between
    // consecutive MFMAs (less switching on the operand paths; the kernel is power limited).
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int ii = 0; ii < MI; ++ii) {
            const int i = (j & 1) ? MI - 1 - ii : ii;
            mfma_tile<EPI>(acc[i][j], af[i], bf[j]);
        }
}

// Phase stamps of the optional timeline (measurement aid): per workgroup and tile, the constant
// 100 MHz counter and the shader clock at tile start, after the prologue's first barrier, at the
// end of the main loop and at the end of the epilogue (stores issued, not necessarily landed).
constexpr int TRACE_STAMPS = 8;          // 4 phases x {real time, shader clock}
constexpr int TRACE_HEADER = 8;          // words before the first record
template <bool TRACE>
__device__ __forceinline__ void trace_stamp(const GemmBf16Params& g, int tile_idx, int phase) {
    if constexpr (TRACE) {
        if (threadIdx.x == 0 && tile_idx < g.trace_cap) {
            unsigned long long* r = g.trace + TRACE_HEADER + ((size_t)blockIdx.x * g.trace_cap + tile_idx) * TRACE_STAMPS;
            r[2 * phase] = wall_clock64();
            r[2 * phase + 1] = clock64();
        }
    }
}

// Shard that owns tile (or k tile) t of the concatenated dimension.
__device__ __forceinline__ int shard_of(const GemmBf16Group& gg, int t) {
    int r = 0;
#pragma unroll
    for (int i = 1; i < GEMM_GROUP_MAX; ++i) r += t >= gg.first[i] ? 1 : 0;
    return __builtin_amdgcn_readfirstlane(r);
}

// Several shards in one launch (see GemmBf16Group) because one shard alone leaves the chip partly idle: the last round
// of its tiles is not full, every launch ends with its slowest workgroup and its epilogue's stores, and the small ones
// have fewer tiles than there are compute units.  Whole steps, one launch per shard and product -> one per product:
// N=512 h=2048 V=32000 p=4: 954 -> 290 us; N=1999 h=3072 V=50001 p=8: 3048 -> 1888; N=4096 h=4096 V=32000 p=8: 2940 -> 2692;
// N=4096 h=8192 V=256000 p=16: 52.6 -> 51.5 ms; the loss alone, N=64 h=4096 V=128256 p=8: 653 -> 253 us.
//
// MI: row blocks of 32 per wavefront, tiles of 64 MI rows (row_blocks_for); A's half of a slot then holds 64 MI rows.  Up to 256
// tokens the logits products and dH are bound by reading W (N=64 h=4096 V=64000: 97 us, 5.4 TB/s), if the matrix work of a
// k tile and the loads of A stay below that.
template <bool A_KC, bool B_KC, Epi EPI, bool STREAM, bool TRACE, bool KTAIL, int MI = 4>
__global__ __launch_bounds__(NT) void gemm_bf16_fast_kernel(GemmBf16Group gg) {
    constexpr int TM = 64 * MI;
    static_assert(MI == 4 || A_KC, "the K-strided layout has 256 rows");
    constexpr bool CAT_N = A_KC && B_KC, CAT_M = !A_KC && !B_KC, CAT_K = A_KC && !B_KC;
    const GemmBf16Params& g = gg.base;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform: keeps LDS bases in SGPRs
    const int wm = wave >> 1, wn = wave & 1;

    const int tiles_m = CAT_M ? gg.total : (g.M + TM - 1) / TM;
    const int tiles_n = CAT_N ? gg.total : (g.N + BN - 1) / BN;
    const int plane = tiles_m * tiles_n;
    const int pieces = CAT_K ? gg.slices * (gg.each ? gg.n : 1) : 1;      // of K
    const int total_tiles = plane * pieces;

    const unsigned a_row = CAT_K || CAT_M ? 0u : (unsigned)g.lda;      // row stride of A if the shards share it

    int abase[4], bbase[4];
    frag_offsets<A_KC, MI>(abase, wm, lane);
    frag_offsets<B_KC>(bbase, wn, lane);

    // KTAIL: bits that put the offsets of this lane's chunk in the last k tile's two halves beyond every buffer (operands
    // are smaller than 4 GB - 1 MB) where the chunk lies past the end of K (see half_voffsets; K is a multiple of 8)
    unsigned tail0 = 0u, tail1 = 0u;
    if constexpr (KTAIL) {
        const int k = ((lane & 3) ^ ((lane >> 4) & 3)) * 8, left = g.K % BK;
        tail0 = k >= left ? 0xFFFFFF00u : 0u;
        tail1 = k + 32 >= left ? 0xFFFFFF00u : 0u;
    }

    // Persistent workgroups: one per compute unit, each walking the tile list with stride
    // gridDim.x.  The stores of a tile's epilogue are fire-and-forget, so they drain while the
    // next tile's operands are already streaming in.  Virtual id v keeps the XCD-aware tile
    // order: v % 8 is the XCD of this workgroup for every tile it processes.
    if (TRACE && blockIdx.x == 0 && tid == 0) {
        g.trace[0] = gridDim.x; g.trace[1] = (unsigned long long)total_tiles; g.trace[2] = (unsigned long long)g.trace_cap;
    }
    int tile_idx = 0;
    for (int v = blockIdx.x; v < total_tiles; v += gridDim.x, ++tile_idx) {
    trace_stamp<TRACE>(g, tile_idx, 0);
    int tile_m, tile_n, slice = 0;      // tile_m / tile_n: within the shard
    if (pieces > 1) sliced_tile_of_block(v, gridDim.x, plane, pieces, tiles_m, tiles_n, tile_m, tile_n, slice);
    else tile_of_block(v, gridDim.x, total_tiles, tiles_m, tiles_n, tile_m, tile_n);

    // the shard, and for dH the range [kt_at, kt_end) of k tiles of this work item (over all shards)
    int shard, kt_at = 0, kt_end = 0;
    if constexpr (CAT_K) {
        int from = 0, count = gg.total, part = slice;
        if (gg.each) {
            const int r = slice % gg.n;
            part = slice / gg.n;
            from = gg.first[r];
            count = (r + 1 < gg.n ? gg.first[r + 1] : gg.total) - from;
        }
        kt_at = from + (int)((long long)count * part / gg.slices);
        kt_end = from + (int)((long long)count * (part + 1) / gg.slices);
        shard = shard_of(gg, kt_at);
    } else {
        shard = shard_of(gg, CAT_N ? tile_n : tile_m);
        if constexpr (CAT_N) tile_n -= gg.first[shard];
        else tile_m -= gg.first[shard];
    }
    const int m0 = tile_m * TM, n0 = tile_n * BN;

    // operands of the shard; raw buffer descriptors sized exactly to them: reads beyond return zero
    const u16 *opA, *opB;
    unsigned a_bytes, b_bytes, a_kstep, b_kstep, a_half, b_half;
    int cols_n;                  // columns of the output (N)
    int kt_base, nkt;            // first k tile and number of k tiles of this pass over K
    unsigned avoff[MI], bvoff[4];
    auto bind_shard = [&]() {
        const GemmBf16Shard& s = gg.sh[shard];
        const unsigned lda = CAT_N ? a_row : (unsigned)s.ld;
        opA = CAT_N ? g.A : s.A;
        opB = CAT_M ? g.B : s.B;
        const int K = CAT_K ? s.rows : g.K;
        cols_n = CAT_N ? s.rows : g.N;
        const int rows_m = CAT_M ? s.rows : g.M;
        a_bytes = (unsigned)(A_KC ? rows_m : K) * lda * 2u;
        b_bytes = (unsigned)(B_KC ? cols_n : K) * (unsigned)g.ldb * 2u;
        a_kstep = A_KC ? (unsigned)BK * 2u : (unsigned)BK * lda * 2u;
        b_kstep = B_KC ? (unsigned)BK * 2u : (unsigned)BK * (unsigned)g.ldb * 2u;
        a_half = a_kstep >> 1;
        b_half = b_kstep >> 1;
        const int all = (K + BK - 1) / BK;
        if constexpr (CAT_K) {
            kt_base = kt_at - gg.first[shard];
            nkt = min(all - kt_base, kt_end - kt_at);
        } else {
            kt_base = 0;
            nkt = all;
        }
        half_voffsets<A_KC, MI>(avoff, m0, (int)lda, wave, lane);
        half_voffsets<B_KC>(bvoff, n0, g.ldb, wave, lane);
    };
    bind_shard();

    // Instruction-mix hints for the scheduler: the next N MFMAs, LDS reads, global loads.
#define VP_SCHED_MFMA(n) __builtin_amdgcn_sched_group_barrier(0x008, n, 0)
#define VP_SCHED_DSRD(n) __builtin_amdgcn_sched_group_barrier(0x100, n, 0)
#define VP_SCHED_VMEM(n) __builtin_amdgcn_sched_group_barrier(0x020, n, 0)
    constexpr int DS_PER_STEP = (A_KC ? MI : 2 * MI) + (B_KC ? 4 : 8);   // LDS reads per 16-wide k sub-step

    // Loads of k tile T into the slots (2T) % 5 and (2T + 1) % 5.
#define VP_TAIL(T, x) (KTAIL && (T) == nkt - 1 ? (x) : 0u)
#define VP_LOAD_A(T, S0, S1) issue_operand_loads<false, S0, S1, KTAIL, MI>(opA, a_bytes, (unsigned)(kt_base + (T)) * a_kstep, a_half, avoff, wave, VP_TAIL(T, tail0), VP_TAIL(T, tail1))
#define VP_LOAD_B(T, S0, S1) issue_operand_loads<true, S0, S1, KTAIL, 4>(opB, b_bytes, (unsigned)(kt_base + (T)) * b_kstep, b_half, bvoff, wave, VP_TAIL(T, tail0), VP_TAIL(T, tail1))
    // Waits (s_waitcnt immediates: vmcnt in bits 3:0 and 15:14, lgkmcnt in bits 11:8, expcnt 6:4 left at 7).
#define VP_WAIT_LGKM0() __builtin_amdgcn_s_waitcnt(0xC07F)                 /* lgkmcnt(0), vmcnt(63) */
    // all but the 2 MI + 8 loads of a k tile
#define VP_WAIT_TILE_LGKM0() __builtin_amdgcn_s_waitcnt(((2 * MI + 8) & 15) | (((2 * MI + 8) >> 4) << 14) | 0x70)
#define VP_BARRIER()                          \
    asm volatile("" ::: "memory");            \
    __builtin_amdgcn_s_barrier();             \
    asm volatile("" ::: "memory")

    // prologue: k tiles 0 and 1 are requested at once; tile 0 has landed after the first 16 of the 32 loads
#define VP_PROLOGUE()        \
    VP_LOAD_A(0, 0, 1);      \
    VP_LOAD_B(0, 0, 1);      \
    VP_LOAD_A(1, 2, 3);      \
    VP_LOAD_B(1, 2, 3);      \
    asm volatile("" ::: "memory")
    VP_PROLOGUE();
    // (while those loads are on their way)
    // accumulators are zeroed directly in the AGPR half of the register file: zeroing them as
    // ordinary vectors first would need 256 more VGPRs for a moment and spill everything else
    floatx16 acc[MI][4];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) { float z; asm volatile("v_accvgpr_write_b32 %0, 0" : "=a"(z)); acc[i][j][r] = z; }
    if (EPI == Epi::FwdStats && n0 + BN > cols_n) init_acc_ragged<4, 2, MI>(acc, cols_n, tile_n);

    // one pass per shard whose k tiles this work item has (dH); one pass otherwise
    for (bool first_pass = true;; first_pass = false) {
    VP_WAIT_TILE_LGKM0();
    VP_BARRIER();
    if (first_pass) trace_stamp<TRACE>(g, tile_idx, 1);
    bf16x8 af0[MI], bf0[4], af1[MI], bf1[4];
    read_frags<A_KC, B_KC, MI>(af0, bf0, lds_slot<0>(), abase, bbase, 0);

    // One k tile T = four 16-wide sub-steps, operands fetched one sub-step ahead into the other register
    // set.  M = T % 5 fixes the slots: first half H0 = 2M % 5, second half H1 = (2M+1) % 5, first half
    // of the next tile NX = (2M+2) % 5; the loads of tile T + 2 go to L0 = (2M+4) % 5 (the spare slot,
    // last read before the previous tile's second barrier) and L1 = (2M+5) % 5 = H0.
    //   sub-step 0: last reads of H0, then barrier 1: every wavefront is done with H0.
    //   sub-steps 1, 2: the 16 loads of tile T + 2, one every two MFMAs (the rate the texture-address
    //            unit sustains; a burst stalls the in-order wavefront), A pairs then B pairs.  Sub-step 2
    //            ends with barrier 2, after waiting for all but those 16 loads: tile T + 1 has landed
    //            (it was requested one tile period ago), and every wavefront is done with H1.
    //   sub-step 3: first operands of tile T + 1 from NX.
#define VP_SHARE(q, n, of) (((q) + 1) * (n) / (of) - (q) * (n) / (of))
#define VP_MIX_1(q, L)                                                                                   \
    VP_SCHED_MFMA(VP_SHARE(q, 4 * MI, 8));                                                               \
    VP_SCHED_DSRD((DS_PER_STEP + 7) / 8);                                                                \
    VP_SCHED_VMEM(VP_SHARE(q, L, 8));
#define VP_MIX_LOADS(L)   /* 4 MI MFMAs, the sub-step's operand reads and L global loads */             \
    VP_MIX_1(0, L) VP_MIX_1(1, L) VP_MIX_1(2, L) VP_MIX_1(3, L) VP_MIX_1(4, L) VP_MIX_1(5, L) VP_MIX_1(6, L) VP_MIX_1(7, L)
#define VP_LAST_1(q)                                                                                     \
    VP_SCHED_MFMA(VP_SHARE(q, 4 * MI - 1, 5));                                                           \
    VP_SCHED_DSRD((DS_PER_STEP + 4) / 5);
#define VP_TILE(M, T)                                                                                    \
    {                                                                                                    \
        constexpr int H0 = (2 * (M)) % 5, H1 = (2 * (M) + 1) % 5, NX = (2 * (M) + 2) % 5, L0 = (2 * (M) + 4) % 5; \
        opaque_offsets<A_KC>(abase);   /* keeps "slot address + lane offset" sums from being hoisted out of */ \
        opaque_offsets<B_KC>(bbase);   /* the loop for all five slots at once (they would spill)            */ \
        read_frags<A_KC, B_KC, MI>(af1, bf1, lds_slot<H0>(), abase, bbase, 1);                                \
        mfma_step<EPI, MI>(acc, af0, bf0);                                                                   \
        _Pragma("unroll") for (int q = 0; q < 4; ++q) {   /* operand reads early: they must have */     \
            VP_SCHED_MFMA(1);                               /* landed when the barrier is reached  */     \
            VP_SCHED_DSRD((DS_PER_STEP + 3) / 4);                                                        \
        }                                                                                                \
        VP_SCHED_MFMA(4 * MI - 4);                                                                               \
        VP_WAIT_LGKM0();                                                                                 \
        VP_BARRIER();                                                                                    \
        read_frags<A_KC, B_KC, MI>(af0, bf0, lds_slot<H1>(), abase, bbase, 0);                                \
        VP_LOAD_A((T) + 2, L0, H0);                                                                      \
        mfma_step<EPI, MI>(acc, af1, bf1);                                                                   \
        VP_MIX_LOADS(2 * MI)                                                                                 \
        read_frags<A_KC, B_KC, MI>(af1, bf1, lds_slot<H1>(), abase, bbase, 1);                                \
        VP_LOAD_B((T) + 2, L0, H0);                                                                      \
        mfma_step<EPI, MI>(acc, af0, bf0);                                                                   \
        VP_MIX_LOADS(8)                                                                                  \
        VP_WAIT_TILE_LGKM0();                                                                            \
        VP_BARRIER();                                                                                    \
        read_frags<A_KC, B_KC, MI>(af0, bf0, lds_slot<NX>(), abase, bbase, 0);                                \
        mfma_step<EPI, MI>(acc, af1, bf1);                                                                   \
        VP_LAST_1(0) VP_LAST_1(1) VP_LAST_1(2) VP_LAST_1(3) VP_LAST_1(4)                                 \
        VP_SCHED_MFMA(1);                                                                                \
    }

    // The period of the slot assignment is five tiles: whole periods in a loop without exits (the state of
    // loads in flight is the same at its entry and at its back edge: tile T + 1 on its way into slots 2
    // and 3), the remaining nkt % 5 tiles as straight-line code behind it.
    int kt = 0;
    for (int it = nkt / 5; it > 0; --it) {
        VP_TILE(0, kt)
        VP_TILE(1, kt + 1)
        VP_TILE(2, kt + 2)
        VP_TILE(3, kt + 3)
        VP_TILE(4, kt + 4)
        kt += 5;
    }
    {
        const int rem = nkt - kt;
        if (rem > 0) {
            VP_TILE(0, kt)
            if (rem > 1) {
                VP_TILE(1, kt + 1)
                if (rem > 2) {
                    VP_TILE(2, kt + 2)
                    if (rem > 3) {
                        VP_TILE(3, kt + 3)
                    }
                }
            }
        }
    }
    __syncthreads();   // every wavefront is done with the slots, and no load is in flight, before they are reused
    if constexpr (!CAT_K) break;
    else {
        kt_at += nkt;
        if (kt_at >= kt_end) break;
        ++shard;       // (every shard has at least one k tile)
        bind_shard();
        VP_PROLOGUE();
    }
    }
#undef VP_PROLOGUE
#undef VP_TILE
#undef VP_MIX_LOADS
#undef VP_MIX_1
#undef VP_LAST_1
#undef VP_SHARE
#undef VP_TAIL
#undef VP_LOAD_A
#undef VP_LOAD_B
#undef VP_WAIT_LGKM0
#undef VP_WAIT_TILE_LGKM0
#undef VP_BARRIER
#undef VP_SCHED_MFMA
#undef VP_SCHED_DSRD
#undef VP_SCHED_VMEM
    trace_stamp<TRACE>(g, tile_idx, 2);

    // keep the epilogue's address arithmetic from being hoisted above the main loop, where it
    // would occupy registers (and spill) for the whole kernel
    asm volatile("" : "+s"(tile_m), "+s"(tile_n), "+s"(shard), "+s"(slice));
    GemmBf16Params e = g;        // the shard's output
    {
        const GemmBf16Shard& s = gg.sh[shard];
        if constexpr (CAT_N) {
            e.N = s.rows;
            e.Y = (u16*)s.out;
            e.ldy = s.ld;
            e.shard_offset = s.offset;
            if constexpr (EPI == Epi::FwdStats) {
                e.part_max = g.part_max + (size_t)gg.first[shard] * g.M;
                e.part_sum = g.part_sum + (size_t)gg.first[shard] * g.M;
                e.part_tgt = g.part_tgt + (size_t)shard * g.M;
            }
        } else if constexpr (CAT_M) {
            e.M = s.rows;
            e.C = (float*)s.out;
        } else {
            e.C = g.C + (size_t)slice * g.M * g.ldc;
        }
    }
    // exchange area at the start of slot 0; staging block of wavefront w in slot w (behind the exchange area in slot 0)
    gemm_epilogue<EPI, 4, 2, STREAM, MI>(acc, e, tile_m, tile_n, g_slot0,
                                     wave == 0 ? g_slot0 + EPI_XCHG_BYTES : wave == 1 ? g_slot1 : wave == 2 ? g_slot2 : g_slot3);
    __syncthreads();   // the epilogue's LDS exchange is over before the next tile streams in
    trace_stamp<TRACE>(g, tile_idx, 3);
    }   // persistent tile loop
}

// Compute units of the current device.
int compute_unit_count();
// The measurement aid's buffer if launches of this kernel id are to be traced, else nullptr.
unsigned long long* gemm_bf16_trace_buffer(int kernel_id, size_t& words);
// Row blocks per wavefront for M rows, tn tile columns (times slices) and kt k tiles each (stats: the logits products).
int row_blocks_for(int64_t M, int64_t tn, int64_t kt, bool stats, int cus);

// One instantiation's launch.
template <bool A_KC, bool B_KC, Epi EPI, int MI, bool KTAIL>
static void launch_tiles(const GemmBf16Group& p, int tiles, int cus, hipStream_t st) {
    // more tiles than workgroups: outputs are streamed past the L2 (see gemm_epilogue)
    if (tiles > cus)
        hipLaunchKernelGGL((gemm_bf16_fast_kernel<A_KC, B_KC, EPI, true, false, KTAIL, MI>), dim3(cus), dim3(NT), 0, st, p);
    else
        hipLaunchKernelGGL((gemm_bf16_fast_kernel<A_KC, B_KC, EPI, false, false, KTAIL, MI>), dim3(tiles), dim3(NT), 0, st, p);
}

template <bool A_KC, bool B_KC, Epi EPI>
static hipError_t launch_fast_t(const GemmBf16Group& p0, hipStream_t st) {
    GemmBf16Group p = p0;
    const bool cat_k = A_KC && !B_KC, ktail = A_KC && B_KC && p.base.K % BK != 0;
    const int cus = compute_unit_count();
    const int64_t tn = A_KC && B_KC ? p.total : ceil_div(p.base.N, BN);
    const int pieces = cat_k ? p.slices * (p.each ? p.n : 1) : 1;
    size_t words = 0;
    unsigned long long* tb = gemm_bf16_trace_buffer(p.base.kernel_id, words);
    int mi = 4;
    if (A_KC && !tb) mi = row_blocks_for(p.base.M, tn * pieces, cat_k ? ceil_div(p.total, pieces) : ceil_div(p.base.K, BK), !cat_k, cus);
    const int64_t tm = !A_KC ? p.total : ceil_div(p.base.M, 64 * mi);
    const int tiles = (int)(tm * tn) * pieces;
    if constexpr (A_KC) {
        if (mi < 4) {
            if constexpr (B_KC) {
                if (ktail) {
                    if (mi == 1) launch_tiles<A_KC, B_KC, EPI, 1, true>(p, tiles, cus, st);
                    else if (mi == 2) launch_tiles<A_KC, B_KC, EPI, 2, true>(p, tiles, cus, st);
                    else launch_tiles<A_KC, B_KC, EPI, 3, true>(p, tiles, cus, st);
                    return hipGetLastError();
                }
            }
            if (mi == 1) launch_tiles<A_KC, B_KC, EPI, 1, false>(p, tiles, cus, st);
            else if (mi == 2) launch_tiles<A_KC, B_KC, EPI, 2, false>(p, tiles, cus, st);
            else launch_tiles<A_KC, B_KC, EPI, 3, false>(p, tiles, cus, st);
            return hipGetLastError();
        }
    }
    if constexpr (A_KC && B_KC) {
        if (ktail) {      // (not traced)
            launch_tiles<A_KC, B_KC, EPI, 4, true>(p, tiles, cus, st);
            return hipGetLastError();
        }
    }
    if (tb) {   // measurement aid: the instrumented instantiation, if the buffer holds this launch's records
        const int grid = tiles > cus ? cus : tiles, per_wg = (int)ceil_div(tiles, grid);
        if ((size_t)TRACE_HEADER + (size_t)grid * per_wg * TRACE_STAMPS <= words) {
            p.base.trace = tb;
            p.base.trace_cap = per_wg;
            if (tiles > cus)
                hipLaunchKernelGGL((gemm_bf16_fast_kernel<A_KC, B_KC, EPI, true, true, false>), dim3(grid), dim3(NT), 0, st, p);
            else
                hipLaunchKernelGGL((gemm_bf16_fast_kernel<A_KC, B_KC, EPI, false, true, false>), dim3(grid), dim3(NT), 0, st, p);
            return hipGetLastError();
        }
    }
    launch_tiles<A_KC, B_KC, EPI, 4, false>(p, tiles, cus, st);
    return hipGetLastError();
}

}  // namespace vp
