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
#include <atomic>
#include <climits>

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
__shared__ __attribute__((aligned(1024))) char g_slot0[SLOT_BYTES];
__shared__ __attribute__((aligned(1024))) char g_slot1[SLOT_BYTES];
__shared__ __attribute__((aligned(1024))) char g_slot2[SLOT_BYTES];
__shared__ __attribute__((aligned(1024))) char g_slot3[SLOT_BYTES];
__shared__ __attribute__((aligned(1024))) char g_slot4[SLOT_BYTES];
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

// Byte offsets (within the operand's buffer, before the k advance) of the 4 chunks this lane fetches
// for one operand half tile: wave w fills 1 KB pieces 4w .. 4w+3 of the half.  The same offsets serve
// both halves of a k tile (the half is selected by the descriptor's base).
template <bool KC>
__device__ __forceinline__ void half_voffsets(unsigned (&voff)[4], int r0, int ld, int wave, int lane) {
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {
        const int piece = wave * 4 + jj;
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
template <bool IS_B, int S0, int S1, bool KTAIL>
__device__ __forceinline__ void issue_operand_loads(const void* base, unsigned bytes, unsigned kadv, unsigned half_adv,
                                                    const unsigned (&voff)[4], int wave, unsigned tail0, unsigned tail1) {
    const unsigned adv0 = kadv < bytes ? kadv : bytes;
    const unsigned adv1 = kadv + half_adv < bytes ? kadv + half_adv : bytes;
    const __amdgpu_buffer_rsrc_t rs0 = __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)base + adv0), 0,
                                                                         (int)(bytes - adv0), 0x00020000);
    const __amdgpu_buffer_rsrc_t rs1 = __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)base + adv1), 0,
                                                                         (int)(bytes - adv1), 0x00020000);
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {
        const int off = (IS_B ? HALF_OP_BYTES : 0) + (wave * 4 + jj) * 1024;
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
template <bool KC>
__device__ __forceinline__ void frag_offsets(int (&base)[4], int wt, int lane) {
    if (KC) {
        const int l32 = lane & 31, hf = lane >> 5;
#pragma unroll
        for (int kk = 0; kk < 2; ++kk)
            base[kk] = (wt * 128 + l32) * 64 + ((((kk << 1) | hf) ^ ((l32 >> 2) & 3)) << 4);
        base[2] = base[3] = 0;
    } else {
        const int b = lane >> 4, s = lane & 15;
        const int f = seg_swizzle(s >> 2);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int seg = (wt * 8 + t * 2 + (b & 1)) ^ f;
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

// MI: row blocks of 32 of the wavefront's 128 rows that are multiplied (the others lie past the end of M).
template <bool A_KC, bool B_KC, int MI>
__device__ __forceinline__ void read_frags(bf16x8 (&af)[4], bf16x8 (&bf)[4], const char* slot, const int (&abase)[4],
                                           const int (&bbase)[4], int kk) {
#pragma unroll
    for (int t = 0; t < MI; ++t) af[t] = read_operand<A_KC>(slot, abase, t, kk);
#pragma unroll
    for (int t = 0; t < 4; ++t) bf[t] = read_operand<B_KC>(slot + HALF_OP_BYTES, bbase, t, kk);
}

template <Epi EPI, int MI>
__device__ __forceinline__ void mfma_step(floatx16 (&acc)[4][4], const bf16x8 (&af)[4], const bf16x8 (&bf)[4]) {
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
// MI = 2: at most 64 rows (tokens): every wavefront multiplies the first two of its four row blocks, so half the tile (the
// half of it that the lower two wavefronts have are rows past the end).  The products are then bound by reading W, and the
// loads of a k tile wait for the wavefront's matrix work no longer: N=16 h=2048 V=32000: 46 -> 36 us (3.7 TB/s), N=64 h=4096
// V=128256 p=8: 230 -> 198 us (5.3 TB/s).  A third row block would be the next step: 65 and 96 tokens take 231 and 228 us
// with the whole tile, 128 take 248.
template <bool A_KC, bool B_KC, Epi EPI, bool STREAM, bool TRACE, bool KTAIL, int MI = 4>
__global__ __launch_bounds__(NT) void gemm_bf16_fast_kernel(GemmBf16Group gg) {
    constexpr bool CAT_N = A_KC && B_KC, CAT_M = !A_KC && !B_KC, CAT_K = A_KC && !B_KC;
    const GemmBf16Params& g = gg.base;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform: keeps LDS bases in SGPRs
    const int wm = wave >> 1, wn = wave & 1;

    const int tiles_m = CAT_M ? gg.total : (g.M + BM - 1) / BM;
    const int tiles_n = CAT_N ? gg.total : (g.N + BN - 1) / BN;
    const int plane = tiles_m * tiles_n;
    const int pieces = CAT_K ? gg.slices * (gg.each ? gg.n : 1) : 1;      // of K
    const int total_tiles = plane * pieces;

    const unsigned a_row = CAT_K || CAT_M ? 0u : (unsigned)g.lda;      // row stride of A if the shards share it

    int abase[4], bbase[4];
    frag_offsets<A_KC>(abase, wm, lane);
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
    const int m0 = tile_m * BM, n0 = tile_n * BN;

    // operands of the shard; raw buffer descriptors sized exactly to them: reads beyond return zero
    const u16 *opA, *opB;
    unsigned a_bytes, b_bytes, a_kstep, b_kstep, a_half, b_half;
    int cols_n;                  // columns of the output (N)
    int kt_base, nkt;            // first k tile and number of k tiles of this pass over K
    unsigned avoff[4], bvoff[4];
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
        half_voffsets<A_KC>(avoff, m0, (int)lda, wave, lane);
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
#define VP_LOAD_A(T, S0, S1) issue_operand_loads<false, S0, S1, KTAIL>(opA, a_bytes, (unsigned)(kt_base + (T)) * a_kstep, a_half, avoff, wave, VP_TAIL(T, tail0), VP_TAIL(T, tail1))
#define VP_LOAD_B(T, S0, S1) issue_operand_loads<true, S0, S1, KTAIL>(opB, b_bytes, (unsigned)(kt_base + (T)) * b_kstep, b_half, bvoff, wave, VP_TAIL(T, tail0), VP_TAIL(T, tail1))
    // Waits (s_waitcnt immediates: vmcnt in bits 3:0 and 15:14, lgkmcnt in bits 11:8, expcnt 6:4 left at 7).
#define VP_WAIT_LGKM0() __builtin_amdgcn_s_waitcnt(0xC07F)                 /* lgkmcnt(0), vmcnt(63) */
#define VP_WAIT_VM16_LGKM0() __builtin_amdgcn_s_waitcnt(0x4070)            /* vmcnt(16) lgkmcnt(0) */
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
    floatx16 acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) { float z; asm volatile("v_accvgpr_write_b32 %0, 0" : "=a"(z)); acc[i][j][r] = z; }
    if (EPI == Epi::FwdStats && n0 + BN > cols_n) init_acc_ragged<4, 2>(acc, cols_n, tile_n);

    // one pass per shard whose k tiles this work item has (dH); one pass otherwise
    for (bool first_pass = true;; first_pass = false) {
    VP_WAIT_VM16_LGKM0();
    VP_BARRIER();
    if (first_pass) trace_stamp<TRACE>(g, tile_idx, 1);
    bf16x8 af0[4], bf0[4], af1[4], bf1[4];
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
#define VP_MIX_LOADS()   /* 16 MFMAs, the sub-step's operand reads and 8 global loads */              \
    _Pragma("unroll") for (int q = 0; q < 8; ++q) {                                                       \
        VP_SCHED_MFMA(MI == 4 ? 2 : 1);                                                                                \
        VP_SCHED_DSRD((DS_PER_STEP + 7) / 8);                                                            \
        VP_SCHED_VMEM(1);                                                                                \
    }
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
        VP_SCHED_MFMA(MI == 4 ? 12 : 4);                                                                               \
        VP_WAIT_LGKM0();                                                                                 \
        VP_BARRIER();                                                                                    \
        read_frags<A_KC, B_KC, MI>(af0, bf0, lds_slot<H1>(), abase, bbase, 0);                                \
        VP_LOAD_A((T) + 2, L0, H0);                                                                      \
        mfma_step<EPI, MI>(acc, af1, bf1);                                                                   \
        VP_MIX_LOADS()                                                                                   \
        read_frags<A_KC, B_KC, MI>(af1, bf1, lds_slot<H1>(), abase, bbase, 1);                                \
        VP_LOAD_B((T) + 2, L0, H0);                                                                      \
        mfma_step<EPI, MI>(acc, af0, bf0);                                                                   \
        VP_MIX_LOADS()                                                                                   \
        VP_WAIT_VM16_LGKM0();                                                                            \
        VP_BARRIER();                                                                                    \
        read_frags<A_KC, B_KC, MI>(af0, bf0, lds_slot<NX>(), abase, bbase, 0);                                \
        mfma_step<EPI, MI>(acc, af1, bf1);                                                                   \
        _Pragma("unroll") for (int q = 0; q < 5; ++q) {                                                   \
            VP_SCHED_MFMA(MI == 4 ? 3 : 1);                                                                            \
            VP_SCHED_DSRD((DS_PER_STEP + 4) / 5);                                                        \
        }                                                                                                \
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
#undef VP_TAIL
#undef VP_LOAD_A
#undef VP_LOAD_B
#undef VP_WAIT_LGKM0
#undef VP_WAIT_VM16_LGKM0
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
    gemm_epilogue<EPI, 4, 2, STREAM>(acc, e, tile_m, tile_n, g_slot0,
                                     wave == 0 ? g_slot0 + EPI_XCHG_BYTES : wave == 1 ? g_slot1 : wave == 2 ? g_slot2 : g_slot3);
    __syncthreads();   // the epilogue's LDS exchange is over before the next tile streams in
    trace_stamp<TRACE>(g, tile_idx, 3);
    }   // persistent tile loop
}

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
__shared__ __attribute__((aligned(1024))) char g_twin0[TWIN_SLOT_BYTES];
__shared__ __attribute__((aligned(1024))) char g_twin1[TWIN_SLOT_BYTES];
__shared__ __attribute__((aligned(1024))) char g_twin2[TWIN_SLOT_BYTES];
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
        gemm_epilogue_f32<Epi::StoreF32, 2, 2, true>(acc, e, tile_m, tile_n,
                                                     (wave < 2 ? g_twin0 : g_twin1) + (wave & 1) * StageF32<64>::BYTES);
        __syncthreads();   // the staging blocks are read before the next tile streams in
    }
}

// Compute units of the current device (one persistent workgroup each); queried once per device.
static int compute_unit_count() {
    static std::atomic<int> cached[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    int n = cached[dev].load(std::memory_order_relaxed);
    if (n == 0) {
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
        cached[dev].store(n, std::memory_order_relaxed);   // every thread computes the same value
    }
    return n;
}

// Timeline buffer of the measurement aid (device memory owned by the caller of vp_profile_gemm_trace).
static std::atomic<unsigned long long*> g_trace_buf{nullptr};
static std::atomic<size_t> g_trace_words{0};
static std::atomic<int> g_trace_kernel{-1};

void gemm_bf16_set_trace(void* buf, size_t bytes, int kernel_id) {
    g_trace_words.store(buf ? bytes / sizeof(unsigned long long) : 0);
    g_trace_kernel.store(kernel_id);
    g_trace_buf.store((unsigned long long*)buf);
}

template <bool A_KC, bool B_KC, Epi EPI>
static hipError_t launch_fast_t(const GemmBf16Group& p0, hipStream_t st) {
    GemmBf16Group p = p0;
    const int64_t tm = !A_KC && !B_KC ? p.total : ceil_div(p.base.M, BM), tn = A_KC && B_KC ? p.total : ceil_div(p.base.N, BN);
    const int tiles = (int)(tm * tn) * (A_KC && !B_KC ? p.slices * (p.each ? p.n : 1) : 1);
    const int cus = compute_unit_count();
    const int grid = tiles > cus ? cus : tiles;
    if constexpr (A_KC && B_KC) {
        if (p.base.M <= 64 && !g_trace_buf.load()) {
            if (p.base.K % BK)
                hipLaunchKernelGGL((gemm_bf16_fast_kernel<A_KC, B_KC, EPI, false, false, true, 2>), dim3(grid), dim3(NT), 0, st, p);
            else
                hipLaunchKernelGGL((gemm_bf16_fast_kernel<A_KC, B_KC, EPI, false, false, false, 2>), dim3(grid), dim3(NT), 0, st, p);
            return hipGetLastError();
        }
        if (p.base.K % BK) {      // (not traced)
            if (tiles > cus)
                hipLaunchKernelGGL((gemm_bf16_fast_kernel<A_KC, B_KC, EPI, true, false, true>), dim3(grid), dim3(NT), 0, st, p);
            else
                hipLaunchKernelGGL((gemm_bf16_fast_kernel<A_KC, B_KC, EPI, false, false, true>), dim3(grid), dim3(NT), 0, st, p);
            return hipGetLastError();
        }
    }
    unsigned long long* tb = g_trace_buf.load();
    const int want = g_trace_kernel.load();
    if (tb && (want < 0 || want == p.base.kernel_id)) {   // measurement aid: the instrumented instantiation, if the buffer holds this launch's records
        const int per_wg = (int)ceil_div(tiles, grid);
        if ((size_t)TRACE_HEADER + (size_t)grid * per_wg * TRACE_STAMPS <= g_trace_words.load()) {
            p.base.trace = tb;
            p.base.trace_cap = per_wg;
            if (tiles > cus)
                hipLaunchKernelGGL((gemm_bf16_fast_kernel<A_KC, B_KC, EPI, true, true, false>), dim3(grid), dim3(NT), 0, st, p);
            else
                hipLaunchKernelGGL((gemm_bf16_fast_kernel<A_KC, B_KC, EPI, false, true, false>), dim3(grid), dim3(NT), 0, st, p);
            return hipGetLastError();
        }
    }
    // more tiles than workgroups: outputs are streamed past the L2 (see gemm_epilogue)
    if (tiles > cus)
        hipLaunchKernelGGL((gemm_bf16_fast_kernel<A_KC, B_KC, EPI, true, false, false>), dim3(grid), dim3(NT), 0, st, p);
    else
        hipLaunchKernelGGL((gemm_bf16_fast_kernel<A_KC, B_KC, EPI, false, false, false>), dim3(grid), dim3(NT), 0, st, p);
    return hipGetLastError();
}

// Up to this many tokens dW takes the kernel with two workgroups per compute unit.  Large tile -> this one, us per launch:
// K = 64 (h=4096, V=128256) 497 -> 375, 200 (4096, 64000) 343 -> 287, 512 (2048, 32000) 118 -> 98, 700 (1512, 50001)
// 169 -> 153, 1024 (4096, 32000) 334 -> 320, 1999 (3072, 50001) 635 -> 634, 4096 (4096, 32000) 986 -> 1030.
constexpr int DW_TWIN_MAX_K = 1536;
static hipError_t launch_dw(const GemmBf16Group& g, hipStream_t st) {
    const bool traced = g_trace_buf.load() && (g_trace_kernel.load() < 0 || g_trace_kernel.load() == g.base.kernel_id);
    if (g.base.K > DW_TWIN_MAX_K || traced) return launch_fast_t<false, false, Epi::StoreF32>(g, st);
    const int tiles = (int)(g.total * ceil_div(g.base.N, TWIN_BN)), room = 2 * compute_unit_count();
    hipLaunchKernelGGL(gemm_bf16_dw_twin_kernel, dim3(tiles > room ? room : tiles), dim3(NT), 0, st, g);
    return hipGetLastError();
}

bool gemm_bf16_fast_ok(const GemmBf16Params& p) {
    if (!p.vec_ok) return false;
    if (((uintptr_t)p.A | (uintptr_t)p.B) & 15u) return false;
    if ((p.lda % 8) || (p.ldb % 8)) return false;
    if (p.K % 8 && p.a_kcontig && p.b_kcontig) return false;
    // byte offsets are 32-bit: the furthest lane of the zero-filled overhang must still not wrap
    const uint64_t lim = ((uint64_t)1 << 32) - ((uint64_t)1 << 20);
    const uint64_t a_ext = p.a_kcontig ? ((uint64_t)p.M + BM) * p.lda * 2 + 2 * (uint64_t)p.K + 256
                                       : ((uint64_t)p.K + BK) * p.lda * 2 + 2 * ((uint64_t)p.M + BM);
    const uint64_t b_ext = p.b_kcontig ? ((uint64_t)p.N + BN) * p.ldb * 2 + 2 * (uint64_t)p.K + 256
                                       : ((uint64_t)p.K + BK) * p.ldb * 2 + 2 * ((uint64_t)p.N + BN);
    return a_ext < lim && b_ext < lim;
}

// Shard r of a group as a product of its own.
static GemmBf16Params shard_params(const GemmBf16Group& g, int r) {
    GemmBf16Params p = g.base;
    const GemmBf16Shard& s = g.sh[r];
    if (p.a_kcontig && p.b_kcontig) { p.B = s.B; p.N = s.rows; p.Y = (u16*)s.out; p.ldy = s.ld; }
    else if (p.a_kcontig) { p.A = s.A; p.lda = s.ld; p.B = s.B; p.K = s.rows; }
    else { p.A = s.A; p.lda = s.ld; p.M = s.rows; p.C = (float*)s.out; }
    return p;
}

bool gemm_bf16_group_ok(const GemmBf16Group& g) {
    if (g.n < 1 || g.n > GEMM_GROUP_MAX || gemm_bf16_generic_forced()) return false;
    for (int r = 0; r < g.n; ++r) {
        const GemmBf16Params p = shard_params(g, r);
        if (p.M < 1 || p.N < 1 || p.K < 1 || !gemm_bf16_fast_ok(p) || !gemm_bf16_out_ok(p)) return false;
    }
    return true;
}

void gemm_bf16_group_finish(GemmBf16Group& g, int n) {
    const int unit = g.base.a_kcontig ? (g.base.b_kcontig ? BN : BK) : BM;
    g.n = n;
    g.slices = g.slices > 1 ? g.slices : 1;
    g.total = 0;
    for (int r = 0; r < GEMM_GROUP_MAX; ++r) {
        g.first[r] = r < n ? g.total : INT_MAX;
        if (r < n) g.total += (int)ceil_div(g.sh[r].rows, unit);
    }
}

hipError_t launch_gemm_bf16_group(const GemmBf16Group& g, hipStream_t st) {
    const GemmBf16Params& p = g.base;
    ProfScope prof(p.kernel_id, st);
    if (p.a_kcontig && p.b_kcontig && p.epi == Epi::FwdStats) return launch_fast_t<true, true, Epi::FwdStats>(g, st);
    if (p.a_kcontig && p.b_kcontig && p.epi == Epi::DLogits) return launch_fast_t<true, true, Epi::DLogits>(g, st);
    if (p.a_kcontig && !p.b_kcontig && p.epi == Epi::AccumF32) return launch_fast_t<true, false, Epi::AccumF32>(g, st);
    if (p.a_kcontig && !p.b_kcontig && p.epi == Epi::StoreF32) return launch_fast_t<true, false, Epi::StoreF32>(g, st);
    if (!p.a_kcontig && !p.b_kcontig && p.epi == Epi::StoreF32) return launch_dw(g, st);
    return hipErrorInvalidValue;
}

hipError_t launch_gemm_bf16_fast(const GemmBf16Params& p, hipStream_t st) {
    GemmBf16Group g{};
    g.base = p;
    GemmBf16Shard& s = g.sh[0];
    s.A = p.A; s.B = p.B; s.offset = p.shard_offset;
    if (p.a_kcontig && p.b_kcontig) { s.out = p.Y; s.rows = p.N; s.ld = p.ldy; }
    else if (p.a_kcontig) { s.rows = p.K; s.ld = p.lda; }
    else { s.out = p.C; s.rows = p.M; s.ld = p.lda; }
    gemm_bf16_group_finish(g, 1);
    return launch_gemm_bf16_group(g, st);
}

// A dH product has only N h / 65536 tiles but the whole vocabulary as K, so with few tokens most compute units would
// idle (512 tokens, h = 2048: 16 tiles).  The k tiles are cut into S equal slices per output tile; the least estimated
// time wins: rounds of 256 workgroups at 1.1 us per k tile (256 x 256 x 64 at 2400 cycles) and 5 us per tile for its
// start and its stores, and for S > 1 the partial outputs written and read once at 4 TB/s and another launch.  The products
// A_r = softmax'_r W_r of Algorithm 2 are n outputs of kt k tiles each in one launch: N=71 h=896 V=14003 p=8, step 619 -> 121 us
// (with the logits of all shards in one launch too), N=136 h=7040 V=79658 p=2 2356 -> 1369, N=4096 h=4096 V=32000 p=8 3132 -> 2947.
static int slices_of(int64_t M, int64_t N, int64_t kt, int n) {
    const int64_t tiles = ceil_div(M, BM) * ceil_div(N, BN) * n;
    int best = 1;
    double best_us = 0;
    for (int64_t S = 1; S <= 32 && (S == 1 || S * 8 <= kt) && (S == 1 || S * n * M * N <= (int64_t)1 << 28); ++S) {
        double us = (double)ceil_div(tiles * S, 256) * ((double)ceil_div(kt, S) * 1.1 + 5.0);
        if (S > 1) us += (double)(S * n * M * N) * 8.0 / 4e6 + 5.0;
        if (S == 1 || us < best_us) {
            best = (int)S;
            best_us = us;
        }
    }
    return best;
}
int gemm_bf16_slices(int64_t M, int64_t N, int64_t kt) { return slices_of(M, N, kt, 1); }
int gemm_bf16_slices_each(int64_t M, int64_t N, int64_t kt, int n) { return slices_of(M, N, kt, n); }

}  // namespace vp
