// Host side of the fast bf16 kernels (vp_gemm_bf16_fast.h): preconditions, groups, the choice of kernel, tile and slices; and the
// instantiations of dH and dW.
#include <atomic>
#include <climits>

#include "vp_gemm_bf16_fast.h"

namespace vp {

hipError_t launch_gemm_bf16_fwd_stats(const GemmBf16Group& g, hipStream_t st);     // vp_gemm_bf16_logits.hip
hipError_t launch_gemm_bf16_dlogits(const GemmBf16Group& g, hipStream_t st);
hipError_t launch_gemm_bf16_dw_twin(const GemmBf16Group& g, hipStream_t st);       // vp_gemm_bf16_twin.hip

// Compute units of the current device (one persistent workgroup each); queried once per device.
int compute_unit_count() {
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

// Estimated time of a tile of 64 mi rows with kt k tiles.  stats: the epilogues of the logits products, else fp32 stores.
// Fitted to N=1024 h=4096 and h=1024, V=64000 p=4, us per launch for mi = 4, 3, 2, 1: logits 433, 459, 525, 786 and 161, 156, 170,
// 229; dH (4 slices) 409, 615 (a second round), 488, 718.
static double tile_us(int mi, int64_t kt, bool stats) {
    static const double step[5] = {0, 0.72, 0.93, 1.04, 1.42}, end[5] = {0, 2.8, 6.2, 9.3, 17.4};
    return (double)kt * step[mi] + (stats ? end[mi] : 1.0 + mi);
}
// dH and A of Algorithm 2 of more tokens than this (fewer: tile_us).  Estimated time of `tiles` tiles of 64 mi rows (mi = 2, 3, 4)
// with kt k tiles each: the part is power limited, so a k tile takes the longer the more compute units work at once (`all` of them, or
// close to none), and a lower tile must save rows that do not exist, not only fill the last round.  An estimate without that
// (tile_us) took 192 rows and other slices where 256 are faster, h=6144 V=128256, us: 3100 tokens 4077 -> 4480, 1536: 1865 -> 1982,
// h=4096 V=128256: 1800: 1517 -> 1718, 800: 775 -> 849; with 256 rows only, it loses 520 (h=4096 V=128256): 528 -> 615, 1300
// (h=3072 V=50001): 353 -> 386, 2600: 709 -> 788.  Of 126 sizes of 520 to 4000 tokens this one is more than 2 % of the product behind
// the better of the two at three, 12 us at most.  (128 rows: 6 % more than measured, which keeps them to where they save the most.)
constexpr int DH_FEW = 512;
static double dh_us(int mi, int64_t tiles, int64_t kt, int cus) {
    static const double none[5] = {0, 0, 0.51, 0.85, 0.98}, all[5] = {0, 0, 1.02, 1.30, 1.56}, end[5] = {0, 0, 1.5, 3.3, 5.2};
    const int64_t full = tiles / cus, last = tiles % cus;
    double us = (double)full * ((double)kt * all[mi] + end[mi]);
    if (last) us += (double)kt * (none[mi] + (all[mi] - none[mi]) * (double)last / cus) + end[mi];
    return us;
}
// Row blocks per wavefront of the least estimated time for M rows, tn tile columns (times slices) and kt k tiles each: with
// few tokens (or a token count just past a multiple of 256) 256 rows are mostly rows that do not exist.  256 rows -> this
// choice, logits and dH, us, h=4096 V=64000: 64 tokens 130 -> 97 and 115 -> 97, 128: 131 -> 106 and 122 -> 105, 192: 137 -> 124 and
// 129 -> 121, 384: 239 -> 196 and 225 -> 200.  By tile_us, lower tiles must promise 15 %: the part is power limited, so a round of
// tiles that is not full lets the others run faster (N=1999 h=3072 V=50001 p=8: 11 % promised, the same time; N=700 h=4096 V=100000: 3 %
// promised, 3 % longer).
int row_blocks_for(int64_t M, int64_t tn, int64_t kt, bool stats, int cus) {
    if (!stats && M > DH_FEW) {
        int low = 4;
        for (int mi = 3; mi >= 2; --mi)
            if (dh_us(mi, ceil_div(M, 64 * mi) * tn, kt, cus) < dh_us(low, ceil_div(M, 64 * low) * tn, kt, cus)) low = mi;
        return low;
    }
    auto us = [&](int mi) { return (double)ceil_div(ceil_div(M, 64 * mi) * tn, cus) * tile_us(mi, kt, stats); };
    int best = 3;
    for (int mi = 2; mi >= 1; --mi)
        if (us(mi) < us(best)) best = mi;
    if (us(best) > 0.85 * us(4)) best = 4;
    return best;
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

unsigned long long* gemm_bf16_trace_buffer(int kernel_id, size_t& words) {
    unsigned long long* buf = g_trace_buf.load();
    const int want = g_trace_kernel.load();
    words = g_trace_words.load();
    return want < 0 || want == kernel_id ? buf : nullptr;
}

// Up to this many tokens dW takes the kernel with two workgroups per compute unit.  Large tile -> this one, us per launch:
// K = 64 (h=4096, V=128256) 497 -> 375, 200 (4096, 64000) 343 -> 287, 512 (2048, 32000) 118 -> 98, 700 (1512, 50001)
// 169 -> 153, 1024 (4096, 32000) 334 -> 320, 1999 (3072, 50001) 635 -> 634, 4096 (4096, 32000) 986 -> 1030.
constexpr int DW_TWIN_MAX_K = 1536;
static hipError_t launch_dw(const GemmBf16Group& g, hipStream_t st) {
    size_t words = 0;
    if (g.base.K > DW_TWIN_MAX_K || gemm_bf16_trace_buffer(g.base.kernel_id, words)) return launch_fast_t<false, false, Epi::StoreF32>(g, st);
    return launch_gemm_bf16_dw_twin(g, st);
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
    if (p.a_kcontig && p.b_kcontig && p.epi == Epi::FwdStats) return launch_gemm_bf16_fwd_stats(g, st);
    if (p.a_kcontig && p.b_kcontig && p.epi == Epi::DLogits) return launch_gemm_bf16_dlogits(g, st);
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
// time wins: rounds of 256 workgroups, and for S > 1 the partial outputs written and read once (4 TB/s; 5.5 where they are large) and another launch.  The products
// A_r = softmax'_r W_r of Algorithm 2 are n outputs of kt k tiles each in one launch: N=71 h=896 V=14003 p=8, step 619 -> 121 us
// (with the logits of all shards in one launch too), N=136 h=7040 V=79658 p=2 2356 -> 1369, N=4096 h=4096 V=32000 p=8 3132 -> 2947.
static int slices_of(int64_t M, int64_t N, int64_t kt, int n) {
    const int64_t tn = ceil_div(N, BN) * n;
    int best = 1;
    double best_us = 0;
    for (int64_t S = 1; S <= 32 && (S == 1 || S * 8 <= kt) && (S == 1 || S * n * M * N <= (int64_t)1 << 28); ++S) {
        const int mi = row_blocks_for(M, tn * S, ceil_div(kt, S), false, 256);
        const int64_t tiles = ceil_div(M, 64 * mi) * tn * S;
        double us = M > DH_FEW ? dh_us(mi, tiles, ceil_div(kt, S), 256) : (double)ceil_div(tiles, 256) * tile_us(mi, ceil_div(kt, S), false);
        if (S > 1) us += (double)(S * n * M * N) * 8.0 / (M > DH_FEW ? 5.5e6 : 4e6) + 5.0;
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
