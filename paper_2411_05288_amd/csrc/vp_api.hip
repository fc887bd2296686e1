// extern "C" entry points of libvp: argument validation, workspace carving and the order of
// kernel launches for each pass.  No allocation, no synchronisation, no state.
#include <mutex>

#include "vp_internal.h"

using namespace vp;

namespace {

constexpr int64_t MAX_ELEMS = (int64_t)1 << 31;

bool aligned16(const void* p) { return ((uintptr_t)p & 15u) == 0; }

bool sizes_ok(int64_t N, int64_t h, int64_t Vs) { return N >= 1 && h >= 1 && Vs >= 1; }

// Row lengths are limited to 2^20 elements: the GEMM epilogues address 256 rows of an output with 32-bit byte offsets.
constexpr int64_t MAX_ROW = (int64_t)1 << 20;

bool sizes_supported(int64_t N, int64_t h, int64_t Vs) {
    return N < MAX_ELEMS && h <= MAX_ROW && Vs <= MAX_ROW && N * Vs < MAX_ELEMS && N * h < MAX_ELEMS &&
           Vs * h < MAX_ELEMS;
}

bool dtype_ok(vp_dtype dt) { return dt == VP_F32 || dt == VP_BF16; }

int64_t fwd_tiles(int64_t Vs) { return ceil_div(Vs, GEMM_BN); }

// Row stride (elements) of the bf16 D matrix in the backward workspace: rows start on 128-byte
// boundaries, so the 128-byte row pieces the dH product fetches never straddle two cache lines
// (worth 9 % on that product when Vs * 2 is not a multiple of 128).
int64_t d_row_stride(int64_t Vs) { return (Vs + 63) / 64 * 64; }

size_t max3(size_t a, size_t b, size_t c) { return a > b ? (a > c ? a : c) : (b > c ? b : c); }

// fp32 path: bytes of K-slice scratch behind the [N, Vs] matrix at the start of the workspace
size_t f32_fwd_scratch(int64_t N, int64_t h, int64_t Vs) {
    return gemm_f32_scratch_floats(F32Product::Logits, N, Vs, h) * sizeof(float);
}
size_t f32_bwd_scratch(int64_t N, int64_t h, int64_t Vs) {
    return max3(gemm_f32_scratch_floats(F32Product::Logits, N, Vs, h), gemm_f32_scratch_floats(F32Product::DH, N, h, Vs),
                gemm_f32_scratch_floats(F32Product::DW, Vs, h, N)) *
           sizeof(float);
}
size_t f32_matrix_bytes(int64_t N, int64_t Vs) { return align_up((size_t)N * Vs * sizeof(float), 256); }

// One shard as a list for the kernels that take several.
ShardList one_shard(int64_t Vs, int64_t off, const void* Y = nullptr) {
    ShardList l{};
    l.n = 1;
    l.rows[0] = (int)Vs;
    l.first[1] = (int)fwd_tiles(Vs);
    l.offset[0] = off;
    l.ldd[0] = d_row_stride(Vs);
    l.Y[0] = Y;
    l.ldy[0] = Vs;
    return l;
}

// The shards of a group call are taken in parts of at most GEMM_GROUP_MAX shards whose D matrices (all kept until the
// part's dH and dW products are done) take at most this much workspace together, or of one shard.
constexpr size_t GROUP_D_BYTES = (size_t)4 << 30;
// fp32: a part whose dH slices would take more scratch than this goes shard by shard.
constexpr size_t GROUP_SLICE_BYTES = (size_t)1 << 30;

int64_t d_ld(int64_t Vs, vp_dtype dt) { return dt == VP_BF16 ? d_row_stride(Vs) : (Vs + 3) / 4 * 4; }
size_t d_bytes(int64_t N, int64_t Vs, vp_dtype dt) { return align_up((size_t)N * d_ld(Vs, dt) * (dt == VP_BF16 ? 2 : 4), 256); }

// Shards of the part that begins at shard r0.
int part_shards(const int64_t* rows, int p, int r0, int64_t N, vp_dtype dt) {
    size_t b = d_bytes(N, rows[r0], dt);
    int n = 1;
    while (r0 + n < p && n < GEMM_GROUP_MAX && b + d_bytes(N, rows[r0 + n], dt) <= GROUP_D_BYTES)
        b += d_bytes(N, rows[r0 + n++], dt);
    return n;
}

struct PartSizes {
    size_t d, slices, stats;     // bytes: D matrices, K-slice partials of dH, statistics partials of the bf16 forward pass
    int64_t tiles;               // bf16: column tiles of the forward pass
    int S;                       // K slices of dH: bf16 over all shards, fp32 per shard
    int S_logits, S_dw;          // fp32: K slices of the logits and of dW
    size_t logits_slices, dw_slices;     // fp32: bytes of their partials
};
PartSizes part_sizes(const int64_t* rows, int r0, int n, int64_t N, int64_t h, vp_dtype dt) {
    PartSizes z{};
    int64_t kt = 0, longest = 0;
    size_t dw = 0;
    for (int r = r0; r < r0 + n; ++r) {
        z.d += d_bytes(N, rows[r], dt);
        dw += align_up((size_t)rows[r] * h * sizeof(float), 256);
        z.tiles += fwd_tiles(rows[r]);
        kt += ceil_div(rows[r], 64);
        longest = rows[r] > longest ? rows[r] : longest;
    }
    if (dt == VP_BF16) {
        z.S = h % 8 == 0 ? gemm_bf16_slices(N, h, kt) : 1;
        z.slices = z.S > 1 ? (size_t)z.S * N * h * sizeof(float) : 0;
        z.stats = align_up((size_t)(2 * z.tiles + n) * N * sizeof(float), 256);
    } else {
        z.S = gemm_f32_dh_slices(N, h, longest, n);
        z.slices = z.S * n > 1 ? (size_t)z.S * n * N * h * sizeof(float) : 0;
        z.S_logits = gemm_f32_group_slices(ceil_div(N, 64) * kt, h);
        z.S_dw = gemm_f32_group_slices(ceil_div(h, 64) * kt, N);
        z.logits_slices = z.S_logits > 1 ? z.S_logits * z.d : 0;
        z.dw_slices = z.S_dw > 1 ? z.S_dw * dw : 0;
    }
    return z;
}
// K slices of each product A_r = softmax'_r W_r of a group.
int each_slices(const int64_t* rows, int p, int64_t N, int64_t h, vp_dtype dt) {
    int64_t longest = 0;
    for (int r = 0; r < p; ++r) longest = rows[r] > longest ? rows[r] : longest;
    if (dt == VP_F32) return gemm_f32_each_slices(N, h, longest, p);
    return h % 8 == 0 ? gemm_bf16_slices_each(N, h, ceil_div(longest, 64), p) : 1;
}
// Whether a part of the fp32 path is computed as a group (a single shard has K slices in every product: launch_gemm_f32).
bool f32_grouped(int n, const PartSizes& z, int64_t N) { return n > 1 && N <= MAX_ROW && z.slices <= GROUP_SLICE_BYTES; }

GemmBf16Params logits_product(const void* H, const int64_t* labels, int64_t N, int64_t h, Epi epi) {
    GemmBf16Params g{};
    g.A = (const u16*)H;
    g.M = (int)N; g.K = (int)h;
    g.lda = (int)h; g.ldb = (int)h;
    g.a_kcontig = 1; g.b_kcontig = 1;
    g.vec_ok = (h % 8 == 0) ? 1 : 0;
    g.epi = epi;
    g.labels = labels;
    g.kernel_id = epi == Epi::FwdStats ? K_GEMM_FWD_STATS : K_GEMM_DLOGITS;
    return g;
}

vp_status dev(hipError_t e) { return e == hipSuccess ? VP_OK : VP_ERR_DEVICE; }

// Scratch of vp_output_fwd_noalloc: device memory that belongs to the library's code object, so the
// entry point has nothing to allocate.  Every GPU the library runs on holds its own copy until the
// process ends.  In host code the array's name is only a handle: its device address is looked up
// once per device (with that device current) and that address is what the kernels are given.
constexpr size_t NOALLOC_SCRATCH_BYTES = (size_t)4 << 20;
constexpr int NOALLOC_MAX_DEVICES = 64;
static __device__ __align__(256) unsigned char scratch[NOALLOC_SCRATCH_BYTES];
std::mutex g_scratch_mu;
void* g_scratch_ptr[NOALLOC_MAX_DEVICES] = {nullptr};

// Device address of `scratch` on the current device, nullptr if the runtime refuses.
void* scratch_of_current_device() {
    int d = -1;
    if (hipGetDevice(&d) != hipSuccess || d < 0 || d >= NOALLOC_MAX_DEVICES) return nullptr;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[d]) {
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess) return nullptr;
        g_scratch_ptr[d] = ptr;
    }
    return g_scratch_ptr[d];
}

}  // namespace

extern "C" {

int vp_version(void) { return 100; }

const char* vp_status_string(vp_status s) {
    switch (s) {
        case VP_OK: return "VP_OK";
        case VP_ERR_INVALID_ARG: return "VP_ERR_INVALID_ARG";
        case VP_ERR_UNSUPPORTED: return "VP_ERR_UNSUPPORTED";
        case VP_ERR_WORKSPACE: return "VP_ERR_WORKSPACE";
        case VP_ERR_DEVICE: return "VP_ERR_DEVICE";
    }
    return "VP_ERR_UNKNOWN";
}

size_t vp_workspace_bytes(vp_call which, int64_t N, int64_t h, int64_t Vs, vp_dtype dt, uint32_t flags) {
    const uint32_t allowed =
        which == VP_CALL_OUTPUT_BWD ? (uint32_t)(VP_SAVE_LOGITS | VP_SKIP_DH | VP_DH_OVERWRITE) : (uint32_t)VP_SAVE_LOGITS;
    if (!dtype_ok(dt) || (flags & ~allowed)) return (size_t)-1;
    switch (which) {
        case VP_CALL_OUTPUT_FWD_ALG2:
            // the statistics partials of the forward pass, then the softmax' operand of A = softmax' W
            if (!sizes_ok(N, h, Vs) || !sizes_supported(N, h, Vs)) return (size_t)-1;
            if (dt == VP_BF16) {
                if (N * d_row_stride(Vs) >= MAX_ELEMS) return (size_t)-1;
                return align_up((size_t)(2 * fwd_tiles(Vs) + 1) * N * sizeof(float), 256) +
                       align_up((size_t)N * d_row_stride(Vs) * 2, 256);
            }
            return f32_matrix_bytes(N, Vs) + align_up(f32_bwd_scratch(N, h, Vs), 256);
        case VP_CALL_OUTPUT_DX_ALG2:
            return 0;
        case VP_CALL_OUTPUT_FWD:
            if (!sizes_ok(N, h, Vs) || !sizes_supported(N, h, Vs)) return (size_t)-1;
            if (dt == VP_BF16) return align_up((size_t)(2 * fwd_tiles(Vs) + 1) * N * sizeof(float), 256);
            // fp32: the logits live in the workspace unless the caller keeps them; then K-slice scratch
            return ((flags & VP_SAVE_LOGITS) ? 0 : f32_matrix_bytes(N, Vs)) + align_up(f32_fwd_scratch(N, h, Vs), 256);
        case VP_CALL_OUTPUT_BWD:
            if (!sizes_ok(N, h, Vs) || !sizes_supported(N, h, Vs)) return (size_t)-1;
            if (dt == VP_BF16) {
                if (N * d_row_stride(Vs) >= MAX_ELEMS) return (size_t)-1;
                return align_up((size_t)N * d_row_stride(Vs) * 2, 256);
            }
            return f32_matrix_bytes(N, Vs) + align_up(f32_bwd_scratch(N, h, Vs), 256);
        case VP_CALL_EMBED_BWD:
            if (N < 1 || N > ((int64_t)1 << 24)) return (size_t)-1;
            return align_up(embed_bwd_workspace(N, h, Vs, dt == VP_BF16 ? 2 : 4), 256);
        case VP_CALL_COMBINE_STATS:
        case VP_CALL_EMBED_FWD:
            return 0;
    }
    return (size_t)-1;
}

vp_status vp_output_fwd(const void* H, const void* W_shard, const int64_t* labels, int64_t N, int64_t h, int64_t Vs,
                        int64_t shard_offset, vp_dtype dt, uint32_t flags, float* local_max, float* local_sumexp,
                        float* local_target, void* logits_out, void* workspace, size_t workspace_bytes, void* stream) {
    if (!H || !W_shard || !labels || !local_max || !local_sumexp || !local_target) return VP_ERR_INVALID_ARG;
    if (!sizes_ok(N, h, Vs) || !dtype_ok(dt) || shard_offset < 0) return VP_ERR_INVALID_ARG;
    if (flags & ~(uint32_t)VP_SAVE_LOGITS) return VP_ERR_INVALID_ARG;
    if (((flags & VP_SAVE_LOGITS) != 0) != (logits_out != nullptr)) return VP_ERR_INVALID_ARG;
    if (!aligned16(H) || !aligned16(W_shard) || !aligned16(logits_out) || !aligned16(workspace))
        return VP_ERR_INVALID_ARG;
    if (!sizes_supported(N, h, Vs)) return VP_ERR_UNSUPPORTED;
    const size_t need = vp_workspace_bytes(VP_CALL_OUTPUT_FWD, N, h, Vs, dt, flags);
    if (need > 0 && (!workspace || workspace_bytes < need)) return VP_ERR_WORKSPACE;
    hipStream_t st = (hipStream_t)stream;

    if (dt == VP_BF16) {
        const int64_t tiles = fwd_tiles(Vs);
        float* pm = (float*)workspace;
        float* ps = pm + tiles * N;
        float* pt = ps + tiles * N;
        GemmBf16Params g{};
        g.A = (const u16*)H; g.B = (const u16*)W_shard;
        g.M = (int)N; g.N = (int)Vs; g.K = (int)h;
        g.lda = (int)h; g.ldb = (int)h;
        g.a_kcontig = 1; g.b_kcontig = 1;
        g.vec_ok = (h % 8 == 0) ? 1 : 0;
        g.epi = Epi::FwdStats;
        g.Y = (u16*)logits_out; g.ldy = (int)Vs;
        g.labels = labels; g.shard_offset = shard_offset;
        g.part_max = pm; g.part_sum = ps; g.part_tgt = pt;
        hipError_t e = launch_gemm_bf16(g, st);
        if (e != hipSuccess) return VP_ERR_DEVICE;
        return dev(launch_fold_partials(pm, ps, pt, one_shard(Vs, shard_offset), (int)N, labels, local_max, local_sumexp,
                                        local_target, st));
    }
    float* Y = logits_out ? (float*)logits_out : (float*)workspace;
    float* scratch = f32_fwd_scratch(N, h, Vs) ? (float*)((char*)workspace + (logits_out ? 0 : f32_matrix_bytes(N, Vs)))
                                               : nullptr;
    hipError_t e = launch_gemm_f32(F32Product::Logits, (const float*)H, h, (const float*)W_shard, h, Y, (int)N, (int)Vs, (int)h,
                                   false, scratch, st);
    if (e != hipSuccess) return VP_ERR_DEVICE;
    return dev(launch_row_stats_f32(one_shard(Vs, shard_offset, Y), labels, (int)N, local_max, local_sumexp, local_target, st));
}

size_t vp_output_fwd_noalloc_max_scratch(void) { return NOALLOC_SCRATCH_BYTES; }

vp_status vp_output_fwd_noalloc(const void* H, const void* W_shard, const int64_t* labels, int64_t N, int64_t h,
                                int64_t Vs, int64_t shard_offset, vp_dtype dt, uint32_t flags, float* local_max,
                                float* local_sumexp, float* local_target, void* logits_out, void* stream) {
    // sizes first: a request whose scratch does not fit the static array is refused before anything else
    if (!sizes_ok(N, h, Vs) || !dtype_ok(dt)) return VP_ERR_INVALID_ARG;
    if (flags & ~(uint32_t)VP_SAVE_LOGITS) return VP_ERR_INVALID_ARG;
    if (!sizes_supported(N, h, Vs)) return VP_ERR_UNSUPPORTED;
    const size_t need = vp_workspace_bytes(VP_CALL_OUTPUT_FWD, N, h, Vs, dt, flags);
    if (need == (size_t)-1 || need > NOALLOC_SCRATCH_BYTES) return VP_ERR_UNSUPPORTED;
    void* ws = scratch_of_current_device();
    if (!ws) return VP_ERR_DEVICE;
    // nothing in the scratch has to start at zero: every partial the fold reads is written by this call's
    // GEMM first (the target partial only for rows whose label the shard owns, and only those are read)
    return vp_output_fwd(H, W_shard, labels, N, h, Vs, shard_offset, dt, flags, local_max, local_sumexp, local_target,
                         logits_out, ws, NOALLOC_SCRATCH_BYTES, stream);
}

vp_status vp_combine_stats(const float* local_max, const float* local_sumexp, const float* local_target, int32_t p,
                           int64_t N, float* global_max, float* global_sumexp, float* loss_per_row, float* loss_mean,
                           void* stream) {
    if (!local_max || !local_sumexp || !local_target || !global_max || !global_sumexp || !loss_mean)
        return VP_ERR_INVALID_ARG;
    if (p < 1 || N < 1) return VP_ERR_INVALID_ARG;
    if (N >= MAX_ELEMS || (int64_t)p * N >= MAX_ELEMS) return VP_ERR_UNSUPPORTED;
    return dev(launch_combine(local_max, local_sumexp, local_target, p, (int)N, global_max, global_sumexp,
                              loss_per_row, loss_mean, (hipStream_t)stream));
}

int64_t vp_dlogits_row_stride(int64_t Vs, vp_dtype dt) {
    if (Vs < 1 || !dtype_ok(dt)) return -1;
    return dt == VP_BF16 ? d_row_stride(Vs) : Vs;
}

vp_status vp_output_bwd(const void* H, const void* W_shard, const int64_t* labels, int64_t N, int64_t h, int64_t Vs,
                        int64_t shard_offset, vp_dtype dt, uint32_t flags, const float* global_max,
                        const float* global_sumexp, const void* logits_saved, float grad_scale, float* dH_accum,
                        float* dW_shard, void* workspace, size_t workspace_bytes, void* stream) {
    if (!H || !W_shard || !labels || !global_max || !global_sumexp || !dW_shard) return VP_ERR_INVALID_ARG;
    if (!dH_accum && !(flags & VP_SKIP_DH)) return VP_ERR_INVALID_ARG;
    if (!sizes_ok(N, h, Vs) || !dtype_ok(dt) || shard_offset < 0) return VP_ERR_INVALID_ARG;
    if (flags & ~(uint32_t)(VP_SAVE_LOGITS | VP_SKIP_DH | VP_DH_OVERWRITE)) return VP_ERR_INVALID_ARG;
    if ((flags & VP_SKIP_DH) && (flags & VP_DH_OVERWRITE)) return VP_ERR_INVALID_ARG;
    if (((flags & VP_SAVE_LOGITS) != 0) != (logits_saved != nullptr)) return VP_ERR_INVALID_ARG;
    if (!aligned16(H) || !aligned16(W_shard) || !aligned16(logits_saved) || !aligned16(workspace) ||
        !aligned16(dH_accum) || !aligned16(dW_shard))
        return VP_ERR_INVALID_ARG;
    const bool skip_dh = (flags & VP_SKIP_DH) != 0;
    const bool dh_overwrite = (flags & VP_DH_OVERWRITE) != 0;
    if (!sizes_supported(N, h, Vs)) return VP_ERR_UNSUPPORTED;
    const size_t need = vp_workspace_bytes(VP_CALL_OUTPUT_BWD, N, h, Vs, dt, flags);
    if (need == (size_t)-1) return VP_ERR_UNSUPPORTED;
    if (!workspace || workspace_bytes < need) return VP_ERR_WORKSPACE;
    hipStream_t st = (hipStream_t)stream;
    hipError_t e;

    if (dt == VP_BF16) {
        u16* D = (u16*)workspace;
        const int64_t ldd = d_row_stride(Vs);
        const int vec_ok = (h % 8 == 0) ? 1 : 0;
        if (logits_saved) {
            e = launch_dlogits(logits_saved, Vs, D, ldd, 1, labels, shard_offset, global_max, global_sumexp, grad_scale,
                               (int)N, (int)Vs, st);
        } else {
            GemmBf16Params g{};
            g.A = (const u16*)H; g.B = (const u16*)W_shard;
            g.M = (int)N; g.N = (int)Vs; g.K = (int)h;
            g.lda = (int)h; g.ldb = (int)h;
            g.a_kcontig = 1; g.b_kcontig = 1;
            g.vec_ok = (h % 8 == 0) ? 1 : 0;
            g.epi = Epi::DLogits;
            g.Y = D; g.ldy = (int)ldd;
            g.labels = labels; g.shard_offset = shard_offset;
            g.gmax = global_max; g.gsum = global_sumexp; g.scale = grad_scale;
            e = launch_gemm_bf16(g, st);
            if (e == hipSuccess) {
                ShardList l = one_shard(Vs, shard_offset);
                l.D[0] = D;
                e = launch_zero_pad_columns(l, (int)N, st);
            }
        }
        if (e != hipSuccess) return VP_ERR_DEVICE;
        if (!skip_dh) {   // dH += D W_shard : M = N tokens, N = h, K = Vs; W_shard is stored [K][N]
            GemmBf16Params g{};
            g.A = D; g.B = (const u16*)W_shard;
            g.M = (int)N; g.N = (int)h; g.K = (int)Vs;
            g.lda = (int)ldd; g.ldb = (int)h;
            g.a_kcontig = 1; g.b_kcontig = 0;
            g.vec_ok = vec_ok;
            g.epi = dh_overwrite ? Epi::StoreF32 : Epi::AccumF32;
            g.kernel_id = K_GEMM_DH;
            g.C = dH_accum; g.ldc = (int)h;
            e = launch_gemm_bf16(g, st);
            if (e != hipSuccess) return VP_ERR_DEVICE;
        }
        {   // dW = D^T H : M = Vs, N = h, K = N tokens; D is stored [K][M], H is stored [K][N]
            GemmBf16Params g{};
            g.A = D; g.B = (const u16*)H;
            g.M = (int)Vs; g.N = (int)h; g.K = (int)N;
            g.lda = (int)ldd; g.ldb = (int)h;
            g.a_kcontig = 0; g.b_kcontig = 0;
            g.vec_ok = vec_ok;
            g.epi = Epi::StoreF32;
            g.C = dW_shard; g.ldc = (int)h;
            e = launch_gemm_bf16(g, st);
        }
        return dev(e);
    }

    // fp32: every step in fp32
    float* D = (float*)workspace;
    float* scratch = f32_bwd_scratch(N, h, Vs) ? (float*)((char*)workspace + f32_matrix_bytes(N, Vs)) : nullptr;
    const float* Y = (const float*)logits_saved;
    if (!Y) {
        e = launch_gemm_f32(F32Product::Logits, (const float*)H, h, (const float*)W_shard, h, D, (int)N, (int)Vs, (int)h, false,
                            scratch, st);
        if (e != hipSuccess) return VP_ERR_DEVICE;
        Y = D;   // D is formed in place
    }
    e = launch_dlogits(Y, Vs, D, Vs, 0, labels, shard_offset, global_max, global_sumexp, grad_scale, (int)N, (int)Vs, st);
    if (e != hipSuccess) return VP_ERR_DEVICE;
    if (!skip_dh) {
        e = launch_gemm_f32(F32Product::DH, D, Vs, (const float*)W_shard, h, dH_accum, (int)N, (int)h, (int)Vs, !dh_overwrite,
                            scratch, st);
        if (e != hipSuccess) return VP_ERR_DEVICE;
    }
    e = launch_gemm_f32(F32Product::DW, D, Vs, (const float*)H, h, dW_shard, (int)Vs, (int)h, (int)N, false, scratch, st);
    return dev(e);
}

// ---- several shards on this device

size_t vp_output_group_workspace_bytes(vp_call which, int32_t p, int64_t N, int64_t h, const int64_t* rows, vp_dtype dt,
                                       uint32_t flags) {
    const bool alg2 = which == VP_CALL_OUTPUT_FWD_ALG2;
    if ((which != VP_CALL_OUTPUT_FWD && which != VP_CALL_OUTPUT_BWD && !alg2) || p < 1 || !rows) return (size_t)-1;
    size_t need = 0;
    for (int32_t r = 0; r < p; ++r) {       // what the shards need one by one (paths that are not grouped)
        const size_t b = vp_workspace_bytes(which, N, h, rows[r], dt, flags);
        if (b == (size_t)-1) return b;
        need = b > need ? b : need;
    }
    if (alg2) {      // one part: its softmax' matrices stay until A = softmax' W is done
        if (part_shards(rows, p, 0, N, dt) < p) return (size_t)-1;
        const PartSizes z = part_sizes(rows, 0, p, N, h, dt);
        const int S = each_slices(rows, p, N, h, dt);
        const size_t slices = S > 1 ? (size_t)S * p * N * h * sizeof(float) : 0;
        const size_t b = (dt == VP_BF16 ? z.stats : 0) + z.d + max3(align_up(slices, 256), z.logits_slices, 0);
        return b > need ? b : need;
    }
    if (dt == VP_BF16 && h % 8) return need;
    for (int r = 0; r < p;) {
        const int n = part_shards(rows, p, r, N, dt);
        const PartSizes z = part_sizes(rows, r, n, N, h, dt);
        // the slices' partials of one product at a time
        const size_t logits = which == VP_CALL_OUTPUT_BWD && (flags & VP_SAVE_LOGITS) ? 0 : z.logits_slices;
        size_t b = z.d + max3((flags & VP_SKIP_DH) ? 0 : align_up(z.slices, 256), logits, z.dw_slices);
        if (dt == VP_F32 && !f32_grouped(n, z, N)) b = 0;
        else if (which == VP_CALL_OUTPUT_FWD) b = dt == VP_BF16 ? z.stats : ((flags & VP_SAVE_LOGITS) ? 0 : z.d) + logits;
        need = b > need ? b : need;
        r += n;
    }
    return need;
}

vp_status vp_output_fwd_group(const void* H, const void* const* W_shards, const int64_t* rows, const int64_t* shard_offsets,
                              int32_t p, const int64_t* labels, int64_t N, int64_t h, vp_dtype dt, uint32_t flags,
                              float* local_max, float* local_sumexp, float* local_target, void* const* logits_out,
                              void* workspace, size_t workspace_bytes, void* stream) {
    if (!H || !W_shards || !rows || !shard_offsets || p < 1 || !labels || !local_max || !local_sumexp || !local_target)
        return VP_ERR_INVALID_ARG;
    if (!dtype_ok(dt) || (flags & ~(uint32_t)VP_SAVE_LOGITS)) return VP_ERR_INVALID_ARG;
    if (((flags & VP_SAVE_LOGITS) != 0) != (logits_out != nullptr)) return VP_ERR_INVALID_ARG;
    if (!aligned16(H) || !aligned16(workspace)) return VP_ERR_INVALID_ARG;
    for (int32_t r = 0; r < p; ++r) {
        if (!W_shards[r] || !aligned16(W_shards[r]) || !sizes_ok(N, h, rows[r]) || shard_offsets[r] < 0) return VP_ERR_INVALID_ARG;
        if (logits_out && (!logits_out[r] || !aligned16(logits_out[r]))) return VP_ERR_INVALID_ARG;
        if (!sizes_supported(N, h, rows[r])) return VP_ERR_UNSUPPORTED;
    }
    const size_t need = vp_output_group_workspace_bytes(VP_CALL_OUTPUT_FWD, p, N, h, rows, dt, flags);
    if (need == (size_t)-1) return VP_ERR_UNSUPPORTED;
    if (need > 0 && (!workspace || workspace_bytes < need)) return VP_ERR_WORKSPACE;
    hipStream_t st = (hipStream_t)stream;
    for (int r0 = 0; r0 < p;) {
        const int n = part_shards(rows, p, r0, N, dt);
        const PartSizes z = part_sizes(rows, r0, n, N, h, dt);
        if (dt == VP_F32 && f32_grouped(n, z, N)) {
            GemmF32Shard sh[GEMM_GROUP_MAX];
            ShardList l{};
            l.n = n;
            char* d = (char*)workspace;
            for (int k = 0; k < n; ++k) {
                const int r = r0 + k;
                const int ld = (int)(logits_out ? rows[r] : d_ld(rows[r], dt));
                float* Y = logits_out ? (float*)logits_out[r] : (float*)d;
                sh[k] = {nullptr, (const float*)W_shards[r], Y, (int)rows[r], ld};
                l.rows[k] = (int)rows[r];
                l.ldy[k] = ld;
                l.offset[k] = shard_offsets[r];
                l.Y[k] = Y;
                d += logits_out ? 0 : d_bytes(N, rows[r], dt);
            }
            if (launch_gemm_f32_logits((const float*)H, N, h, sh, n, z.S_logits, (float*)d, st) != hipSuccess ||
                launch_row_stats_f32(l, labels, (int)N, local_max + r0 * N, local_sumexp + r0 * N, local_target + r0 * N, st) !=
                    hipSuccess)
                return VP_ERR_DEVICE;
            r0 += n;
            continue;
        }
        if (dt == VP_BF16 && n > 1) {
            float* pm = (float*)workspace;
            GemmBf16Group g{};
            ShardList l{};
            g.base = logits_product(H, labels, N, h, Epi::FwdStats);
            g.base.part_max = pm;
            g.base.part_sum = pm + z.tiles * N;
            g.base.part_tgt = pm + 2 * z.tiles * N;
            l.n = n;
            for (int k = 0; k < n; ++k) {
                const int r = r0 + k;
                g.sh[k].B = (const u16*)W_shards[r];
                g.sh[k].out = logits_out ? logits_out[r] : nullptr;
                g.sh[k].ld = g.sh[k].rows = l.rows[k] = (int)rows[r];
                g.sh[k].offset = l.offset[k] = shard_offsets[r];
                l.first[k + 1] = l.first[k] + (int)fwd_tiles(rows[r]);
            }
            gemm_bf16_group_finish(g, n);
            if (gemm_bf16_group_ok(g)) {
                if (launch_gemm_bf16_group(g, st) != hipSuccess ||
                    launch_fold_partials(g.base.part_max, g.base.part_sum, g.base.part_tgt, l, (int)N, labels,
                                         local_max + r0 * N, local_sumexp + r0 * N, local_target + r0 * N, st) != hipSuccess)
                    return VP_ERR_DEVICE;
                r0 += n;
                continue;
            }
        }
        for (int r = r0; r < r0 + n; ++r) {
            const vp_status s = vp_output_fwd(H, W_shards[r], labels, N, h, rows[r], shard_offsets[r], dt, flags,
                                              local_max + r * N, local_sumexp + r * N, local_target + r * N,
                                              logits_out ? logits_out[r] : nullptr, workspace, workspace_bytes, stream);
            if (s != VP_OK) return s;
        }
        r0 += n;
    }
    return VP_OK;
}

vp_status vp_output_bwd_group(const void* H, const void* const* W_shards, const int64_t* rows, const int64_t* shard_offsets,
                              int32_t p, const int64_t* labels, int64_t N, int64_t h, vp_dtype dt, uint32_t flags,
                              const float* global_max, const float* global_sumexp, const void* const* logits_saved,
                              float grad_scale, float* dH_accum, float* const* dW_shards, void* workspace,
                              size_t workspace_bytes, void* stream) {
    if (!H || !W_shards || !rows || !shard_offsets || p < 1 || !labels || !global_max || !global_sumexp || !dW_shards)
        return VP_ERR_INVALID_ARG;
    if (!dH_accum && !(flags & VP_SKIP_DH)) return VP_ERR_INVALID_ARG;
    if (!dtype_ok(dt) || (flags & ~(uint32_t)(VP_SAVE_LOGITS | VP_SKIP_DH | VP_DH_OVERWRITE))) return VP_ERR_INVALID_ARG;
    if ((flags & VP_SKIP_DH) && (flags & VP_DH_OVERWRITE)) return VP_ERR_INVALID_ARG;
    if (((flags & VP_SAVE_LOGITS) != 0) != (logits_saved != nullptr)) return VP_ERR_INVALID_ARG;
    if (!aligned16(H) || !aligned16(workspace) || !aligned16(dH_accum)) return VP_ERR_INVALID_ARG;
    for (int32_t r = 0; r < p; ++r) {
        if (!W_shards[r] || !aligned16(W_shards[r]) || !dW_shards[r] || !aligned16(dW_shards[r]) || !sizes_ok(N, h, rows[r]) ||
            shard_offsets[r] < 0)
            return VP_ERR_INVALID_ARG;
        if (logits_saved && (!logits_saved[r] || !aligned16(logits_saved[r]))) return VP_ERR_INVALID_ARG;
        if (!sizes_supported(N, h, rows[r])) return VP_ERR_UNSUPPORTED;
    }
    const size_t need = vp_output_group_workspace_bytes(VP_CALL_OUTPUT_BWD, p, N, h, rows, dt, flags);
    if (need == (size_t)-1) return VP_ERR_UNSUPPORTED;
    if (!workspace || workspace_bytes < need) return VP_ERR_WORKSPACE;
    hipStream_t st = (hipStream_t)stream;
    const bool skip_dh = (flags & VP_SKIP_DH) != 0;
    for (int r0 = 0; r0 < p;) {
        const bool overwrite = (flags & VP_DH_OVERWRITE) != 0 && r0 == 0;
        const int n = part_shards(rows, p, r0, N, dt);
        const PartSizes z = part_sizes(rows, r0, n, N, h, dt);
        if (dt == VP_F32 && f32_grouped(n, z, N)) {
            GemmF32Shard y[GEMM_GROUP_MAX], g[GEMM_GROUP_MAX];     // logits again; dH and dW
            ShardList l{};
            l.n = n;
            char* d = (char*)workspace;
            float* slices = (float*)(d + z.d);
            for (int k = 0; k < n; ++k) {
                const int r = r0 + k;
                const int ld = (int)d_ld(rows[r], dt);
                y[k] = {nullptr, (const float*)W_shards[r], (float*)d, (int)rows[r], ld};
                g[k] = {(const float*)d, (const float*)W_shards[r], dW_shards[r], (int)rows[r], ld};
                l.rows[k] = (int)rows[r];
                l.offset[k] = shard_offsets[r];
                l.Y[k] = logits_saved ? logits_saved[r] : d;       // (D is formed in place where the logits are formed again)
                l.ldy[k] = logits_saved ? rows[r] : ld;
                l.D[k] = d;
                l.ldd[k] = ld;
                d += d_bytes(N, rows[r], dt);
            }
            hipError_t e = logits_saved ? hipSuccess : launch_gemm_f32_logits((const float*)H, N, h, y, n, z.S_logits, slices, st);
            if (e == hipSuccess) e = launch_dlogits_group(l, 0, labels, global_max, global_sumexp, 0, grad_scale, (int)N, st);
            if (e == hipSuccess)
                e = skip_dh ? launch_gemm_f32_dw((const float*)H, N, h, g, n, z.S_dw, slices, st)
                            : launch_gemm_f32_dh_dw((const float*)H, N, h, g, n, z.S, z.S_dw, dH_accum, !overwrite, slices, st);
            if (e != hipSuccess) return VP_ERR_DEVICE;
            r0 += n;
            continue;
        }
        if (dt == VP_BF16 && h % 8 == 0) {
            GemmBf16Group y{}, gh{}, gw{};      // logits again, dH, dW
            ShardList l{};
            y.base = logits_product(H, labels, N, h, Epi::DLogits);
            y.base.gmax = global_max; y.base.gsum = global_sumexp; y.base.scale = grad_scale;
            float* slices = (float*)((char*)workspace + z.d);
            gh.base.M = (int)N; gh.base.N = (int)h;
            gh.base.ldb = (int)h;
            gh.base.a_kcontig = 1; gh.base.b_kcontig = 0;
            gh.base.vec_ok = 1;
            gh.base.epi = (z.S > 1 || overwrite) ? Epi::StoreF32 : Epi::AccumF32;
            gh.base.kernel_id = K_GEMM_DH;
            gh.base.C = z.S > 1 ? slices : dH_accum; gh.base.ldc = (int)h;
            gh.slices = z.S;
            gw.base.B = (const u16*)H;
            gw.base.N = (int)h; gw.base.K = (int)N;
            gw.base.ldb = (int)h;
            gw.base.a_kcontig = 0; gw.base.b_kcontig = 0;
            gw.base.vec_ok = 1;
            gw.base.epi = Epi::StoreF32;
            gw.base.kernel_id = K_GEMM_DW;
            gw.base.ldc = (int)h;
            l.n = n;
            char* d = (char*)workspace;
            for (int k = 0; k < n; ++k) {
                const int r = r0 + k;
                const int ldd = (int)d_row_stride(rows[r]);
                y.sh[k].B = gh.sh[k].B = (const u16*)W_shards[r];
                y.sh[k].out = d;
                gh.sh[k].A = gw.sh[k].A = (const u16*)d;
                gw.sh[k].out = dW_shards[r];
                y.sh[k].ld = gh.sh[k].ld = gw.sh[k].ld = ldd;
                y.sh[k].rows = gh.sh[k].rows = gw.sh[k].rows = l.rows[k] = (int)rows[r];
                y.sh[k].offset = l.offset[k] = shard_offsets[r];
                l.ldd[k] = ldd;
                l.ldy[k] = rows[r];
                l.Y[k] = logits_saved ? logits_saved[r] : nullptr;
                l.D[k] = d;
                d += d_bytes(N, rows[r], dt);
            }
            gemm_bf16_group_finish(y, n);
            gemm_bf16_group_finish(gh, n);
            gemm_bf16_group_finish(gw, n);
            if ((n > 1 || z.S > 1) && N <= MAX_ROW && (logits_saved || gemm_bf16_group_ok(y)) &&
                (skip_dh || gemm_bf16_group_ok(gh)) && gemm_bf16_group_ok(gw)) {
                hipError_t e;
                if (logits_saved) {
                    e = launch_dlogits_group(l, 1, labels, global_max, global_sumexp, 0, grad_scale, (int)N, st);
                } else {
                    e = launch_gemm_bf16_group(y, st);
                    if (e == hipSuccess) e = launch_zero_pad_columns(l, (int)N, st);
                }
                if (e == hipSuccess && !skip_dh) {
                    e = launch_gemm_bf16_group(gh, st);
                    if (e == hipSuccess && z.S > 1) {
                        ProfScope prof(K_SUM_SLICES, st);
                        e = launch_sum_slices(slices, z.S, N * h, dH_accum, !overwrite, st);
                    }
                }
                if (e == hipSuccess) e = launch_gemm_bf16_group(gw, st);
                if (e != hipSuccess) return VP_ERR_DEVICE;
                r0 += n;
                continue;
            }
        }
        for (int r = r0; r < r0 + n; ++r) {
            const uint32_t f = (flags & ~(uint32_t)VP_DH_OVERWRITE) | (r == r0 && overwrite ? (uint32_t)VP_DH_OVERWRITE : 0u);
            const vp_status s = vp_output_bwd(H, W_shards[r], labels, N, h, rows[r], shard_offsets[r], dt, f, global_max,
                                              global_sumexp, logits_saved ? logits_saved[r] : nullptr, grad_scale, dH_accum,
                                              dW_shards[r], workspace, workspace_bytes, stream);
            if (s != VP_OK) return s;
        }
        r0 += n;
    }
    return VP_OK;
}

vp_status vp_output_fwd_alg2(const void* H, const void* W_shard, const int64_t* labels, int64_t N, int64_t h,
                             int64_t Vs, int64_t shard_offset, vp_dtype dt, uint32_t flags, float* local_max,
                             float* local_sumexp, float* local_target, void* logits_out, float* A_out, void* B_out,
                             void* workspace, size_t workspace_bytes, void* stream) {
    if (!H || !W_shard || !labels || !local_max || !local_sumexp || !local_target || !A_out || !B_out)
        return VP_ERR_INVALID_ARG;
    if (!sizes_ok(N, h, Vs) || !dtype_ok(dt) || shard_offset < 0) return VP_ERR_INVALID_ARG;
    if (flags & ~(uint32_t)VP_SAVE_LOGITS) return VP_ERR_INVALID_ARG;
    if (((flags & VP_SAVE_LOGITS) != 0) != (logits_out != nullptr)) return VP_ERR_INVALID_ARG;
    if (!aligned16(H) || !aligned16(W_shard) || !aligned16(logits_out) || !aligned16(workspace) ||
        !aligned16(A_out) || !aligned16(B_out))
        return VP_ERR_INVALID_ARG;
    if (!sizes_supported(N, h, Vs)) return VP_ERR_UNSUPPORTED;
    const size_t need = vp_workspace_bytes(VP_CALL_OUTPUT_FWD_ALG2, N, h, Vs, dt, flags);
    if (need == (size_t)-1) return VP_ERR_UNSUPPORTED;
    if (!workspace || workspace_bytes < need) return VP_ERR_WORKSPACE;
    hipStream_t st = (hipStream_t)stream;
    hipError_t e;

    if (dt == VP_BF16) {
        const int64_t tiles = fwd_tiles(Vs);
        const int64_t ldd = d_row_stride(Vs);
        float* pm = (float*)workspace;
        float* ps = pm + tiles * N;
        float* pt = ps + tiles * N;
        u16* P = (u16*)((char*)workspace + align_up((size_t)(2 * tiles + 1) * N * sizeof(float), 256));
        // the logits go to the caller's buffer when it keeps them, else into the softmax' buffer (in place)
        u16* Y = logits_out ? (u16*)logits_out : P;
        const int64_t ldy = logits_out ? Vs : ldd;
        GemmBf16Params g{};
        g.A = (const u16*)H; g.B = (const u16*)W_shard;
        g.M = (int)N; g.N = (int)Vs; g.K = (int)h;
        g.lda = (int)h; g.ldb = (int)h;
        g.a_kcontig = 1; g.b_kcontig = 1;
        g.vec_ok = (h % 8 == 0) ? 1 : 0;
        g.epi = Epi::FwdStats;
        g.Y = Y; g.ldy = (int)ldy;
        g.labels = labels; g.shard_offset = shard_offset;
        g.part_max = pm; g.part_sum = ps; g.part_tgt = pt;
        if ((e = launch_gemm_bf16(g, st)) != hipSuccess) return VP_ERR_DEVICE;
        if ((e = launch_fold_partials(pm, ps, pt, one_shard(Vs, shard_offset), (int)N, labels, local_max, local_sumexp,
                                      local_target, st)) != hipSuccess)
            return VP_ERR_DEVICE;
        // softmax' with the shard's own statistics (no one-hot term, scale 1), rows padded and zero-filled
        if ((e = launch_dlogits(Y, ldy, P, ldd, 1, nullptr, shard_offset, local_max, local_sumexp, 1.0f, (int)N,
                                (int)Vs, st)) != hipSuccess)
            return VP_ERR_DEVICE;
        GemmBf16Params a{};   // A = softmax' W_shard : M = N tokens, N = h, K = Vs; W_shard is stored [K][N]
        a.A = P; a.B = (const u16*)W_shard;
        a.M = (int)N; a.N = (int)h; a.K = (int)Vs;
        a.lda = (int)ldd; a.ldb = (int)h;
        a.a_kcontig = 1; a.b_kcontig = 0;
        a.vec_ok = (h % 8 == 0) ? 1 : 0;
        a.epi = Epi::StoreF32;
        a.C = A_out; a.ldc = (int)h;
        a.kernel_id = K_GEMM_A_ALG2;
        if ((e = launch_gemm_bf16(a, st)) != hipSuccess) return VP_ERR_DEVICE;
        return dev(launch_embed_fwd(&W_shard, labels, 1, (int)N, (int)h, (int)Vs, shard_offset, 2, &B_out, st));
    }

    // fp32: logits in the caller's buffer or the workspace, softmax' in the workspace (in place when they coincide)
    float* P = (float*)workspace;
    float* Y = logits_out ? (float*)logits_out : P;
    float* scratch = f32_bwd_scratch(N, h, Vs) ? (float*)((char*)workspace + f32_matrix_bytes(N, Vs)) : nullptr;
    if ((e = launch_gemm_f32(F32Product::Logits, (const float*)H, h, (const float*)W_shard, h, Y, (int)N, (int)Vs, (int)h, false,
                             scratch, st)) != hipSuccess)
        return VP_ERR_DEVICE;
    if ((e = launch_row_stats_f32(one_shard(Vs, shard_offset, Y), labels, (int)N, local_max, local_sumexp, local_target, st)) != hipSuccess)
        return VP_ERR_DEVICE;
    if ((e = launch_dlogits(Y, Vs, P, Vs, 0, nullptr, shard_offset, local_max, local_sumexp, 1.0f, (int)N, (int)Vs,
                            st)) != hipSuccess)
        return VP_ERR_DEVICE;
    if ((e = launch_gemm_f32(F32Product::DH, P, Vs, (const float*)W_shard, h, A_out, (int)N, (int)h, (int)Vs, false, scratch, st)) !=
        hipSuccess)
        return VP_ERR_DEVICE;
    return dev(launch_embed_fwd(&W_shard, labels, 1, (int)N, (int)h, (int)Vs, shard_offset, 4, &B_out, st));
}

vp_status vp_output_fwd_alg2_group(const void* H, const void* const* W_shards, const int64_t* rows,
                                   const int64_t* shard_offsets, int32_t p, const int64_t* labels, int64_t N, int64_t h,
                                   vp_dtype dt, uint32_t flags, float* local_max, float* local_sumexp, float* local_target,
                                   void* const* logits_out, float* A_out, void* const* B_out, void* workspace,
                                   size_t workspace_bytes, void* stream) {
    if (!H || !W_shards || !rows || !shard_offsets || p < 1 || !labels || !local_max || !local_sumexp || !local_target ||
        !A_out || !B_out)
        return VP_ERR_INVALID_ARG;
    if (!dtype_ok(dt) || (flags & ~(uint32_t)VP_SAVE_LOGITS)) return VP_ERR_INVALID_ARG;
    if (((flags & VP_SAVE_LOGITS) != 0) != (logits_out != nullptr)) return VP_ERR_INVALID_ARG;
    if (!aligned16(H) || !aligned16(workspace) || !aligned16(A_out)) return VP_ERR_INVALID_ARG;
    for (int32_t r = 0; r < p; ++r) {
        if (!W_shards[r] || !aligned16(W_shards[r]) || !sizes_ok(N, h, rows[r]) || shard_offsets[r] < 0) return VP_ERR_INVALID_ARG;
        if (logits_out && (!logits_out[r] || !aligned16(logits_out[r]))) return VP_ERR_INVALID_ARG;
        if (!B_out[r] || !aligned16(B_out[r])) return VP_ERR_INVALID_ARG;
        if (!sizes_supported(N, h, rows[r])) return VP_ERR_UNSUPPORTED;
    }
    const size_t need = vp_output_group_workspace_bytes(VP_CALL_OUTPUT_FWD_ALG2, p, N, h, rows, dt, flags);
    if (need == (size_t)-1) return VP_ERR_UNSUPPORTED;
    if (!workspace || workspace_bytes < need) return VP_ERR_WORKSPACE;
    hipStream_t st = (hipStream_t)stream;
    const PartSizes z = part_sizes(rows, 0, p, N, h, dt);
    const int S = each_slices(rows, p, N, h, dt);
    const bool bf16 = dt == VP_BF16;

    // the logits go to the caller's buffers when it keeps them, else into the softmax' buffers (in place)
    ShardList l{};
    l.n = p;
    char* d = (char*)workspace + (bf16 ? z.stats : 0);
    for (int r = 0; r < p; ++r) {
        l.rows[r] = (int)rows[r];
        l.first[r + 1] = l.first[r] + (int)fwd_tiles(rows[r]);
        l.offset[r] = shard_offsets[r];
        l.D[r] = d;
        l.ldd[r] = d_ld(rows[r], dt);
        l.Y[r] = logits_out ? logits_out[r] : d;
        l.ldy[r] = logits_out ? rows[r] : l.ldd[r];
        d += d_bytes(N, rows[r], dt);
    }
    float* slices = (float*)d;
    hipError_t e = hipSuccess;

    if (bf16) {
        GemmBf16Group y{}, a{};
        y.base = logits_product(H, labels, N, h, Epi::FwdStats);
        y.base.part_max = (float*)workspace;
        y.base.part_sum = y.base.part_max + z.tiles * N;
        y.base.part_tgt = y.base.part_max + 2 * z.tiles * N;
        a.base.M = (int)N; a.base.N = (int)h;      // A_r = softmax'_r W_r : K = rows, W_r is stored [K][N]
        a.base.ldb = a.base.ldc = (int)h;
        a.base.a_kcontig = 1;
        a.base.vec_ok = h % 8 == 0 ? 1 : 0;
        a.base.epi = Epi::StoreF32;
        a.base.kernel_id = K_GEMM_A_ALG2;
        a.base.C = S > 1 ? slices : A_out;
        a.slices = S;
        a.each = 1;
        for (int r = 0; r < p; ++r) {
            y.sh[r].B = a.sh[r].B = (const u16*)W_shards[r];
            y.sh[r].out = (void*)l.Y[r];
            y.sh[r].ld = (int)l.ldy[r];
            y.sh[r].offset = shard_offsets[r];
            a.sh[r].A = (const u16*)l.D[r];
            a.sh[r].ld = (int)l.ldd[r];
            y.sh[r].rows = a.sh[r].rows = (int)rows[r];
        }
        gemm_bf16_group_finish(y, p);
        gemm_bf16_group_finish(a, p);
        if (gemm_bf16_group_ok(y)) {
            e = launch_gemm_bf16_group(y, st);
        } else {      // shapes that the fast kernel does not take
            for (int r = 0; r < p && e == hipSuccess; ++r) {
                GemmBf16Params g = y.base;
                g.B = y.sh[r].B;
                g.N = y.sh[r].rows;
                g.Y = (u16*)y.sh[r].out; g.ldy = y.sh[r].ld;
                g.shard_offset = shard_offsets[r];
                g.part_max += (int64_t)l.first[r] * N;
                g.part_sum += (int64_t)l.first[r] * N;
                g.part_tgt += r * N;
                e = launch_gemm_bf16(g, st);
            }
        }
        if (e == hipSuccess)
            e = launch_fold_partials(y.base.part_max, y.base.part_sum, y.base.part_tgt, l, (int)N, labels, local_max,
                                     local_sumexp, local_target, st);
        // softmax' with the shards' own statistics (no one-hot term, scale 1), rows padded and zero-filled
        if (e == hipSuccess) e = launch_dlogits_group(l, 1, nullptr, local_max, local_sumexp, N, 1.0f, (int)N, st);
        if (e != hipSuccess) return VP_ERR_DEVICE;
        if (gemm_bf16_group_ok(a)) {
            e = launch_gemm_bf16_group(a, st);
            if (e == hipSuccess && S > 1) {
                ProfScope prof(K_SUM_SLICES, st);
                e = launch_sum_slices(slices, S, (int64_t)p * N * h, A_out, false, st);
            }
        } else {
            for (int r = 0; r < p && e == hipSuccess; ++r) {
                GemmBf16Params g = a.base;
                g.A = a.sh[r].A; g.lda = a.sh[r].ld;
                g.B = a.sh[r].B;
                g.K = a.sh[r].rows;
                g.C = A_out + (int64_t)r * N * h;
                e = launch_gemm_bf16(g, st);
            }
        }
    } else {
        GemmF32Shard y[GEMM_GROUP_MAX], a[GEMM_GROUP_MAX];
        for (int r = 0; r < p; ++r) {
            y[r] = {nullptr, (const float*)W_shards[r], (float*)l.Y[r], (int)rows[r], (int)l.ldy[r]};
            a[r] = {(const float*)l.D[r], (const float*)W_shards[r], nullptr, (int)rows[r], (int)l.ldd[r]};
        }
        e = launch_gemm_f32_logits((const float*)H, N, h, y, p, z.S_logits, slices, st);
        if (e == hipSuccess) e = launch_row_stats_f32(l, labels, (int)N, local_max, local_sumexp, local_target, st);
        if (e == hipSuccess) e = launch_dlogits_group(l, 0, nullptr, local_max, local_sumexp, N, 1.0f, (int)N, st);
        if (e == hipSuccess) e = launch_gemm_f32_each(N, h, a, p, S, A_out, slices, st);
    }
    // B_r = G W_r, the gather of the labels' rows: shards of one size that follow one another in one launch
    for (int r = 0; r < p && e == hipSuccess;) {
        int n = 1;
        while (r + n < p && rows[r + n] == rows[r] && shard_offsets[r + n] == shard_offsets[r] + n * rows[r]) ++n;
        e = launch_embed_fwd(W_shards + r, labels, n, (int)N, (int)h, (int)rows[r], shard_offsets[r], bf16 ? 2 : 4, B_out + r, st);
        r += n;
    }
    return dev(e);
}

vp_status vp_output_dx_alg2_gather(const float* A, const void* const* W_shards, const int64_t* rows,
                                   const int64_t* shard_offsets, int32_t p, const int64_t* labels, const float* local_max,
                                   const float* local_sumexp, const float* global_max, const float* global_sumexp, int64_t N,
                                   int64_t h, vp_dtype dt, uint32_t flags, float grad_scale, float* dH_accum, void* stream) {
    if (!A || !W_shards || !rows || !shard_offsets || p < 1 || !labels || !local_max || !local_sumexp || !global_max ||
        !global_sumexp || !dH_accum)
        return VP_ERR_INVALID_ARG;
    if (!dtype_ok(dt) || (flags & ~(uint32_t)VP_DH_OVERWRITE) || !aligned16(A) || !aligned16(dH_accum)) return VP_ERR_INVALID_ARG;
    for (int32_t r = 0; r < p; ++r) {
        if (!W_shards[r] || !aligned16(W_shards[r]) || !sizes_ok(N, h, rows[r]) || shard_offsets[r] < 0) return VP_ERR_INVALID_ARG;
        if (!sizes_supported(N, h, rows[r])) return VP_ERR_UNSUPPORTED;
    }
    if (p > GEMM_GROUP_MAX) return VP_ERR_UNSUPPORTED;
    return dev(launch_dx_alg2_gather(A, W_shards, rows, shard_offsets, p, dt == VP_BF16 ? 1 : 0, labels, local_max, local_sumexp,
                                     global_max, global_sumexp, (int)N, (int)h, grad_scale, (flags & VP_DH_OVERWRITE) != 0,
                                     dH_accum, (hipStream_t)stream));
}

vp_status vp_output_dx_alg2_group(const float* const* A, const void* const* B, int32_t p, const float* local_max,
                                  const float* local_sumexp, const float* global_max, const float* global_sumexp, int64_t N,
                                  int64_t h, vp_dtype dt, uint32_t flags, float grad_scale, float* dH_accum, void* stream) {
    if (!A || !B || p < 1 || !local_max || !local_sumexp || !global_max || !global_sumexp || !dH_accum)
        return VP_ERR_INVALID_ARG;
    if (N < 1 || h < 1 || !dtype_ok(dt) || (flags & ~(uint32_t)VP_DH_OVERWRITE)) return VP_ERR_INVALID_ARG;
    if (!aligned16(dH_accum)) return VP_ERR_INVALID_ARG;
    for (int32_t r = 0; r < p; ++r)
        if (!A[r] || !B[r] || !aligned16(A[r]) || !aligned16(B[r])) return VP_ERR_INVALID_ARG;
    if (N >= MAX_ELEMS || h >= MAX_ELEMS || N * h >= MAX_ELEMS) return VP_ERR_UNSUPPORTED;
    return dev(launch_dx_alg2(A, B, p, dt == VP_BF16 ? 1 : 0, local_max, local_sumexp, global_max, global_sumexp, (int)N,
                              (int)h, grad_scale, (flags & VP_DH_OVERWRITE) != 0, dH_accum, (hipStream_t)stream));
}

vp_status vp_output_dx_alg2(const float* A, const void* B, const float* local_max, const float* local_sumexp,
                            const float* global_max, const float* global_sumexp, int64_t N, int64_t h, vp_dtype dt,
                            uint32_t flags, float grad_scale, float* dH_accum, void* stream) {
    return vp_output_dx_alg2_group(&A, &B, 1, local_max, local_sumexp, global_max, global_sumexp, N, h, dt, flags, grad_scale,
                                   dH_accum, stream);
}

vp_status vp_embed_fwd_group(const void* const* table_shards, const int64_t* ids, int32_t p, int64_t N, int64_t h, int64_t Vs,
                             int64_t shard_offset, vp_dtype dt, void* const* outs, void* stream) {
    if (!table_shards || !ids || !outs || p < 1) return VP_ERR_INVALID_ARG;
    if (!sizes_ok(N, h, Vs) || !dtype_ok(dt) || shard_offset < 0) return VP_ERR_INVALID_ARG;
    for (int32_t r = 0; r < p; ++r)
        if (!table_shards[r] || !outs[r] || !aligned16(table_shards[r]) || !aligned16(outs[r])) return VP_ERR_INVALID_ARG;
    if (!sizes_supported(N, h, Vs)) return VP_ERR_UNSUPPORTED;
    return dev(launch_embed_fwd(table_shards, ids, p, (int)N, (int)h, (int)Vs, shard_offset, dt == VP_BF16 ? 2 : 4, outs,
                                (hipStream_t)stream));
}

vp_status vp_embed_bwd_group(const void* grad_out, const int64_t* ids, int32_t p, int64_t N, int64_t h, int64_t Vs,
                             int64_t shard_offset, vp_dtype dt, float* const* dtable_shards, void* workspace,
                             size_t workspace_bytes, void* stream) {
    if (!grad_out || !ids || !dtable_shards || p < 1) return VP_ERR_INVALID_ARG;
    if (!sizes_ok(N, h, Vs) || !dtype_ok(dt) || shard_offset < 0) return VP_ERR_INVALID_ARG;
    if (!aligned16(grad_out) || !aligned16(workspace)) return VP_ERR_INVALID_ARG;
    for (int32_t r = 0; r < p; ++r)
        if (!dtable_shards[r] || !aligned16(dtable_shards[r])) return VP_ERR_INVALID_ARG;
    if (!sizes_supported(N, h, Vs) || N > ((int64_t)1 << 24)) return VP_ERR_UNSUPPORTED;
    const size_t need = vp_workspace_bytes(VP_CALL_EMBED_BWD, N, h, Vs, dt, 0);
    if (!workspace || workspace_bytes < need) return VP_ERR_WORKSPACE;
    return dev(launch_embed_bwd(grad_out, ids, p, (int)N, (int)h, (int)Vs, shard_offset, dt == VP_BF16 ? 1 : 0, dtable_shards,
                                workspace, (hipStream_t)stream));
}

vp_status vp_embed_fwd(const void* table_shard, const int64_t* ids, int64_t N, int64_t h, int64_t Vs,
                       int64_t shard_offset, vp_dtype dt, void* out, void* stream) {
    return vp_embed_fwd_group(&table_shard, ids, 1, N, h, Vs, shard_offset, dt, &out, stream);
}

vp_status vp_embed_bwd(const void* grad_out, const int64_t* ids, int64_t N, int64_t h, int64_t Vs,
                       int64_t shard_offset, vp_dtype dt, float* dtable_shard, void* workspace, size_t workspace_bytes,
                       void* stream) {
    return vp_embed_bwd_group(grad_out, ids, 1, N, h, Vs, shard_offset, dt, &dtable_shard, workspace, workspace_bytes, stream);
}

}  // extern "C"
