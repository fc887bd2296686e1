// Internal declarations shared by the libvp translation units (host side only; device
// code does not call across files).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "vp.h"

namespace vp {

typedef unsigned short u16;  // bf16 bit pattern

static inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
static inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Kernel ids for the optional per-kernel timing (names in vp_profile.hip, same order).
enum KernelId : int {
    K_GEMM_FWD_STATS = 0, K_GEMM_DLOGITS, K_GEMM_DH, K_GEMM_DW, K_FOLD, K_COMBINE, K_DLOGITS_EW, K_GEMM_F32,
    K_ROWSTATS_F32, K_EMBED_FWD, K_EMBED_SORT, K_EMBED_ACCUM, K_GEMM_A_ALG2, K_DX_ALG2, K_SUM_SLICES, K_ZERO_PAD, K_COUNT
};

// Brackets the launches made during its lifetime with two events when timing is enabled;
// does nothing (and touches no HIP API) otherwise.
class ProfScope {
public:
    ProfScope(int id, hipStream_t st);
    ~ProfScope();
    ProfScope(const ProfScope&) = delete;
    ProfScope& operator=(const ProfScope&) = delete;
private:
    int id_;
    hipStream_t st_;
    void* a_;
};

// Macro tile of the bf16 MFMA kernels (rows x cols of the output per workgroup).
constexpr int GEMM_BM = 256;
constexpr int GEMM_BN = 256;

// What the bf16 GEMM does with its accumulators.
enum class Epi : int {
    FwdStats = 0,   // per-row partial max / sum-exp / target logit (+ optional bf16 store of Y)
    DLogits = 1,    // D = (exp(Y - m)/sum - onehot) * scale, stored as bf16
    StoreF32 = 2,   // C = acc
    AccumF32 = 3    // C += acc
};

struct GemmBf16Params {
    // operands: A is logically [M, K], B is logically [N, K]
    const u16* A;
    const u16* B;
    int M, N, K;
    int lda, ldb;        // leading dimension in elements of the matrices as stored
    int a_kcontig;       // 1: A stored [M][K]; 0: stored [K][M]
    int b_kcontig;       // 1: B stored [N][K]; 0: stored [K][N]
    int vec_ok;          // 1: all rows of A and B start 16-byte aligned (16-byte loads allowed)
    // epilogue
    Epi epi;
    float* C;            // StoreF32 / AccumF32: [M, N] fp32, ldc
    int ldc;
    u16* Y;              // FwdStats: optional bf16 [M, N] store (ldy); DLogits: D output
    int ldy;
    const int64_t* labels;   // [M]
    int64_t shard_offset;
    float* part_max;     // FwdStats: [tiles_n, M]
    float* part_sum;     // FwdStats: [tiles_n, M]
    float* part_tgt;     // FwdStats: [M], written only for rows whose label is in this shard
    const float* gmax;   // DLogits: [M]
    const float* gsum;   // DLogits: [M]
    float scale;         // DLogits
    int kernel_id;       // timing slot; 0 = chosen from the epilogue (resolved by launch_gemm_bf16)
    unsigned long long* trace;   // measurement aid: phase stamps per workgroup and tile (nullptr: none)
    int trace_cap;               // tiles per workgroup the trace buffer holds
};

// One product of the output layer over several shards on this device as ONE launch of the fast kernel.  The shards'
// matrices are laid end to end in the dimension the vocabulary has in the product:
//   logits (A, B K-contiguous)        along N: a tile column belongs to one shard,
//   dW     (A, B K-strided)           along M: a tile row belongs to one shard,
//   dH     (A K-contiguous, B K-str.) along K: a tile walks the k tiles of one shard after the other.
// `base` holds what the shards share, sh[r] what they do not.
constexpr int GEMM_GROUP_MAX = 16;     // shards per launch (they travel in the kernel arguments)
struct GemmBf16Shard {
    const u16* A;        // dW, dH: D_r
    const u16* B;        // logits, dH: W_r
    void* out;           // logits: Y_r or D_r (may be nullptr); dW: dW_r
    int64_t offset;      // first vocabulary row
    int rows;            // vocabulary rows of the shard
    int ld;              // row stride of A (dW, dH) or of out (logits), elements
};
struct GemmBf16Group {
    GemmBf16Params base;
    int n;                         // shards
    int slices;                    // dH: K slices, slice z writes base.C + z M ldc
    int each;                      // not 0: a product per shard in place of their sum over the shards, every one in `slices`
                                   // slices; slice z of shard r writes base.C + (z n + r) M ldc
    int total;                     // tile columns / tile rows / k tiles of all shards
    int first[GEMM_GROUP_MAX];     // the first of them that belongs to shard r (INT_MAX from n on)
    GemmBf16Shard sh[GEMM_GROUP_MAX];
};
// Fills n, total and first from sh[].rows.
void gemm_bf16_group_finish(GemmBf16Group& g, int n);
// Whether every shard meets the fast kernel's preconditions (and the generic kernel has not been forced).
bool gemm_bf16_group_ok(const GemmBf16Group& g);
hipError_t launch_gemm_bf16_group(const GemmBf16Group& g, hipStream_t st);
// K slices of a dH product [M, N] over kt k tiles (the slices' partial outputs take slices * M * N floats of scratch).
int gemm_bf16_slices(int64_t M, int64_t N, int64_t kt);
// The same for n products of at most kt k tiles each (n * slices * M * N floats of scratch).
int gemm_bf16_slices_each(int64_t M, int64_t N, int64_t kt, int n);
// Outputs of a sum over partial matrices: output r of count[r] floats, whose partials start at float first[r] of each slice.
struct SumList {
    int n;
    int64_t first[GEMM_GROUP_MAX], count[GEMM_GROUP_MAX];
    float* C[GEMM_GROUP_MAX];
};
// C_r (+)= sum over S slices (in a fixed order), consecutive slices `stride` floats apart.  Timed by the caller: alone, or
// with the product it ends.
hipError_t launch_sum_slices(const float* part, int S, int64_t stride, const SumList& l, bool accumulate, hipStream_t st);
// the same for one output of MN floats
hipError_t launch_sum_slices(const float* part, int S, int64_t MN, float* C, bool accumulate, hipStream_t st);

// Dispatches to the fast kernel when its preconditions hold (and the generic kernel has not been
// forced through vp_profile_force_generic_gemm), else to the generic kernel.
hipError_t launch_gemm_bf16(const GemmBf16Params& p, hipStream_t st);
void gemm_bf16_force_generic(bool on);
// Measurement aid: device buffer into which the fast kernel's next launches write their phase stamps
// (nullptr: off); kernel_id >= 0 restricts it to the launches timed under that kernel id.
void gemm_bf16_set_trace(void* buf, size_t bytes, int kernel_id);
bool gemm_bf16_generic_forced();
bool gemm_bf16_out_ok(const GemmBf16Params& p);
bool gemm_bf16_fast_ok(const GemmBf16Params& p);
hipError_t launch_gemm_bf16_fast(const GemmBf16Params& p, hipStream_t st);

// The fp32 products of one shard.  Logits: C[m,n] = sum_k A[m lda + k] B[n ldb + k]; DH (and A of Algorithm 2): A[m lda + k]
// B[k ldb + n]; DW: A[k lda + m] B[k ldb + n].  C is dense [M, N].
enum class F32Product { Logits, DH, DW };
// scratch: at least gemm_f32_scratch_floats(kind, M, N, K) floats (outputs with few tiles and a long K are computed in K slices).
hipError_t launch_gemm_f32(F32Product kind, const float* A, int64_t lda, const float* B, int64_t ldb, float* C, int M, int N, int K,
                           bool accumulate, float* scratch, hipStream_t st);
size_t gemm_f32_scratch_floats(F32Product kind, int64_t M, int64_t N, int64_t K);
// Floats that the launches of this product write to scratch, from their arguments.
size_t gemm_f32_written_floats(F32Product kind, int64_t M, int64_t N, int64_t K);

// The fp32 products over several shards in one launch (n <= GEMM_GROUP_MAX).
struct GemmF32Shard {
    const float* A;      // dH, dW: D_r
    const float* B;      // logits, dH: W_r
    float* C;            // logits: Y_r; dW: dW_r
    int rows;            // vocabulary rows
    int ld;              // row stride of Y_r or D_r
};
// K slices of a logits or dW product with this many 64 x 64 tiles (of all its shards)
int gemm_f32_group_slices(int64_t tiles, int64_t K);
// scratch, if slices > 1: slices * (N * ld of every shard, each rounded up to 4) floats
hipError_t launch_gemm_f32_logits(const float* H, int64_t N, int64_t h, const GemmF32Shard* sh, int n, int slices, float* scratch,
                                  hipStream_t st);
// scratch: n * slices * N * h floats unless n * slices == 1
hipError_t launch_gemm_f32_dh(int64_t N, int64_t h, const GemmF32Shard* sh, int n, int slices, float* dH, bool accumulate,
                              float* scratch, hipStream_t st);
// scratch, if slices > 1: slices * (rows * h of every shard, each rounded up to 4) floats
hipError_t launch_gemm_f32_dw(const float* H, int64_t N, int64_t h, const GemmF32Shard* sh, int n, int slices, float* scratch,
                              hipStream_t st);
// dH, then dW, or both in one launch (scratch as for the two)
hipError_t launch_gemm_f32_dh_dw(const float* H, int64_t N, int64_t h, const GemmF32Shard* sh, int n, int dh_slices, int dw_slices,
                                 float* dH, bool accumulate, float* scratch, hipStream_t st);
int gemm_f32_dh_slices(int64_t N, int64_t h, int64_t rows, int n);
// A_r = P_r W_r of every shard (A in sh[].A), out [n, N, h]; scratch, if slices > 1: n * slices * N * h floats
hipError_t launch_gemm_f32_each(int64_t N, int64_t h, const GemmF32Shard* sh, int n, int slices, float* out, float* scratch,
                                hipStream_t st);
int gemm_f32_each_slices(int64_t N, int64_t h, int64_t rows, int n);

// Per-shard arguments of the small kernels that serve all shards of a group in one launch.
struct ShardList {
    int n;
    int rows[GEMM_GROUP_MAX];
    int first[GEMM_GROUP_MAX + 1];     // fold: first column tile of shard r; first[n] = all of them
    int64_t offset[GEMM_GROUP_MAX];
    int64_t ldy[GEMM_GROUP_MAX], ldd[GEMM_GROUP_MAX];
    const void* Y[GEMM_GROUP_MAX];
    void* D[GEMM_GROUP_MAX];
};

// Row statistics of stored fp32 logits (fp32 path): m', sum', t' of shard r from Y[r] (row stride ldy[r]) into row r of
// lmax, lsum and ltgt.
hipError_t launch_row_stats_f32(const ShardList& l, const int64_t* labels, int N, float* lmax, float* lsum, float* ltgt,
                                hipStream_t st);

// Fold the per-column-tile partial statistics written by the FwdStats epilogue: shard r's partials are the rows
// first[r] .. first[r+1]-1 of part_max / part_sum, its target logits row r of part_tgt, its results row r of lmax, lsum
// and ltgt (all rows of N).
hipError_t launch_fold_partials(const float* part_max, const float* part_sum, const float* part_tgt, const ShardList& l,
                                int N, const int64_t* labels, float* lmax, float* lsum, float* ltgt, hipStream_t st);

hipError_t launch_combine(const float* lmax, const float* lsum, const float* ltgt, int p, int N,
                          float* gmax, float* gsum, float* loss_row, float* loss_mean, hipStream_t st);

// D = (exp(Y - m)/sum - onehot) * scale from stored logits of one shard; is_bf16 selects the type of Y and D.
// Y has row stride ldy, D row stride ldd (elements); columns Vs..ldd-1 of D are zeroed.
// labels == nullptr: no one-hot term (softmax' of Algorithm 2 with the local statistics).
hipError_t launch_dlogits(const void* Y, int64_t ldy, void* D, int64_t ldd, int is_bf16, const int64_t* labels,
                          int64_t off, const float* gmax, const float* gsum, float scale, int N, int Vs,
                          hipStream_t st);

// The same for all shards of a list (D_r from Y_r, whose row stride is ldy[r]; D_r may be Y_r).  Shard r takes its
// statistics r * shard_stats floats on (0: all the same).
hipError_t launch_dlogits_group(const ShardList& l, int is_bf16, const int64_t* labels, const float* gmax, const float* gsum,
                                int64_t shard_stats, float scale, int N, hipStream_t st);

// dH += (A_r * c_r - B_r) * scale over p shards, c_ri = lsum_ri exp(lmax_ri - gmax_i) / gsum_i  (Algorithm 2)
// (overwrite: dH = ... instead of +=; A and B are host arrays, lmax and lsum [p, N])
hipError_t launch_dx_alg2(const float* const* A, const void* const* B, int p, int b_is_bf16, const float* lmax,
                          const float* lsum, const float* gmax, const float* gsum, int N, int h, float scale, bool overwrite,
                          float* dH, hipStream_t st);

// The same for p <= GEMM_GROUP_MAX shards with A [p, N, h] and the rows of B taken from the shards: row labels[i] of W.
hipError_t launch_dx_alg2_gather(const float* A, const void* const* W, const int64_t* rows, const int64_t* offsets, int p,
                                 int is_bf16, const int64_t* labels, const float* lmax, const float* lsum, const float* gmax,
                                 const float* gsum, int N, int h, float scale, bool overwrite, float* dH, hipStream_t st);

// Zeroes the padding columns rows[r] .. ldd[r]-1 of the bf16 matrices D_r [N, ldd[r]].
hipError_t launch_zero_pad_columns(const ShardList& l, int N, hipStream_t st);

// Input layer of p consecutive shards of Vs rows each, the first at row `off` of the vocabulary (host arrays of device
// pointers, one per shard).
constexpr int EMBED_GROUP_MAX = 32;    // shards per launch
hipError_t launch_embed_fwd(const void* const* tables, const int64_t* ids, int p, int N, int h, int Vs, int64_t off,
                            int elem_bytes, void* const* outs, hipStream_t st);

size_t embed_bwd_workspace(int64_t N, int64_t h, int64_t Vs, int elem_bytes);
hipError_t launch_embed_bwd(const void* gout, const int64_t* ids, int p, int N, int h, int Vs, int64_t off,
                            int is_bf16, float* const* dtables, void* ws, hipStream_t st);

}  // namespace vp
