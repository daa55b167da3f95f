// Internal declarations shared by the translation units of libpsd (not installed).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "psd.h"
#include "psd_rules.h"

namespace psd {

// Records a failing HIP call for psd_last_hip_error() and maps it to PSD_E_HIP.
psd_status hip_failed(hipError_t e);

#define PSD_HIP_TRY(expr)                                        \
    do {                                                         \
        hipError_t e__ = (expr);                                 \
        if (e__ != hipSuccess) return ::psd::hip_failed(e__);    \
    } while (0)

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// Value of a psd_tune_set() knob; -1 = let the library choose.
int tune_value(int knob);
// Compute units of the current device (queried once per device, then cached).
int device_cu_count();

// ---- launchers (one per kernel family); arguments are already validated ----------------
struct DenseSeg {
    const float* G[PSD_MAX_MULTI_WORKERS];
    float* W;
    float* Mom;
    int64_t q, r;          // keys = q * S + r, 0 <= r < S
    int32_t P;
    int32_t S;
    FastDiv by_S, by_chunks;       // (chunks: workgroups per shard)
};
struct DenseTable {
    int32_t begin[PSD_MAX_MULTI_SEGMENTS];       // first workgroup of each segment; past the last one: none
    DenseSeg seg[PSD_MAX_MULTI_SEGMENTS];
    int32_t threads;       // lanes per workgroup (dense_threads_for)
};
struct DenseWide {          // single layer, up to PSD_MAX_WORKERS copies
    const float* G[PSD_MAX_WORKERS];
    float* W;
    float* Mom;
    int64_t n;
    int64_t q, r;          // n = q * S + r, 0 <= r < S
    int32_t P;
    int32_t S;
    FastDiv by_S, by_chunks;       // filled in by launch_dense_wide
};
psd_status launch_dense_table(const DenseTable& t, int32_t total_blocks, float lr, float mu, float wd, hipStream_t st);
psd_status launch_dense_wide(DenseWide& a, float lr, float mu, float wd, hipStream_t st);

struct PackSide {            // one of the two stacked matrices of a layer
    const float* src[PSD_MAX_WORKERS];
    void* dst;
    int64_t cols, ld;
    FastDiv chunks;          // by the 16-byte chunks of a row (this and what follows is filled in by launch_pack)
};
struct PackArgs {
    PackSide u, v;           // errors (B x N blocks -> K x ldu), activations (B x M blocks -> K x ldv)
    int64_t B;
    int32_t P;
    int32_t groups_u;        // workgroups serving u
    uint32_t row0, rows;     // rows of this launch
    FastDiv block;           // by B
};
psd_status launch_pack(PackArgs& a, int32_t out_dtype, hipStream_t st);

// ---- reconstruction (factors in reach of 32-bit offsets).  part / most_splits: with a workspace for most_splits > 1 partial sums the contraction
// may be split over up to that many workgroups per tile, each storing a partial dW (N x M, sfb_part_stride
// apart) to `part`, and the partials are summed in split order and the update applied by launch_sfb_reduce.
psd_status launch_sfb_f32(const float* U, int64_t ldu, const float* V, int64_t ldv, float* W, float* Mom,
                          int64_t N, int64_t M, int64_t K, float lr, float mu, float wd, float* part, int most_splits,
                          hipStream_t st);
// ... on the bf16 pipe, from factors cut into three bf16 planes; `tile`: see kPlaneTiles
psd_status launch_sfb_f32_planes(int tile, const float* U, int64_t ldu, const float* V, int64_t ldv, float* W, float* Mom, int64_t N,
                                 int64_t M, int64_t K, float lr, float mu, float wd, hipStream_t st);
psd_status launch_sfb_f32_planes_blocks(int tile, const float* const* U_p, int64_t ldu, const float* const* V_p, int64_t ldv, int64_t P,
                                        int64_t B, float* W, float* Mom, int64_t N, int64_t M, float lr, float mu, float wd, hipStream_t st);
// ... for the smallest layers; `tile`: see choose_small_f32 and choose_small_bf16
psd_status launch_sfb_small(int32_t dtype, const SmallTile& tile, const void* U, int64_t ldu, const void* V, int64_t ldv, float* W, float* Mom,
                            int64_t N, int64_t M, int64_t K, float lr, float mu, float wd, hipStream_t st);
psd_status launch_sfb_small_blocks(int32_t dtype, const SmallTile& tile, const void* const* U_p, int64_t ldu, const void* const* V_p, int64_t ldv,
                                   int64_t P, int64_t B, float* W, float* Mom, int64_t N, int64_t M, float lr, float mu, float wd,
                                   hipStream_t st);
psd_status launch_sfb_bf16(const uint16_t* U, int64_t ldu, const uint16_t* V, int64_t ldv, float* W, float* Mom,
                           int64_t N, int64_t M, int64_t K, float lr, float mu, float wd, float* part, int most_splits,
                           bool beside, hipStream_t st);       // beside: see choose_bf16
// reconstruction straight from the P per-worker blocks (B x ld each, no stacked copy); served when a block
// holds whole k-stages of the kernel (16 rows fp32, 32 rows bf16)
bool sfb_f32_blocks_supported(int64_t B);
bool sfb_bf16_blocks_supported(int64_t B);
psd_status launch_sfb_f32_blocks(const float* const* U_p, int64_t ldu, const float* const* V_p, int64_t ldv, int64_t P,
                                 int64_t B, float* W, float* Mom, int64_t N, int64_t M, float lr, float mu, float wd,
                                 hipStream_t st);
psd_status launch_sfb_bf16_blocks(const uint16_t* const* U_p, int64_t ldu, const uint16_t* const* V_p, int64_t ldv,
                                  int64_t P, int64_t B, float* W, float* Mom, int64_t N, int64_t M, float lr, float mu,
                                  float wd, bool beside, hipStream_t st);
// how many ways each kernel may split K for this layer when it is given a workspace (1 = not at all)
int sfb_f32_splits(int64_t N, int64_t M, int64_t K);
int sfb_bf16_splits(int64_t N, int64_t M, int64_t K);
psd_status launch_sfb_reduce(const float* part, int splits, int64_t N, int64_t M, float* W, float* Mom, float lr,
                             float mu, float wd, hipStream_t st);

// elements between two partials: N*M rounded up so that every partial starts 16-byte aligned
inline int64_t sfb_part_stride(int64_t N, int64_t M) { return (N * M + 3) / 4 * 4; }

psd_status launch_bias(const void* U, int64_t ldu, int32_t dtype, int64_t N, int64_t K, float* bias, float* mom,
                       float lr, float mu, float wd, hipStream_t st);

}  // namespace psd
