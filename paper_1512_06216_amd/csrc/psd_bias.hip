// Bias gradient of an FC layer under sufficient-factor broadcasting, with the momentum-SGD
// update fused: for z = W a + b the per-sample gradient w.r.t. b is the error vector itself
// (the same chain rule that gives Eq. 5 for W), so with the stacked errors U (K x N) that a
// worker holds after SFB step 2
//     db[n] = sum_k U[k][n] ;  mom_b = mu*mom_b + lr*(db + wd*b) ;  b = b - mom_b.
// The paper's volume analysis counts weights only (Table 3); the bias needs no extra
// communication because U is already there.
//
// Column sum (K*N factor elements read once, N outputs), bound by how many bytes are in flight and by the latency of one
// load.  A workgroup of 8 wavefronts owns COLS adjacent columns; every lane reads 16 bytes of a row (8 bf16 or 4 fp32
// columns) and keeps 8 such loads in flight, so K = 1024 rows of 32 bf16 columns are one round of loads.  The row partials
// of a column meet in LDS in two steps.  us behind a pack, 16 wavefronts -> 8, 32 columns: N = 1000, bf16, K = 256 3.26 -> 3.02, K = 2048 6.4 -> 6.3,
// N = 4096, K = 2048 6.8 -> 6.3, fp32 7.5 -> 7.3, N = 128, K = 128 2.5 -> 2.2; with 4 N = 1000, K = 2048 7.5, with 16 loads in flight
// 0.3 more everywhere, with 16 columns the same up to N = 4096.
#include "psd_device.h"
#include "psd_internal.h"

namespace psd {
namespace {

constexpr int kThreads = 512, kInFlight = 8;

template <bool BF16, int COLS>
__global__ void __launch_bounds__(kThreads)
bias_kernel(const void* __restrict__ Uv, int64_t ldu, int N, int K, float* __restrict__ bias,
            float* __restrict__ mom, float lr, float mu, float wd)
{
    constexpr int E = BF16 ? 8 : 4;                                  // columns per lane
    constexpr int LPR = COLS / E, ROWS = kThreads / LPR;             // lanes per row, rows per load of the workgroup
    constexpr int SPLIT = kThreads / COLS, PER = ROWS / SPLIT;       // second step: SPLIT threads per column, PER partials each
    static_assert(ROWS % SPLIT == 0 && PER >= 1, "whole partials per thread");
    __shared__ __attribute__((aligned(16))) float part[ROWS][COLS + 4];          // + 4: neighbouring rows on other banks
    __shared__ float part2[SPLIT][COLS];
    const int t = threadIdx.x;
    const int T = gridDim.x, xcd = blockIdx.x & 7;                   // neighbouring column blocks share an XCD (and its cache lines)
    const int blk = xcd * (T >> 3) + (xcd < (T & 7) ? xcd : (T & 7)) + (blockIdx.x >> 3);
    const int r = t / LPR, cl = (t % LPR) * E;
    const int64_t c0 = int64_t(blk) * COLS + cl;                     // first of this lane's columns
    float s[E];
#pragma unroll
    for (int e = 0; e < E; ++e) s[e] = 0.f;
    if (c0 < ldu) {                                                  // ldu is a multiple of E: all E columns exist
        const uint4* __restrict__ U = reinterpret_cast<const uint4*>(static_cast<const char*>(Uv) + c0 * (16 / E));
        const int64_t ld16 = ldu / E;                                // row length in 16-byte pieces
        for (int k = r; k < K; k += kInFlight * ROWS) {
            uint4 v[kInFlight];
#pragma unroll
            for (int u = 0; u < kInFlight; ++u)
                v[u] = k + u * ROWS < K ? U[int64_t(k + u * ROWS) * ld16] : make_uint4(0, 0, 0, 0);
#pragma unroll
            for (int u = 0; u < kInFlight; ++u) {
                const uint32_t w[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    if constexpr (BF16) {
                        s[2 * q] += __uint_as_float(w[q] << 16);     // bf16 -> fp32 is a shift
                        s[2 * q + 1] += __uint_as_float(w[q] & 0xffff0000u);
                    } else {
                        s[q] += __uint_as_float(w[q]);
                    }
                }
            }
        }
    }
#pragma unroll
    for (int e = 0; e < E; e += 4) *reinterpret_cast<float4*>(&part[r][cl + e]) = make_float4(s[e], s[e + 1], s[e + 2], s[e + 3]);
    __syncthreads();
    {
        const int c = t % COLS, g = t / COLS;
        float d = part[g * PER][c];
#pragma unroll
        for (int i = 1; i < PER; ++i) d += part[g * PER + i][c];
        part2[g][c] = d;
    }
    __syncthreads();
    if (t < COLS) {
        const int64_t n = int64_t(blk) * COLS + t;
        if (n < N) {
            float d = part2[0][t];
#pragma unroll
            for (int g = 1; g < SPLIT; ++g) d += part2[g][t];
            float b = bias[n], m = mom[n];
            upd(d, b, m, lr, mu, wd);
            mom[n] = m;
            bias[n] = b;
        }
    }
}

template <int COLS>
psd_status launch_cols(const void* U, int64_t ldu, int32_t dtype, int64_t N, int64_t K, float* bias, float* mom,
                       float lr, float mu, float wd, hipStream_t st)
{
    const int64_t blocks = (N + COLS - 1) / COLS;
    if (blocks < 1 || blocks > 0x7fffffff) return PSD_E_INVALID;
    auto kern = dtype == PSD_BF16 ? bias_kernel<true, COLS> : bias_kernel<false, COLS>;
    hipLaunchKernelGGL(kern, dim3(static_cast<uint32_t>(blocks)), dim3(kThreads), 0, st, U, ldu, static_cast<int>(N),
                       static_cast<int>(K), bias, mom, lr, mu, wd);
    PSD_HIP_TRY(hipGetLastError());
    return PSD_OK;
}

}  // namespace

psd_status launch_bias(const void* U, int64_t ldu, int32_t dtype, int64_t N, int64_t K, float* bias, float* mom,
                       float lr, float mu, float wd, hipStream_t st)
{
    // 32 columns put a workgroup on every compute unit as early as possible; once 32-column workgroups would queue (N above
    // 32 x CUs) wide rows are the better choice: N = 9216, K = 2048, bf16 11.3 us with 32 columns, 7.8 with 64, 9.3 with 128
    if (N <= 32 * int64_t(device_cu_count())) return launch_cols<32>(U, ldu, dtype, N, K, bias, mom, lr, mu, wd, st);
    // ... and 64 while those still find a compute unit each: N = 12000, K = 2048, bf16 8.3 us with 128 columns, 7.8 with 64, fp32
    // 16.9 and 14.1, K = 128 3.15 and 2.99, 3.47 and 3.44; N = 21841, K = 2048 14.4 and 17.2, 30.5 and 36.3
    if (N <= 64 * int64_t(device_cu_count())) return launch_cols<64>(U, ldu, dtype, N, K, bias, mom, lr, mu, wd, st);
    return launch_cols<128>(U, ldu, dtype, N, K, bias, mom, lr, mu, wd, st);
}

}  // namespace psd
