// Factor stacking (SFB steps 1-2 of Section 4.3.1, receiver side): P per-worker blocks of
// B samples become one K x ld matrix, row k = p*B + b, optionally rounded to bf16.
//
// Memcpy-class, HBM-bound.  One lane produces one 16-byte output chunk (4 fp32 or 8 bf16).  A stacked matrix is dealt out
// as one sequence of chunks, 256 to a workgroup, so the lanes are all busy and a workgroup reads one contiguous piece
// whatever the width (a workgroup per 2048 columns of a row left most lanes of narrow rows idle and the last workgroup of
// every row part empty; us: 64 + 64 columns, 4096 rows, bf16 5.4 -> 3.2; 4096 + 4096, 2048 rows, fp32 26.1 -> 24.5;
// 3000 + 21841, 2048 rows, bf16 54.5 -> 52.7).  One chunk per lane: with two or four the loads of a workgroup wait for each
// other (9216 + 4096 in units of 4 columns: 31.4, 33.1 and 34.2 us with one, two and four).
// Source rows start at b*cols floats, which is only 4-byte aligned when cols is odd (e.g. 21841 classes); loads therefore use
// a 4-byte-aligned vector type and leave the choice of instruction to the compiler.  U (errors) and V (activations) of a
// layer are stacked by ONE launch: the first workgroups serve U, the rest V.
#include "psd_device.h"
#include "psd_internal.h"

namespace psd {
namespace {

constexpr int kThreads = 256;

typedef float f32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));

// fp32 -> bf16 bits, round to nearest even; NaN keeps sign and top payload bits, made quiet.
__device__ __forceinline__ uint32_t bf16_rne(float f)
{
    const uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (u >> 16) | 0x40u;
    return (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
}

template <bool BF16>
__global__ void __launch_bounds__(kThreads) pack_kernel(const PackArgs a)
{
    constexpr int E = BF16 ? 8 : 4;                    // columns per lane: one 16-byte store
    const bool is_v = static_cast<int>(blockIdx.x) >= a.groups_u;
    const PackSide& s = is_v ? a.v : a.u;
    const uint32_t first = static_cast<uint32_t>(is_v ? blockIdx.x - a.groups_u : blockIdx.x) * kThreads;
    const int cols = static_cast<int>(s.cols);
    // Nearly always all of the workgroup's rows come from one worker's block: its address is then a scalar.
    const uint32_t k_first = a.row0 + divide(first, s.chunks);
    const uint32_t p_first = __builtin_amdgcn_readfirstlane(divide(k_first, a.block));
    const float* __restrict__ src = s.src[p_first];
    const uint32_t q = first + threadIdx.x, row = divide(q, s.chunks);
    const int col = static_cast<int>(q - row * s.chunks.d) * E;
    if (row >= a.rows) return;
    const uint32_t k = a.row0 + row;
    uint32_t b = k - p_first * a.block.d;              // row of the block
    if (b >= a.block.d) {                              // not the first row's block
        const uint32_t p = divide(k, a.block);
        src = s.src[p];
        b = k - p * a.block.d;
    }
    src += int64_t(b) * cols + col;
    float v[E];
    if (col + E <= cols) {
#pragma unroll
        for (int e = 0; e < E; e += 4) {
            const f32x4_a4 t = *reinterpret_cast<const f32x4_a4*>(src + e);
            v[e] = t.x; v[e + 1] = t.y; v[e + 2] = t.z; v[e + 3] = t.w;
        }
    } else {
#pragma unroll
        for (int e = 0; e < E; ++e) v[e] = col + e < cols ? src[e] : 0.0f;   // zero the padding columns
    }
    const int64_t at = int64_t(k) * s.ld + col;
    if constexpr (BF16) {
        uint4 o;
        o.x = bf16_rne(v[0]) | (bf16_rne(v[1]) << 16);
        o.y = bf16_rne(v[2]) | (bf16_rne(v[3]) << 16);
        o.z = bf16_rne(v[4]) | (bf16_rne(v[5]) << 16);
        o.w = bf16_rne(v[6]) | (bf16_rne(v[7]) << 16);
        *reinterpret_cast<uint4*>(static_cast<uint16_t*>(s.dst) + at) = o;
    } else {
        *reinterpret_cast<float4*>(static_cast<float*>(s.dst) + at) = make_float4(v[0], v[1], v[2], v[3]);
    }
}

}  // namespace

psd_status launch_pack(PackArgs& a, int32_t out_dtype, hipStream_t st)
{
    const int64_t K = a.B * a.P;
    if (K < 1) return PSD_E_INVALID;
    const int64_t E = out_dtype == PSD_BF16 ? 8 : 4;              // ld is a multiple of E (validated)
    const int64_t cu = a.u.ld / E, cv = a.v.ld / E;               // chunks per row
    a.u.chunks = fast_div(static_cast<uint32_t>(cu));
    a.v.chunks = fast_div(static_cast<uint32_t>(cv));
    a.block = fast_div(static_cast<uint32_t>(a.B));
    const int64_t most = pack_rows_per_launch(cu, cv);
    for (int64_t row0 = 0; row0 < K; row0 += most) {
        a.row0 = static_cast<uint32_t>(row0);
        a.rows = static_cast<uint32_t>(K - row0 < most ? K - row0 : most);
        const int64_t gu = (a.rows * cu + kThreads - 1) / kThreads, gv = (a.rows * cv + kThreads - 1) / kThreads;
        a.groups_u = static_cast<int32_t>(gu);
        auto kern = out_dtype == PSD_BF16 ? pack_kernel<true> : pack_kernel<false>;
        hipLaunchKernelGGL(kern, dim3(static_cast<uint32_t>(gu + gv)), dim3(kThreads), 0, st, a);
        PSD_HIP_TRY(hipGetLastError());
    }
    return PSD_OK;
}

}  // namespace psd
