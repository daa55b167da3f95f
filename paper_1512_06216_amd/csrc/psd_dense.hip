// Parameter-server route on one GPU: per key, sum the P dense gradient copies and apply
// the momentum-SGD update (Algorithm 1 master node; Algorithm 3 non-FC branch).
//
// HBM-bound streaming kernel: (4P + 16) bytes per key, P + 3 flops.  The reduction runs
// over the P copies, which all sit in one lane's registers, so there is nothing to reduce
// across lanes and nothing to stage in LDS: the design is all about keeping many 16-byte
// loads in flight per lane and every wavefront access a full 1 KiB contiguous segment.
//
// Grid: shard-major.  Workgroup g serves chunk g % chunks of shard g / chunks, so consecutive
// workgroups (which the hardware deals round-robin over the 8 XCDs) stream consecutive
// memory and the whole launch walks the key space once, shard after shard.  Giving each
// XCD its own shard instead (workgroup g -> shard g % S) was measured 6% slower at S = 8 and
// 10% slower at S = 64: eight far-apart streams per array collide on HBM channels.
#include "psd_device.h"
#include "psd_internal.h"

namespace psd {

namespace {

// 16-byte streaming load: the gradient copies are read exactly once
__device__ __forceinline__ float4 ld_stream(const float* p) { return load_stream4(p); }

// W and Mom of a layer of at least this many keys are read and written with the streaming hint as well.
// Below it, leaving them to the caches is faster (W + Mom of such a layer, 8 bytes per key, fit the 256 MB
// last-level cache beside the gradient copies streaming past); above it the hint is: measured at P = 8,
// 16.8 M keys 83.8 % of 8 TB/s cached against 75.2 % streamed, 20 M 73.2 / 75.1, 37.7 M 70.0 / 73.8,
// 89.5 M 67.8 / 70.5.
constexpr int64_t kDenseStreamKeys = 19000000;

// keys [lo, hi) of one layer, at most 4 per lane; PC > 0: number of copies known at compile time; stream: W / Mom streamed
// (the same for every lane of the launch's layer: a uniform branch around each access)
template <int PC>
__device__ __forceinline__ void dense_span(const float* const* __restrict__ G, int P, float* __restrict__ W,
                                           float* __restrict__ Mom, int64_t lo, int64_t hi, float lr, float mu, float wd, bool stream)
{
    const int nP = PC > 0 ? PC : P;
    // W, Mom and every G[p] are 16-byte aligned, so key i is float4-aligned iff i % 4 == 0
    int64_t lo4 = (lo + 3) & ~int64_t(3);
    if (lo4 > hi) lo4 = hi;
    const int64_t hi4 = lo4 + ((hi - lo4) & ~int64_t(3));

    const int64_t i = lo4 + int64_t(threadIdx.x) * 4;
    if (i < hi4) {
        float4 acc, w, m;
        if constexpr (PC > 0) {
            float4 g[PC];
#pragma unroll
            for (int p = 0; p < PC; ++p) g[p] = ld_stream(G[p] + i);
            w = stream ? load_stream4(W + i) : *reinterpret_cast<const float4*>(W + i);
            m = stream ? load_stream4(Mom + i) : *reinterpret_cast<const float4*>(Mom + i);
            acc = g[0];
#pragma unroll
            for (int p = 1; p < PC; ++p) {
                acc.x += g[p].x; acc.y += g[p].y; acc.z += g[p].z; acc.w += g[p].w;
            }
        } else {
            w = stream ? load_stream4(W + i) : *reinterpret_cast<const float4*>(W + i);
            m = stream ? load_stream4(Mom + i) : *reinterpret_cast<const float4*>(Mom + i);
            // Any number of copies: eight at a time, then four, two and one, each group's loads in flight together and the copies
            // added in order (one copy after the other, each waited for: 3 M keys, P = 7 27.5 us against 25.3).
            bool none = true;
            auto add = [&](const float4& g) {
                if (none) acc = g;
                else { acc.x += g.x; acc.y += g.y; acc.z += g.z; acc.w += g.w; }
                none = false;
            };
            int p = 0;
            for (; p + 8 <= nP; p += 8) {
                float4 g[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) g[j] = ld_stream(G[p + j] + i);
#pragma unroll
                for (int j = 0; j < 8; ++j) add(g[j]);
            }
            float4 g4[4], g2[2], g1;
            if (nP & 4) {
#pragma unroll
                for (int j = 0; j < 4; ++j) g4[j] = ld_stream(G[p + j] + i);
            }
            const int p2 = p + (nP & 4), p1 = p2 + (nP & 2);
            if (nP & 2) {
                g2[0] = ld_stream(G[p2] + i);
                g2[1] = ld_stream(G[p2 + 1] + i);
            }
            if (nP & 1) g1 = ld_stream(G[p1] + i);
            if (nP & 4) {
#pragma unroll
                for (int j = 0; j < 4; ++j) add(g4[j]);
            }
            if (nP & 2) {
                add(g2[0]);
                add(g2[1]);
            }
            if (nP & 1) add(g1);
        }
        upd(acc.x, w.x, m.x, lr, mu, wd);
        upd(acc.y, w.y, m.y, lr, mu, wd);
        upd(acc.z, w.z, m.z, lr, mu, wd);
        upd(acc.w, w.w, m.w, lr, mu, wd);
        if (stream) {
            store_stream4(Mom + i, m);
            store_stream4(W + i, w);
        } else {
            *reinterpret_cast<float4*>(Mom + i) = m;
            *reinterpret_cast<float4*>(W + i) = w;
        }
    }
    // at most 3 unaligned keys at each end of the span
    const int nh = static_cast<int>(lo4 - lo), nt = static_cast<int>(hi - hi4);
    const int t = threadIdx.x;
    if (t < nh + nt) {
        const int64_t i = t < nh ? lo + t : hi4 + (t - nh);
        float g = G[0][i];
        for (int p = 1; p < nP; ++p) g += G[p][i];
        float wv = W[i], mv = Mom[i];
        upd(g, wv, mv, lr, mu, wd);
        Mom[i] = mv;
        W[i] = wv;
    }
}

// Where a workgroup's keys lie is a chain of scalar loads and divisions before its first load of data: everything is requested at
// once, with the line of the pointers that the span will need, nothing comes from the hidden arguments of a launch (the size of a
// workgroup: one more round trip), and the divisions are by multiplication.  Before, with a loop over the segments: 16 segments of
// 65536 keys, P = 4 11.7 us, now 7.7; the five convolution layers of AlexNet, P = 8 20.5 and 19.4; one layer of 1 M keys, P = 2
// 5.8 and 5.6; of 37.7 M keys 307 and 307.
template <int THREADS, class Layer>
__device__ __forceinline__ void dense_block(const Layer& a, int local_block, float lr, float mu, float wd)
{
    const float* const* G = a.G;
    const int P = a.P, S = a.S;
    const int64_t q = a.q, r = a.r;
    const FastDiv by_S = a.by_S, by_chunks = a.by_chunks;
    asm volatile("" : : "s"(G[0]), "s"(a.W), "s"(a.Mom));
    const int s = static_cast<int>(divide(static_cast<uint32_t>(local_block), by_chunks));
    const int64_t c = local_block - s * static_cast<int>(by_chunks.d);
    // shard s owns [floor(s n / S), floor((s+1) n / S)).  With n = q S + r this is s q + floor(s r / S): exact, and for
    // S < 2^16 the division is a 32-bit one
    int64_t begin, end;
    if (S < (1 << 16)) {
        const uint32_t rr = static_cast<uint32_t>(r), su = static_cast<uint32_t>(s);
        begin = int64_t(s) * q + divide(su * rr, by_S);
        end = int64_t(s + 1) * q + divide((su + 1u) * rr, by_S);
    } else {
        begin = int64_t(s) * q + (int64_t(s) * r) / S;
        end = int64_t(s + 1) * q + (int64_t(s + 1) * r) / S;
    }
    float* const W = a.W;
    float* const Mom = a.Mom;
    constexpr int64_t chunk = int64_t(THREADS) * 4;
    const int64_t lo = begin + c * chunk;
    if (lo >= end) return;
    const int64_t hi = lo + chunk < end ? lo + chunk : end;
    const bool stream = q * S + r >= kDenseStreamKeys;       // n = q S + r
    switch (P) {
        case 8: dense_span<8>(G, P, W, Mom, lo, hi, lr, mu, wd, stream); break;
        case 4: dense_span<4>(G, P, W, Mom, lo, hi, lr, mu, wd, stream); break;
        case 2: dense_span<2>(G, P, W, Mom, lo, hi, lr, mu, wd, stream); break;
        case 16: dense_span<16>(G, P, W, Mom, lo, hi, lr, mu, wd, stream); break;
        default: dense_span<0>(G, P, W, Mom, lo, hi, lr, mu, wd, stream); break;
    }
}

template <int THREADS>
__global__ void __launch_bounds__(THREADS) dense_ps_table_kernel(const DenseTable t, int first, float lr, float mu, float wd)
{
    // Which layer does this workgroup belong to: its segment by halving, in registers (a loop over the segments is a round trip
    // for each).
    static_assert(PSD_MAX_MULTI_SEGMENTS == 16, "four halvings");
    const int b = first + blockIdx.x;
    int at[16], l = 0;
#pragma unroll
    for (int j = 0; j < 16; ++j) at[j] = t.begin[j];
#pragma unroll
    for (int h = 8; h > 0; h /= 2) {
        const bool upper = b >= at[h];
        l += upper ? h : 0;
#pragma unroll
        for (int j = 1; j < h; ++j) at[j] = upper ? at[h + j] : at[j];
    }
    dense_block<THREADS>(t.seg[l], b - t.begin[l], lr, mu, wd);
}

template <int THREADS>
__global__ void __launch_bounds__(THREADS) dense_ps_wide_kernel(const DenseWide a, int first, float lr, float mu, float wd)
{
    dense_block<THREADS>(a, first + blockIdx.x, lr, mu, wd);
}

// `blocks` workgroups, in as many launches as it takes (one but for millions of short shards)
template <class Args>
psd_status launch_blocks(void (*kern)(Args, int, float, float, float), const Args& a, int threads, int64_t blocks, float lr, float mu,
                         float wd, hipStream_t st)
{
    const int64_t most = kMaxItems / threads;
    for (int64_t first = 0; first < blocks; first += most) {
        const int64_t n = blocks - first < most ? blocks - first : most;
        hipLaunchKernelGGL(kern, dim3(static_cast<uint32_t>(n)), dim3(threads), 0, st, a, static_cast<int>(first), lr, mu, wd);
        PSD_HIP_TRY(hipGetLastError());
    }
    return PSD_OK;
}

}  // namespace

psd_status launch_dense_table(const DenseTable& t, int32_t total_blocks, float lr, float mu, float wd, hipStream_t st)
{
    auto kern = t.threads == 256 ? dense_ps_table_kernel<256> : t.threads == 512 ? dense_ps_table_kernel<512> : dense_ps_table_kernel<1024>;
    return launch_blocks<DenseTable>(kern, t, t.threads, total_blocks, lr, mu, wd, st);
}

psd_status launch_dense_wide(DenseWide& a, float lr, float mu, float wd, hipStream_t st)
{
    const int threads = dense_threads_for(a.n, a.S);
    const int32_t chunks = dense_chunks_for(a.n, a.S, threads);
    a.by_S = fast_div(static_cast<uint32_t>(a.S));
    a.by_chunks = fast_div(static_cast<uint32_t>(chunks));
    const int64_t blocks = int64_t(chunks) * a.S;
    if (blocks < 1 || blocks > (int64_t(1) << 30)) return PSD_E_INVALID;
    auto kern = threads == 256 ? dense_ps_wide_kernel<256> : threads == 512 ? dense_ps_wide_kernel<512> : dense_ps_wide_kernel<1024>;
    return launch_blocks<DenseWide>(kern, a, threads, blocks, lr, mu, wd, st);
}

// Second stage of a split reconstruction: the `splits` partial dW matrices are exactly "several dense
// copies of one gradient", so the parameter-server kernel sums them (in split order) and updates.
psd_status launch_sfb_reduce(const float* part, int splits, int64_t N, int64_t M, float* W, float* Mom, float lr,
                             float mu, float wd, hipStream_t st)
{
    DenseWide a;
    for (int p = 0; p < PSD_MAX_WORKERS; ++p) a.G[p] = p < splits ? part + p * sfb_part_stride(N, M) : nullptr;
    a.W = W; a.Mom = Mom; a.n = N * M; a.P = splits; a.S = 1;
    a.q = a.n; a.r = 0;
    return launch_dense_wide(a, lr, mu, wd, st);
}

}  // namespace psd
