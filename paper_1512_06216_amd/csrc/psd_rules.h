// The rules by which the host shapes a launch: integer arithmetic and fitted costs, no HIP (not installed).
#pragma once
#include <stdint.h>

namespace psd {

// HIP counts the work items of a launch in 32 bits.
constexpr int64_t kMaxItems = (int64_t(1) << 32) - 1;

// ---- parameter-server sum: one float4 of every array per lane
// Lanes per workgroup of a launch over `keys` keys in `shards` shards.  One float4 per lane: with two, a workgroup's loads wait
// for each other's registers.  Small launches take small workgroups (more of them to deal out), large ones large ones (longer
// contiguous pieces of each of the P + 2 arrays).
// us at P = 8, with two float4 per lane of 256 -> now: 100 K keys 4.9 -> 4.0, 2.3 M 21.2 -> 20.2 (256 lanes; 512: 20.5,
// 1024: 23.2), 16.8 M 123.2 -> 120.4 (512; 256: 125.0, 1024: 124.3), 37.7 M 314.8 -> 306.9 (1024; 512: 310.1, 256: 334.9).
// A workgroup serves one shard, so it is never larger than a shard of average length has work for: 20 M keys in 200 000
// shards 1027 us with 1024 lanes, 222 with 256 (in 20 000 shards, 1000 keys each, 166 and 171).
inline int32_t dense_threads_for(int64_t keys, int64_t shards)
{
    int32_t threads = keys < 4000000 ? 256 : keys < 19000000 ? 512 : 1024;
    while (threads > 256 && keys / shards < int64_t(threads) * 4) threads /= 2;
    return threads;
}

// workgroups per shard
inline int32_t dense_chunks_for(int64_t n, int32_t S, int32_t threads)
{
    const int64_t longest = (n + S - 1) / S;   // floor((s+1)n/S) - floor(sn/S) <= ceil(n/S)
    const int64_t chunk = int64_t(threads) * 4;
    return static_cast<int32_t>((longest + chunk - 1) / chunk);
}

// ---- reconstruction
// Is every offset into the two stacked matrices (K rows of ldu and ldv elements of `bytes` bytes) below 2^32, with
// `reserve` rows kept free behind the last one and the columns by which a tile may overhang?
inline bool factors_in_reach(int64_t K, int64_t ldu, int64_t ldv, int64_t bytes, int64_t reserve)
{
    const int64_t ld = ldu > ldv ? ldu : ldv;
    return K * ld <= ((int64_t(1) << 32) - 4096) / bytes - reserve * ld;      // K, ld < 2^31
}

// The fp32 kernels advance the descriptor and read no further ahead than its end: what has to fit 32 bits besides the matrix is
// one stage, 64 rows where four groups contract a tile.  96 rows is what the kernels of all tile sizes have always been given.
constexpr int64_t kF32Reserve = 96;

// The bf16 kernels add the row to every offset: the stages they request past the last row, up to `stages` - 1 of `rows` rows, and
// its rounding up to whole stages have to fit as well.  One more stage for all of them, whatever the depth of the ring, so that
// the choice of the tile does not decide what is accepted; the long stages of grouped tiles fall back to a plain tile.
constexpr int64_t kBf16Stages = 4, kBf16StageRows = 32;
constexpr int64_t bf16_reserve(int64_t rows) { return (kBf16Stages + 1) * rows; }

// ---- pack
// Rows of one launch over rows of `cu` and `cv` 16-byte chunks: one lane per chunk of both matrices, and chunk numbers that fit
// 31 bits with room to spare for the last, partly filled workgroups.  A longer stack takes several launches.
inline int64_t pack_rows_per_launch(int64_t cu, int64_t cv) { return (int64_t(1) << 31) / (cu + cv); }

}  // namespace psd
