// The update of W and Mom: its arithmetic, and the classes that apply it to tiles (not installed).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace psd {

// The update of Algorithm 3's update line with the momentum / weight-decay reading of Lambda
// (Section 3.3, Eq. 3-4):  Mom <- mu*Mom + lr*(d + wd*w) ;  w <- w - Mom.
// The ONE place this arithmetic lives: every kernel (fp32 / bf16 reconstruction, dense
// parameter-server sum, bias) calls it, so the routes cannot drift apart.
__device__ __forceinline__ void upd(float d, float& w, float& mo, float lr, float mu, float wd)
{
    mo = __fmaf_rn(mu, mo, lr * __fmaf_rn(wd, w, d));   // wd = 0 leaves d unchanged
    w = w - mo;
}

// Streaming ("non-temporal") accesses for data that is touched exactly once per launch -- W and Mom in
// every update, the gradient copies of the parameter-server sum.  Without the hint every W / Mom line is
// allocated in the XCD's 4 MB L2 on its way through and the update leaves the L2 full of dirty lines; the
// factor fetches of the workgroups that are in their MFMA loop then have those write-backs on their miss
// path.  Measured on the bf16 reconstruction: the hint on both the loads and the stores takes fc6 from
// 220 to 198 us and the 4096 -> 1000 layer from 38 to 31 us while the bytes that cross the L2 / fabric
// boundary stay the same (636 against 630 MB) and the mean L1 -> L2 read latency falls from 477 to 404
// cycles (either hint alone: no gain; the scope bits sc0 / sc1 on top: slower).  Only for accesses that
// cover whole cache lines: streamed stores to parts of a line are expensive.
typedef float f32x4_nt __attribute__((ext_vector_type(4)));
__device__ __forceinline__ float4 load_stream4(const float* p)
{
    const f32x4_nt v = __builtin_nontemporal_load(reinterpret_cast<const f32x4_nt*>(p));
    return make_float4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void store_stream4(float* p, float4 x)
{
    const f32x4_nt v = {x.x, x.y, x.z, x.w};
    __builtin_nontemporal_store(v, reinterpret_cast<f32x4_nt*>(p));
}

// The same number, of which the compiler does not know that it is: what is computed from it anew does not stay in registers
// from where it was computed before.
__device__ __forceinline__ int anew(int x)
{
#ifdef __HIP_DEVICE_COMPILE__
    asm("" : "+v"(x));
#endif
    return x;
}

// ---- Update of W and Mom from rows of dW in LDS ------------------------------------------------------------
// A cache line holds 32 fp32.  Row n of W starts `line_shift(n)` elements into a line, a different number for every row
// unless M is a multiple of 32, so a fixed split of a tile's columns over lanes makes every 128-byte access straddle two
// lines: twice the requests on the path from L1 to L2, and stores that cover parts of lines.  Here each row of the tile is
// put into LDS `line_shift` elements to the right, and what is read back from aligned places of LDS are whole lines of W.
__device__ __forceinline__ int line_shift(const float* W, int64_t n, int64_t M)
{
    return static_cast<int>((static_cast<uint32_t>(n) * static_cast<uint32_t>(M) +
                             static_cast<uint32_t>(reinterpret_cast<uintptr_t>(W) >> 2)) & 31u);
}

// Row length of the LDS buffer, in floats: room for the shift, and such that (row length + M) / 4 is odd for M a multiple
// of 4: the 16-byte writes of rows r, r + 1, ... then fall on different banks (1500 -> 1400: all on the same ones with
// WIDTH + 36, 8 us of conflicts).
__host__ __device__ constexpr int row_stride(int width, int64_t M) { return width + 32 + (M % 8 == 0 ? 4 : 0); }

// Row r (of ROWS) of the buffer starts at buf + r * row_stride and holds dW[row_n(r)][m0 + c] at place c + line_shift,
// c < WIDTH; with PARTS > 1 there are that many buffers one after the other, whose sum is dW.
// Every wavefront access covers one line of eight rows (8 lanes of 16 bytes each).  W and Mom of DEPTH such line groups
// are requested by fetch<0>() before the rows are even written, and those of the next DEPTH before the present ones are
// used.  The quad in which a row begins and the one in which it ends, where M is not a multiple of 4, are shared with the
// neighbouring tiles: their elements, three at most at each end, are read and written one by one, by lane 4 * end + i of the
// eight that stand for a row, so that no workgroup touches an element of another's (nor one past the end of W).
// Lines that lie inside the tile are streamed (see load_stream4), the ones it shares with its neighbours go
// through the caches, but for the stores of the narrow tiles of small layers: what lies dirty in L2 when a kernel ends has
// to be written back before the next one starts, a microsecond that large layers do not notice.
template <int ROWS, int WIDTH, int WAVES, int DEPTH, int PARTS, class RowN>
struct RowUpdate {
    static constexpr int LINES = WIDTH / 32 + 1, GROUPS = ROWS / 8, ALL = GROUPS * LINES;       // units: one line of eight rows
    static constexpr int UNITS = (ALL + WAVES - 1) / WAVES, BATCHES = (UNITS + DEPTH - 1) / DEPTH;
    static constexpr int ENDS = (GROUPS + WAVES - 1) / WAVES;                                   // a wavefront's groups of eight rows
    static_assert(ROWS % 8 == 0 && WIDTH % 32 == 0, "whole lines of eight rows");
    float* W;
    float* Mom;
    RowN row_n;
    int64_t m0, N, M;
    int wave, lane, cols, stride;                  // cols: columns of the tile that exist
    float4 w[2][DEPTH], mo[2][DEPTH];
    float w_end[ENDS], mo_end[ENDS];

    __device__ __forceinline__ RowUpdate(float* W_, float* Mom_, RowN row, int64_t m0_, int64_t N_, int64_t M_, int wave_, int lane_)
        : W(W_), Mom(Mom_), row_n(row), m0(m0_), N(N_), M(M_), wave(wave_), lane(lane_),
          cols(static_cast<int>(M_ - m0_ < WIDTH ? M_ - m0_ : WIDTH)), stride(row_stride(WIDTH, M_))
    {
    }
    struct Place {
        int64_t off;                               // of this lane's quad in W
        int at;                                    // ... in the row buffer
        bool quad, whole_line;                     // does the tile own all of it, all of its line
    };
    __device__ __forceinline__ Place place(int u) const
    {
        // A wavefront takes the lines of eight rows one after the other, next to wavefronts that do so with the next rows
        // (line by line across the rows, or with rows further apart, the update is 3-8 % slower); with more wavefronts than
        // groups of rows, neighbouring wavefronts take neighbouring lines.
        constexpr bool WALK = GROUPS % WAVES == 0;
        const int id = wave + WAVES * u;
        const int line = WALK ? u % LINES : id % LINES, r = (WALK ? wave + WAVES * (u / LINES) : id / LINES) * 8 + (lane >> 3);
        const int q = 4 * (lane & 7);
        const int64_t n = row_n(r);
        const int first = 32 * line - line_shift(W, n, M);       // column of the line's first element
        const int c = first + q;
        Place p;
        p.at = r * stride + 32 * line + q;
        p.off = n * M + m0 + c;
        p.quad = n < N && (WALK || id < ALL) && c >= 0 && c + 3 < cols;
        p.whole_line = first >= 0 && first + 32 <= cols;
        return p;
    }
    struct End {
        int64_t off;
        int at;
        bool any;
    };
    __device__ __forceinline__ End end(int e, int lane) const
    {
        const int group = wave + WAVES * e, r = group * 8 + (lane >> 3), i = lane & 3;
        const int64_t n = row_n(r);
        const int shift = line_shift(W, n, M), before = -shift & 3;
        const int lead = before < cols ? before : cols;          // columns before the first whole quad
        const int last = ((cols + shift) & ~3) - shift;          // column where the quad begins that the tile owns in part
        const int c = lane & 4 ? (last > lead ? last : lead) + i : i;
        return {n * M + m0 + c, r * stride + shift + c, n < N && group < GROUPS && c < (lane & 4 ? cols : lead)};
    }
    template <int B>
    __device__ __forceinline__ void fetch()
    {
#pragma unroll
        for (int j = 0; j < DEPTH; ++j) {
            if (B * DEPTH + j >= UNITS) continue;
            const Place p = place(B * DEPTH + j);
            if (!p.quad) continue;
            if (p.whole_line) {
                w[B & 1][j] = load_stream4(W + p.off);
                mo[B & 1][j] = load_stream4(Mom + p.off);
            } else {
                w[B & 1][j] = *reinterpret_cast<const float4*>(W + p.off);
                mo[B & 1][j] = *reinterpret_cast<const float4*>(Mom + p.off);
            }
        }
        if (B == 0 && M % 4 != 0) {
#pragma unroll
            for (int e = 0; e < ENDS; ++e) {
                const End p = end(e, lane);
                if (!p.any) continue;
                w_end[e] = W[p.off];
                mo_end[e] = Mom[p.off];
            }
        }
    }
    template <int B = 0>
    __device__ __forceinline__ void run(const float* buf, float lr, float mu, float wd)
    {
        if constexpr (B < BATCHES) {
            if constexpr (B + 1 < BATCHES) fetch<B + 1>();
#pragma unroll
            for (int j = 0; j < DEPTH; ++j) {
                if (B * DEPTH + j >= UNITS) continue;
                const Place p = place(B * DEPTH + j);
                if (!p.quad) continue;
                float4 d = *reinterpret_cast<const float4*>(buf + p.at);
#pragma unroll
                for (int i = 1; i < PARTS; ++i) {
                    const float4 e = *reinterpret_cast<const float4*>(buf + i * ROWS * stride + p.at);
                    d.x += e.x; d.y += e.y; d.z += e.z; d.w += e.w;
                }
                float4 &wv = w[B & 1][j], &mv = mo[B & 1][j];
                upd(d.x, wv.x, mv.x, lr, mu, wd);
                upd(d.y, wv.y, mv.y, lr, mu, wd);
                upd(d.z, wv.z, mv.z, lr, mu, wd);
                upd(d.w, wv.w, mv.w, lr, mu, wd);
                if (WIDTH < 128 || p.whole_line) {
                    store_stream4(Mom + p.off, mv);
                    store_stream4(W + p.off, wv);
                } else {
                    *reinterpret_cast<float4*>(Mom + p.off) = mv;
                    *reinterpret_cast<float4*>(W + p.off) = wv;
                }
            }
            if constexpr (B == 0) run_ends(buf, lr, mu, wd);
            run<B + 1>(buf, lr, mu, wd);
        }
    }
    __device__ __forceinline__ void run_ends(const float* buf, float lr, float mu, float wd)
    {
        if (M % 4 == 0) return;
#pragma unroll
        for (int e = 0; e < ENDS; ++e) {
            const End p = end(e, anew(lane));
            if (!p.any) continue;
            float d = buf[p.at];
#pragma unroll
            for (int i = 1; i < PARTS; ++i) d += buf[i * ROWS * stride + p.at];
            upd(d, w_end[e], mo_end[e], lr, mu, wd);
            Mom[p.off] = mo_end[e];
            W[p.off] = w_end[e];
        }
    }
};

// The same for a tile that lies inside W, with most of the vector instructions gone (the fp32 MFMA pipe runs no faster than
// they leave it time: 9216 -> 4096, K = 512, 384 -> 312 us).  Only the first and the last line of a row are shared with other
// tiles, and the lanes that own quads of the one own none of the other, so that one access takes both.  The elements of a row
// before its first whole quad and behind its last are taken one by one, as in RowUpdate.  ON_LINES: rows of W and Mom start on
// lines (no shift at all).  EDGE, on lines: a tile at the edges of W, of which rows past N (then to be given) and lines past M are
// left out.  The lines are whole, so that it needs no more than two comparisons, and far fewer registers than RowUpdate: beside it
// the bf16 tiles on lines take 215 (128 x 192), 151, 124 and 76 (64 x 64) registers; beside RowUpdate 232, 203, 144, 96.
template <int ROWS, int WIDTH, int WAVES, int DEPTH, bool ON_LINES, class RowN, bool EDGE = false>
struct InnerUpdate {
    static constexpr int LINES = WIDTH / 32, GROUPS = ROWS / 8 / WAVES;       // a wavefront's groups of eight rows
    static constexpr int UNITS = GROUPS * LINES, BATCHES = (UNITS + DEPTH - 1) / DEPTH;
    static_assert(ROWS % (8 * WAVES) == 0 && WIDTH % 32 == 0, "whole lines of eight rows");
    static_assert(ON_LINES || !EDGE, "what a tile owns of a line off lines is for RowUpdate to say");
    float* W;
    float* Mom;
    RowN row_n;
    int64_t m0, M, N;
    int wave, lane, stride;
    float4 w[2][DEPTH], mo[2][DEPTH];
    float w_end[GROUPS], mo_end[GROUPS];

    __device__ __forceinline__ InnerUpdate(float* W_, float* Mom_, RowN row, int64_t m0_, int64_t M_, int wave_, int lane_,
                                           int64_t N_ = 0)
        : W(W_), Mom(Mom_), row_n(row), m0(m0_), M(M_), N(N_), wave(wave_), lane(lane_), stride(row_stride(WIDTH, ON_LINES ? 0 : M_))
    {
    }
    struct Place {
        int64_t off;                               // of this lane's quad in W
        int at;                                    // ... in the row buffer
        bool any;                                  // does the tile own all of it
    };
    __device__ __forceinline__ Place place(int u) const
    {
        const int line = u % LINES, r = (wave + WAVES * (u / LINES)) * 8 + (lane >> 3), q = 4 * (lane & 7);
        const int64_t n = row_n(r);
        Place p = {n * M + m0 + 32 * line + q, r * stride + 32 * line + q, !EDGE || (n < N && m0 + 32 * line < M)};
        if constexpr (ON_LINES) return p;
        const int shift = line_shift(W, n, M);
        p.off -= shift;
        if (line == 0) {                           // the first line, and the last in the lanes before the row begins
            const int far = q < shift ? WIDTH : 0;
            p.off += far;
            p.at += far;
            p.any = q >= shift || q + 3 < shift;
        }
        return p;
    }
    struct End {
        int64_t off;
        int at;
        bool any;
    };
    __device__ __forceinline__ End end(int e, int lane) const
    {
        const int r = (wave + WAVES * e) * 8 + (lane >> 3), i = lane & 3;
        const int64_t n = row_n(r);
        const int shift = line_shift(W, n, M), behind = shift & 3, c = lane & 4 ? WIDTH - behind + i : i;
        return {n * M + m0 + c, r * stride + shift + c, i < (lane & 4 ? behind : -shift & 3)};
    }
    template <int B>
    __device__ __forceinline__ void fetch()
    {
#pragma unroll
        for (int j = 0; j < DEPTH; ++j) {
            const int u = B * DEPTH + j;
            if (u >= UNITS) continue;
            const Place p = place(u);
            if (EDGE && !p.any) continue;
            if (ON_LINES || u % LINES > 0) {
                w[B & 1][j] = load_stream4(W + p.off);
                mo[B & 1][j] = load_stream4(Mom + p.off);
            } else if (p.any) {
                w[B & 1][j] = *reinterpret_cast<const float4*>(W + p.off);
                mo[B & 1][j] = *reinterpret_cast<const float4*>(Mom + p.off);
            }
        }
        if (!ON_LINES && B == 0 && M % 4 != 0) {
#pragma unroll
            for (int e = 0; e < GROUPS; ++e) {
                const End p = end(e, lane);
                if (!p.any) continue;
                w_end[e] = W[p.off];
                mo_end[e] = Mom[p.off];
            }
        }
    }
    __device__ __forceinline__ void update(const float* buf, int at, float4& wv, float4& mv, float lr, float mu, float wd) const
    {
        const float4 d = *reinterpret_cast<const float4*>(buf + at);
        upd(d.x, wv.x, mv.x, lr, mu, wd);
        upd(d.y, wv.y, mv.y, lr, mu, wd);
        upd(d.z, wv.z, mv.z, lr, mu, wd);
        upd(d.w, wv.w, mv.w, lr, mu, wd);
    }
    template <int B = 0>
    __device__ __forceinline__ void run(const float* buf, float lr, float mu, float wd)
    {
        if constexpr (B < BATCHES) {
            if constexpr (B + 1 < BATCHES) fetch<B + 1>();
#pragma unroll
            for (int j = 0; j < DEPTH; ++j) {
                const int u = B * DEPTH + j;
                if (u >= UNITS) continue;
                const Place p = place(u);
                if (!p.any) continue;
                float4 &wv = w[B & 1][j], &mv = mo[B & 1][j];
                update(buf, p.at, wv, mv, lr, mu, wd);
                if (ON_LINES || WIDTH < 128 || u % LINES > 0) {
                    store_stream4(Mom + p.off, mv);
                    store_stream4(W + p.off, wv);
                } else {
                    *reinterpret_cast<float4*>(Mom + p.off) = mv;
                    *reinterpret_cast<float4*>(W + p.off) = wv;
                }
            }
            if constexpr (!ON_LINES && B == 0) run_ends(buf, lr, mu, wd);
            run<B + 1>(buf, lr, mu, wd);
        }
    }
    __device__ __forceinline__ void run_ends(const float* buf, float lr, float mu, float wd)
    {
        if (M % 4 == 0) return;
#pragma unroll
        for (int e = 0; e < GROUPS; ++e) {
            const End p = end(e, anew(lane));
            if (!p.any) continue;
            upd(buf[p.at], w_end[e], mo_end[e], lr, mu, wd);
            Mom[p.off] = mo_end[e];
            W[p.off] = w_end[e];
        }
    }
};

}  // namespace psd
