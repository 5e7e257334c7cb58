// Block-based FAST interest-point detection (Section 3.1.1: the FAST
// operator with a partitioning strategy, so that the interest points are
// spread evenly over the sensed image).  Three launches:
//
//  1. strength + suppression, one 32 x 32 tile per workgroup: the image
//     tile with a 4-pixel halo in LDS; the FAST-9 corner strength V (the
//     largest threshold at which 9 contiguous pixels of the radius-3 circle
//     are all brighter, or all darker, than the centre) for the tile and a
//     1-pixel ring; then 3 x 3 non-maximum suppression with a raster-order
//     tie rule.  Kept corners are sparse: a bit mask, one 32-bit word per
//     row of a tile (from wave ballots), marks them, and their strengths go
//     to a list per tile in raster order; with its bits a mask word holds the
//     place in that list of its first corner.  (A map of the image, written
//     and read at the corners alone, moved a cache line per corner.)
//     Bound by the minima and maxima, 72 a pixel and 13 % of ring pixels
//     (they do not fuse: one a lane and cycle).
//     Only float32 subtractions and min / max are involved, so V is exact.
//  2. selection, one workgroup per block: the threads walk the block's mask
//     words, read the strengths of the set bits from the tiles' lists, and
//     each keeps the best K >= per_block corners it sees as sorted 64-bit keys
//     (strength descending, raster index within the block ascending) in
//     registers; a bitonic sort of all threads' lists in LDS (K = 1: a
//     minimum) gives the block's first per_block.
// 10000 x 10000 pixels, 71 x 71 blocks of one point: strength 580 -> 345 us
// (149 -> 84 VALU instructions a strength, four pixels a tile load, no region
// test inside it, branch-free suppression), selection 98 -> 40 us (lists instead of the map).
//  3. compaction (one workgroup): block counts prefix-summed, each block's
//     interest points copied to its place in one list.
#include <hip/hip_runtime.h>
#include <math.h>

#include <algorithm>

#include "sfoc_dev.h"
#include "sfoc_launch.h"
#include "sfoc_plan.h"
#include "sfoc_trace.h"

namespace sfoc {
namespace fast {

constexpr int kTS = 32, kHalo = 4, kIS = kTS + 2 * kHalo, kVS = kTS + 2;   // tile, image and strength sides
constexpr int kNT = 256;
constexpr int kSelNT = 256, kMaxPer = 32, kMaxBlocks = 1 << 16;
constexpr int kCompNT = 1024;

struct Region {
    int b, H, W;           // detection region rows / columns [b, size - b)
};

struct Blocks {
    int nby, nbx, per;
};

// Corners kept: no two are neighbours (of two, the later one would have to be
// larger and the earlier one not smaller), so one per 2 x 2 pixels of a tile, of
// which those at the right and bottom border may be smaller than 32 x 32.  The
// tiles' lists lie one after the other, row by row.
inline SFOC_HOST_DEVICE int64_t list_start(int64_t H, int64_t W, int64_t ta, int64_t tb) {
    const int64_t h = H - ta * kTS < kTS ? H - ta * kTS : kTS;
    return ta * (kTS / 2) * ((W + 1) / 2) + (h + 1) / 2 * (kTS / 2) * tb;
}
inline int64_t list_total(int64_t H, int64_t W) { return (H + 1) / 2 * ((W + 1) / 2); }

SFOC_DEV int bound(int lo, int n, int i, int nb) { return lo + (int)(((int64_t)i * n) / nb); }

// The radius-3 circle, clockwise from the top, as (dy, dx).  Compile-time
// constants: with the reads addressed from the 7 x 7 neighbourhood's
// top-left element, every circle read is one LDS instruction with a constant
// offset and no address arithmetic.
constexpr int kCy[16] = {-3, -3, -2, -1, 0, 1, 2, 3, 3, 3, 2, 1, 0, -1, -2, -3};
constexpr int kCx[16] = {0, 1, 2, 3, 3, 3, 2, 1, 0, -1, -2, -3, -3, -3, -2, -1};

// Three-operand minimum and maximum (one instruction each; exact).
SFOC_DEV float min3(float a, float b, float c) { return fminf(fminf(a, b), c); }
SFOC_DEV float max3(float a, float b, float c) { return fmaxf(fmaxf(a, b), c); }

// The same of two loaded values, by the instruction itself: before fminf and
// fmaxf the compiler would quiet each of the 16 loads (an instruction each).
SFOC_DEV float min2(float a, float b) {
    float r;
    asm("v_min_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
SFOC_DEV float max2(float a, float b) {
    float r;
    asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// V from the circle's raw values: subtraction rounds monotonically, so the
// minimum (maximum) over an arc of the rounded differences is the rounded
// difference of the arc's minimum (maximum), and the maximum over the arcs of
// those likewise.  The arcs from k and k + 1, k even, share the eight pixels
// k + 1 .. k + 8, four pairs: the larger of their two minima is
// min(pairs, max(p[k], p[k + 9])), 36 instructions a polarity with the pairs
// and the fold (16 arcs by three arcs of three: 40).  Finite pixels.
SFOC_DEV float strength(const float* tile, int ty, int tx) {
    const float* nb = tile + (ty - 3) * kIS + (tx - 3);
    const float c = nb[3 * kIS + 3];
    float p[16], mn[8], mx[8], lo[8], hi[8];
#pragma unroll
    for (int i = 0; i < 16; ++i) p[i] = nb[(kCy[i] + 3) * kIS + kCx[i] + 3];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        mn[j] = min2(p[2 * j + 1], p[(2 * j + 2) & 15]);
        mx[j] = max2(p[2 * j + 1], p[(2 * j + 2) & 15]);
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const float a = p[2 * j], b = p[(2 * j + 9) & 15];
        lo[j] = min3(min3(mn[j], mn[(j + 1) & 7], mn[(j + 2) & 7]), mn[(j + 3) & 7], max2(a, b));
        hi[j] = max3(max3(mx[j], mx[(j + 1) & 7], mx[(j + 2) & 7]), mx[(j + 3) & 7], min2(a, b));
    }
    const float bright = max3(max3(lo[0], lo[1], lo[2]), max3(lo[3], lo[4], lo[5]), fmaxf(lo[6], lo[7]));
    const float dark = min3(min3(hi[0], hi[1], hi[2]), min3(hi[3], hi[4], hi[5]), fminf(hi[6], hi[7]));
    return fmaxf(bright - c, c - dark);
}

// The same where a pixel of the tile is not finite: arc by arc, from the
// differences, of which minima and maxima ignore a NaN.  (A NaN pixel, or inf -
// inf, then counts neither for nor against an arc; in the form above it would be
// ignored by a maximum of two arcs' ends and leave the smaller one.)
SFOC_DEV float strength_any(const float* tile, int ty, int tx) {
    const float* nb = tile + (ty - 3) * kIS + (tx - 3);
    const float c = nb[3 * kIS + 3];
    float u[16], v = -INFINITY;
#pragma unroll
    for (int i = 0; i < 16; ++i) u[i] = nb[(kCy[i] + 3) * kIS + kCx[i] + 3] - c;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        float lo = u[k], hi = u[k];
#pragma unroll
        for (int j = 1; j < 9; ++j) {
            lo = fminf(lo, u[(k + j) & 15]);
            hi = fmaxf(hi, u[(k + j) & 15]);
        }
        v = fmaxf(v, fmaxf(lo, -hi));
    }
    return v;
}

__global__ __launch_bounds__(kNT) void strength_kernel(const float* __restrict__ img, int64_t ld, Region R,
                                                       float thr, float* __restrict__ S,
                                                       uint2* __restrict__ mask, int mask_words, int tiles_x) {
    static_assert(kTS == 32 && kNT % 64 == 0, "a wave covers two tile rows");
    __shared__ __align__(16) float tile[kIS * kIS];
    __shared__ float vs[kVS * kVS];
    __shared__ int wcount[kNT / 64];
    __shared__ int wodd[kNT / 64];   // a wave loaded a pixel that is not finite
    float zero = 0.f;                // the sum of the loaded pixels times zero
    const int t = threadIdx.x, lane = t & 63;
    const int ty0 = (blockIdx.x / tiles_x) * kTS, tx0 = (blockIdx.x % tiles_x) * kTS;
    {   // every load of the tile first, then the stores; pixels outside the
        // image (only tiles at its border have any) read as zero
        constexpr int kLoads = (kIS * kIS + kNT - 1) / kNT;
        const int y0 = ty0 - kHalo, x0 = tx0 - kHalo;
        const bool inside = y0 >= 0 && x0 >= 0 && y0 + kIS <= R.H && x0 + kIS <= R.W;
        const float* src = img + (int64_t)y0 * ld + x0;
        if (inside && (ld & 3) == 0 && ((uintptr_t)src & 15) == 0) {
            // four pixels a load: a tenth of the address arithmetic
            constexpr int kQ = kIS / 4, kQuads = kIS * kQ;
            static_assert(kIS % 4 == 0 && kQuads <= 2 * kNT, "two rounds of four pixels");
            const int e1 = min(t + kNT, kQuads - 1);
            const float4 v0 = *reinterpret_cast<const float4*>(src + (int64_t)(t / kQ) * ld + 4 * (t % kQ));
            const float4 v1 = *reinterpret_cast<const float4*>(src + (int64_t)(e1 / kQ) * ld + 4 * (e1 % kQ));
            zero = fmaf(v0.x, 0.f, fmaf(v0.y, 0.f, fmaf(v0.z, 0.f, v0.w * 0.f))) +
                   fmaf(v1.x, 0.f, fmaf(v1.y, 0.f, fmaf(v1.z, 0.f, v1.w * 0.f)));
            reinterpret_cast<float4*>(tile)[t] = v0;
            if (t + kNT < kQuads) reinterpret_cast<float4*>(tile)[t + kNT] = v1;
        } else {
            float v[kLoads];
#pragma unroll
            for (int k = 0; k < kLoads; ++k) {
                const int e = min(t + k * kNT, kIS * kIS - 1), a = e / kIS, c = e - a * kIS;
                const int y = y0 + a, x = x0 + c;
                v[k] = (y >= 0 && y < R.H && x >= 0 && x < R.W) ? img[(int64_t)y * ld + x] : 0.f;
            }
#pragma unroll
            for (int k = 0; k < kLoads; ++k) {
                zero = fmaf(v[k], 0.f, zero);
                if (t + k * kNT < kIS * kIS) tile[t + k * kNT] = v[k];
            }
        }
    }
    const uint64_t odd = __ballot(!(zero == 0.f));
    if (lane == 0) wodd[t >> 6] = odd != 0;
    __syncthreads();
    int any = 0;
#pragma unroll
    for (int w = 0; w < kNT / 64; ++w) any |= wodd[w];
    const bool finite = __builtin_amdgcn_readfirstlane(any) == 0;
    // strengths of the tile and a 1-pixel ring; -inf outside the region (which
    // only tiles at its border reach)
    if (finite && ty0 - 1 >= R.b && tx0 - 1 >= R.b && ty0 + kTS < R.H - R.b && tx0 + kTS < R.W - R.b) {
        for (int e = t; e < kVS * kVS; e += kNT) {
            const int a = e / kVS, c = e - a * kVS;
            vs[e] = strength(tile, a + kHalo - 1, c + kHalo - 1);
        }
    } else {
        for (int e = t; e < kVS * kVS; e += kNT) {
            const int a = e / kVS, c = e - a * kVS;
            const int y = ty0 - 1 + a, x = tx0 - 1 + c;
            const bool in = y >= R.b && y < R.H - R.b && x >= R.b && x < R.W - R.b;
            vs[e] = !in ? -INFINITY
                        : finite ? strength(tile, a + kHalo - 1, c + kHalo - 1)
                                 : strength_any(tile, a + kHalo - 1, c + kHalo - 1);
        }
    }
    __syncthreads();
    // Thread t suppresses column t % 32 of rows 4 (t / 32) .. + 3, so a wave
    // covers two groups of four rows; every lane takes part in the ballots.
    // Neighbours before in raster order: strictly smaller; after: not larger.
    {
        constexpr int kRows = kTS * kTS / kNT;
        const int c = t % kTS, a0 = (t / kTS) * kRows;
        const float* q = vs + a0 * kVS + c;   // the 3 x 3 block of the first pixel, from its top left
        float l[kRows + 2], m[kRows + 2], r[kRows + 2];
#pragma unroll
        for (int k = 0; k < kRows + 2; ++k) {
            l[k] = q[k * kVS];
            m[k] = q[k * kVS + 1];
            r[k] = q[k * kVS + 2];
        }
        bool keep[kRows];
        uint64_t bal[kRows];
        int before_lo = 0, before_hi = 0;   // kept corners of the wave's first and second group
#pragma unroll
        for (int k = 0; k < kRows; ++k) {
            const float v = m[k + 1];
            const float before = max2(max3(l[k], m[k], r[k]), l[k + 1]);
            const float after = max2(max3(l[k + 2], m[k + 2], r[k + 2]), r[k + 1]);
            // (a strength outside the region is -inf, below any threshold)
            keep[k] = v > thr && v > before && v >= after;
            bal[k] = __ballot(keep[k]);
            before_lo += __popc((uint32_t)bal[k]);
            before_hi += __popc((uint32_t)(bal[k] >> 32));
        }
        if (lane == 0) wcount[t >> 6] = before_lo + before_hi;
        __syncthreads();
        float* const list = S + list_start(R.H, R.W, ty0 / kTS, tx0 / kTS);
        int base = 0;   // kept corners of the tile's rows before this thread's group
        for (int w = 0; w < kNT / 64; ++w) base += w < (t >> 6) ? wcount[w] : 0;
        if (lane & 32) base += before_lo;
#pragma unroll
        for (int k = 0; k < kRows; ++k) {
            const int y = ty0 + a0 + k;
            const uint32_t bits = (uint32_t)(bal[k] >> (lane & 32));
            if (keep[k]) list[base + __popc(bits & ((1u << c) - 1u))] = m[k + 1];
            if (c == 0 && y < R.H) mask[(int64_t)y * mask_words + tx0 / kTS] = make_uint2(bits, (uint32_t)base);
            base += __popc(bits);
        }
    }
}

// Keys: strength (>= 0 for kept corners) descending, then the raster index
// within the block ascending; empty = all ones.
SFOC_DEV uint64_t make_key(float v, uint32_t e) {
    const uint32_t ord = __float_as_uint(v) | 0x80000000u;   // order-preserving for v >= 0
    return ((uint64_t)(~ord) << 32) | e;
}

template <int K>
__global__ __launch_bounds__(kSelNT) void select_kernel(const float* __restrict__ S,
                                                        const uint2* __restrict__ mask, int mask_words, Region R,
                                                        Blocks B, int32_t* __restrict__ bips,
                                                        float* __restrict__ bsc, int32_t* __restrict__ bcnt) {
    extern __shared__ uint64_t keys[];   // kSelNT * K
    const int t = threadIdx.x;
    const int bi = blockIdx.x / B.nbx, bj = blockIdx.x - bi * B.nbx;
    const int Hd = max(0, R.H - 2 * R.b), Wd = max(0, R.W - 2 * R.b);
    const int y0 = bound(R.b, Hd, bi, B.nby), y1 = bound(R.b, Hd, bi + 1, B.nby);
    const int x0 = bound(R.b, Wd, bj, B.nbx), x1 = bound(R.b, Wd, bj + 1, B.nbx);
    const int bw = x1 - x0;
    // mask words of the block: rows y0..y1-1, words x0/32 .. (x1-1)/32
    const int w0 = x0 / 32, nw = bw > 0 ? (x1 - 1) / 32 - w0 + 1 : 0;
    const int nwords = (y1 - y0) * nw;
    uint64_t best[K];
#pragma unroll
    for (int i = 0; i < K; ++i) best[i] = ~0ull;
    constexpr int kU = 4;   // mask loads in flight per thread
    for (int q0 = t; q0 < nwords; q0 += kU * kSelNT) {
        uint2 m[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int q = q0 + u * kSelNT;
            m[u] = make_uint2(0u, 0u);
            if (q < nwords) {
                const int a = q / nw, wi = q - a * nw;
                const int xw = 32 * (w0 + wi);
                const uint2 e = mask[(int64_t)(y0 + a) * mask_words + w0 + wi];
                uint32_t bits = e.x;
                if (xw < x0) bits &= ~0u << (x0 - xw);                              // columns before the block
                if (x1 - xw < 32) bits &= (1u << (x1 - xw)) - 1u;                   // columns after it
                // with the place of the first corner that is left in the tile's list
                m[u] = make_uint2(bits, bits ? e.y + __popc(e.x & ((1u << (__ffs(bits) - 1)) - 1u)) : 0u);
            }
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            uint32_t bits = m[u].x;
            if (!bits) continue;
            const int q = q0 + u * kSelNT;
            const int a = q / nw, wi = q - a * nw, xw = 32 * (w0 + wi);
            const float* list = S + list_start(R.H, R.W, (y0 + a) / kTS, w0 + wi) + m[u].y;
            while (bits) {
                const int x = xw + __ffs(bits) - 1;
                bits &= bits - 1u;
                const float v = *list++;
                const uint64_t k = make_key(v, (uint32_t)a * (uint32_t)bw + (uint32_t)(x - x0));
                if (k >= best[K - 1]) continue;
                // sorted insertion with compile-time indices
#pragma unroll
                for (int i = K - 1; i > 0; --i) best[i] = k < best[i - 1] ? best[i - 1] : (k < best[i] ? k : best[i]);
                best[0] = k < best[0] ? k : best[0];
            }
        }
    }
    if constexpr (K == 1) {   // one point a block: the smallest key, a butterfly and then the waves
        uint64_t k = best[0];
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const uint64_t o = __shfl_xor(k, d, 64);
            k = o < k ? o : k;
        }
        if ((t & 63) == 0) keys[t >> 6] = k;
        __syncthreads();
        if (t == 0)
            for (int w = 1; w < kSelNT / 64; ++w) keys[0] = keys[w] < keys[0] ? keys[w] : keys[0];
    } else {
#pragma unroll
    for (int i = 0; i < K; ++i) keys[t * K + i] = best[i];
    }
    __syncthreads();
    // bitonic sort, ascending, of kSelNT * K keys
    constexpr int N = K == 1 ? 1 : kSelNT * K;
    for (int size = 2; size <= N; size <<= 1) {
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            for (int i = t; i < N / 2; i += kSelNT) {
                const int lo = 2 * i - (i & (stride - 1));
                const int hi = lo + stride;
                const bool up = (lo & size) == 0;
                const uint64_t a = keys[lo], b = keys[hi];
                if ((a > b) == up) {
                    keys[lo] = b;
                    keys[hi] = a;
                }
            }
            __syncthreads();
        }
    }
    const int base = blockIdx.x * B.per;
    if (t < B.per) {
        const uint64_t k = keys[t];
        if (k != ~0ull) {
            const uint32_t e = (uint32_t)k;
            const int a = (int)(e / (uint32_t)bw), c = (int)(e - (uint32_t)a * (uint32_t)bw);
            bips[2 * (base + t)] = y0 + a;
            bips[2 * (base + t) + 1] = x0 + c;
            bsc[base + t] = __uint_as_float(~(uint32_t)(k >> 32) & 0x7fffffffu);
        }
    }
    if (t == 0) {
        int n = 0;
        for (int i = 0; i < B.per; ++i) n += keys[i] != ~0ull;
        bcnt[blockIdx.x] = n;
    }
}

__global__ __launch_bounds__(kCompNT) void compact_kernel(const int32_t* __restrict__ bips,
                                                          const float* __restrict__ bsc,
                                                          const int32_t* __restrict__ bcnt, int nblocks, int per,
                                                          int32_t* __restrict__ ips, float* __restrict__ scores,
                                                          int32_t* __restrict__ counts, int32_t* __restrict__ n_out) {
    __shared__ int scan[kCompNT];
    const int t = threadIdx.x;
    const int chunk = (nblocks + kCompNT - 1) / kCompNT;
    const int lo = min(nblocks, t * chunk), hi = min(nblocks, lo + chunk);
    int c = 0;
    for (int b = lo; b < hi; ++b) c += bcnt[b];
    scan[t] = c;
    __syncthreads();
    for (int d = 1; d < kCompNT; d <<= 1) {
        const int v = t >= d ? scan[t - d] : 0;
        __syncthreads();
        scan[t] += v;
        __syncthreads();
    }
    int o = scan[t] - c;
    for (int b = lo; b < hi; ++b) {
        const int n = bcnt[b];
        if (counts) counts[b] = n;
        for (int i = 0; i < n; ++i) {
            ips[2 * (o + i)] = bips[2 * (b * per + i)];
            ips[2 * (o + i) + 1] = bips[2 * (b * per + i) + 1];
            if (scores) scores[o + i] = bsc[b * per + i];
        }
        o += n;
    }
    if (t == kCompNT - 1) *n_out = scan[t];
}

struct Layout {
    size_t smap, mask, bips, bsc, bcnt, total;
    int mask_words;
};
Layout layout(int64_t H, int64_t W, int nblocks, int per) {
    Layout L;
    size_t o = 0;
    auto take = [&](size_t bytes) {
        const size_t at = o;
        o += align_up(std::max<size_t>(bytes, 1), 256);
        return at;
    };
    L.mask_words = (int)((W + kTS - 1) / kTS);
    // (an image of six rows or columns or fewer has no region)
    const bool any = H > 6 && W > 6;
    L.smap = take(any ? sizeof(float) * (size_t)list_total(H, W) : 0);
    L.mask = take(any ? sizeof(uint2) * (size_t)H * L.mask_words : 0);
    L.bips = take(sizeof(int32_t) * 2 * (size_t)nblocks * per);
    L.bsc = take(sizeof(float) * (size_t)nblocks * per);
    L.bcnt = take(sizeof(int32_t) * (size_t)nblocks);
    // The size asked for is a strength per pixel and a mask word per 32, which
    // callers may have stored: the lists and the wider words always fit (from
    // seven rows and columns on, 4 bytes per 2 x 2 pixels and 8 per 32 pixels of a
    // row are no more than 4 bytes per pixel and 4 per 32).
    const size_t map = align_up(sizeof(float) * (size_t)H * (size_t)W, 256) +
                       align_up(sizeof(uint32_t) * (size_t)H * L.mask_words, 256);
    L.total = map + (o - L.bips);
    return L;
}

int check(int64_t H, int64_t W, int nby, int nbx, int per) {
    if (H < 1 || W < 1 || nby < 1 || nbx < 1 || per < 1) return SFOC_E_INVALID_ARG;
    if (H > (1 << 20) || W > (1 << 20) || H * W > ((int64_t)1 << 32) || per > kMaxPer ||
        (int64_t)nby * nbx > kMaxBlocks)
        return SFOC_E_UNSUPPORTED;
    return SFOC_OK;
}

template <int K>
hipError_t launch_select(const float* S, const uint2* mask, int mask_words, Region R, Blocks B, int32_t* bips,
                         float* bsc, int32_t* bcnt, hipStream_t st) {
    const size_t lds = sizeof(uint64_t) * kSelNT * K;
    hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(&select_kernel<K>), lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(select_kernel<K>, dim3(B.nby * B.nbx), dim3(kSelNT), lds, st, S, mask, mask_words, R, B, bips,
                       bsc, bcnt);
    return hipGetLastError();
}

}  // namespace fast
}  // namespace sfoc

using namespace sfoc;

extern "C" int sfoc_fast_workspace(int64_t H, int64_t W, int32_t nby, int32_t nbx, int32_t per_block, size_t* bytes) {
    const int rc = fast::check(H, W, nby, nbx, per_block);
    if (rc != SFOC_OK) return rc;
    if (!bytes) return SFOC_E_INVALID_ARG;
    *bytes = fast::layout(H, W, nby * nbx, per_block).total;
    return SFOC_OK;
}

extern "C" int sfoc_detect_ips(const float* img, int64_t H, int64_t W, int64_t ld, float threshold, int32_t margin,
                               int32_t nby, int32_t nbx, int32_t per_block, int32_t* ips, float* scores,
                               int32_t* counts, int32_t* n_out, void* ws, size_t ws_bytes, void* stream) {
    using namespace fast;
    const int rc = check(H, W, nby, nbx, per_block);
    if (rc != SFOC_OK) return rc;
    if (!img || !ips || !n_out || !ws || ld < W || margin < 0 || !(threshold >= 0.f) || !isfinite(threshold))
        return SFOC_E_INVALID_ARG;
    const int nblocks = nby * nbx;
    const Layout L = layout(H, W, nblocks, per_block);
    if (ws_bytes < L.total) return SFOC_E_WORKSPACE;
    char* w = (char*)ws;
    float* S = (float*)(w + L.smap);
    uint2* mask = (uint2*)(w + L.mask);
    int32_t* bips = (int32_t*)(w + L.bips);
    float* bsc = (float*)(w + L.bsc);
    int32_t* bcnt = (int32_t*)(w + L.bcnt);
    Region R;
    R.b = std::max(3, margin);
    R.H = (int)H;
    R.W = (int)W;
    Blocks B;
    B.nby = nby;
    B.nbx = nbx;
    B.per = per_block;
    hipStream_t st = (hipStream_t)stream;
    const int tiles_x = (int)((W + kTS - 1) / kTS), tiles_y = (int)((H + kTS - 1) / kTS);
    trace_begin(st, SFOC_K_FAST);
    // (without a region the blocks are empty and the selection reads nothing)
    if (H - R.b > R.b && W - R.b > R.b)
        hipLaunchKernelGGL(strength_kernel, dim3(tiles_x * tiles_y), dim3(kNT), 0, st, img, ld, R, threshold, S, mask,
                           L.mask_words, tiles_x);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) {
        const int K = per_block <= 1 ? 1 : per_block <= 2 ? 2 : per_block <= 4 ? 4 : per_block <= 8 ? 8
                    : per_block <= 16 ? 16 : 32;
        switch (K) {
            case 1: e = launch_select<1>(S, mask, L.mask_words, R, B, bips, bsc, bcnt, st); break;
            case 2: e = launch_select<2>(S, mask, L.mask_words, R, B, bips, bsc, bcnt, st); break;
            case 4: e = launch_select<4>(S, mask, L.mask_words, R, B, bips, bsc, bcnt, st); break;
            case 8: e = launch_select<8>(S, mask, L.mask_words, R, B, bips, bsc, bcnt, st); break;
            case 16: e = launch_select<16>(S, mask, L.mask_words, R, B, bips, bsc, bcnt, st); break;
            default: e = launch_select<32>(S, mask, L.mask_words, R, B, bips, bsc, bcnt, st); break;
        }
    }
    if (e == hipSuccess) {
        hipLaunchKernelGGL(compact_kernel, dim3(1), dim3(kCompNT), 0, st, bips, bsc, bcnt, nblocks, per_block, ips,
                           scores, counts, n_out);
        e = hipGetLastError();
    }
    trace_end(st, SFOC_K_FAST);
    return hip_status(e);
}
