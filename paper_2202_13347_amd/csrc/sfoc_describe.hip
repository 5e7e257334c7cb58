// Dense SFOC descriptor (Section 2.1, Eq. 1-7) as one fused gfx950 kernel
// per 32x32 output tile, plus the float64 integral-image scans (Eq. 14-16).
//
// Per tile, everything stays in LDS (describe_kernel, any parameters; the
// shapes in use, K = 1 at rates 1, 2, 3, have describe_k1_kernel):
//   1. the input tile plus a halo of R (largest kernel radius) + Q (dilated
//      smoothing reach), read once from HBM with reflect-101 indices;
//   2. for each distinct sigma, a separable row pass (1-D Gaussian g, first
//      derivative d, second derivative dd) and a column pass that adds the
//      five basis responses Gx, Gy, Gxx, Gyy, Gxy * I into per-pixel sums
//      over sigma (sum over scales commutes with steering: both linear);
//   3. per group of channels: steer (Eq. 4/6 and the directional reading of
//      Eq. 7), rectify, write to LDS, then the dilated Gaussian smoothing
//      (rates dil[], summed) into registers;
//   4. per-order L2 normalisation, rounding to the storage type, one
//      coalesced store per channel plane, and the per-pixel channel sums
//      sum_c g and sum_c g^2 (float64, from the stored values) for the
//      integral images.
#include "sfoc_dev.h"
#include "sfoc_launch.h"
#include "sfoc_trace.h"

namespace sfoc {

constexpr int kTS = kDescribeTile;   // output tile side
constexpr int kNT = 256;      // threads per tile
constexpr int kRun = 4;       // outputs per thread along a run
constexpr int kPXT = kTS * kTS / kNT;   // output pixels per thread (one run of 4)
static_assert(kPXT == kRun, "one horizontal run of outputs per thread");

// LDS geometry of one tile.  Every side is padded to a multiple of kRun so
// runs never straddle a row; padded rows and columns hold harmless values
// that no output reads.
struct DescribeGeom {
    int BSP;    // basis / channel side incl. the smoothing halo Q, padded
    int ISX;    // image-region side (BSP + 2R)
    int nrun;   // runs per basis row (BSP / kRun)
    int BPP;    // LDS row pitch of the basis / channel / row-pass maps (odd)
    int IPP;    // LDS row pitch of the image region (odd)
    size_t bytes;
};

static DescribeGeom describe_geom(const DescribeConsts& c, int CG) {
    DescribeGeom g;
    g.BSP = (kTS + 2 * c.Q + kRun - 1) / kRun * kRun;
    g.ISX = g.BSP + 2 * c.R;
    g.nrun = g.BSP / kRun;
    // Odd pitches spread the rows of a wave's accesses over all LDS banks.
    g.BPP = g.BSP | 1;
    g.IPP = g.ISX | 1;
    // Phase 2 holds the image region and the row-pass maps; phase 3 the five
    // basis maps (over the same memory) and CG steered channels.
    const size_t img = (size_t)g.ISX * g.IPP;
    const size_t row = 3 * (size_t)g.ISX * g.BPP;
    const size_t bb = (size_t)g.BSP * g.BPP;
    const size_t p2 = img + row, p3 = (5 + (size_t)CG) * bb;
    g.bytes = (p2 > p3 ? p2 : p3) * sizeof(float);
    return g;
}

// LDS geometry of the K = 1, rates 1-3 tile (Q = 3): basis and channel maps of
// 38 x 38 pixels, nothing padded but the pitches.
constexpr int kB = kTS + 6;           // side of the basis and channel maps
constexpr int kCP = kB + 1;           // their pitch (odd)
constexpr int kPix = (kB * kCP + kNT - 1) / kNT;   // map elements per thread, in linear order (6)
constexpr int kCM = kPix * kNT;       // floats of a map
constexpr int kRP = kB + 3;           // pitch of the row-pass maps: ten runs of kRun (odd)
constexpr int kCRun = 3;              // rows of a column-pass run
constexpr int kCRuns = (kB + kCRun - 1) / kCRun;                 // 13
constexpr int kCOwn = (kCRuns * kB + kNT - 1) / kNT;             // column-pass runs per thread (2)
static_assert(kRP % 2 == 1 && kCP % 2 == 1 && kRP >= (kB + kRun - 1) / kRun * kRun, "pitches");
static_assert(kCRuns * kCRun * kCP <= kCM, "the rows of the last run stay inside a map");
static size_t describe_k1_lds(int R) {
    const size_t side = kB + 2 * R;
    // (the last column run reads one row past its map)
    const size_t p2 = side * (side | 1) + (3 * side + 1) * kRP, p3 = 5 * (size_t)kCM;
    return (p2 > p3 ? p2 : p3) * sizeof(float);
}

// Dilated Gaussian smoothing of one channel for a horizontal run of kRun
// outputs, base 3x3 (K = 1) at rates 1, 2, 3.  With weights wc (centre), we
// (edge) and wk (corner) shared by the three rates,
//   out = 3 wc I(p) + we sum_r E_r(p) + wk sum_r C_r(p),
// where E_r / C_r sum the 4 edge / 4 corner neighbours at distance r.  Per
// rate, the vertical pair sums S_r(x) = I(y - r, x) + I(y + r, x) over the
// run's columns widened by r give both: E_r = S_r(x) + I(y, x - r) +
// I(y, x + r) and C_r = S_r(x - r) + S_r(x + r).
// The run's first output is element i0 of map s (pitch P).  Reads are
// addressed from the neighbourhood's top-left element, whose index is kept
// opaque to the compiler: the address then stays in one register and each
// read's constant offset (at most 6 P + kRun + 5 elements) fits the LDS
// instruction's offset field instead of costing an address add.
SFOC_DEV void smooth_run_k1_123(const float* s, int i0, int P, float wc, float we, float wk, float out[kRun]) {
    int b = i0 - 3 * P - 3;
    asm volatile("" : "+v"(b));
    const float* n = s + b;
    float c[kRun + 6];
#pragma unroll
    for (int q = 0; q < kRun + 6; ++q) c[q] = n[3 * P + q];
    float e[kRun], k[kRun];
#pragma unroll
    for (int r = 1; r <= 3; ++r) {
        // one rate's reads in flight at a time keeps registers for the
        // 4 x z accumulators the caller holds
        __builtin_amdgcn_sched_barrier(0);
        float S[kRun + 6];
#pragma unroll
        for (int q = 0; q < kRun + 2 * r; ++q) S[q] = n[(3 - r) * P + 3 - r + q] + n[(3 + r) * P + 3 - r + q];
#pragma unroll
        for (int j = 0; j < kRun; ++j) {
            const float ej = S[j + r] + (c[j + 3 - r] + c[j + 3 + r]);
            const float kj = S[j] + S[j + 2 * r];
            e[j] = r == 1 ? ej : e[j] + ej;
            k[j] = r == 1 ? kj : k[j] + kj;
        }
    }
    const float wc3 = 3.f * wc;
#pragma unroll
    for (int j = 0; j < kRun; ++j) out[j] = fmaf(we, e[j], fmaf(wk, k[j], wc3 * c[j + 3]));
}

// Row pass for a horizontal run of kRun outputs with radius RHO: g, d, dd
// taps paired symmetrically, so odd responses of constant input are exactly
// zero.  p points at the first output's centre.  Correlation form of the
// convolution: out(x) = sum_k t(-k) I(x + k) -> odd taps act on
// I(x - k) - I(x + k).  USE: the orders that have this sigma (bit 0 the first,
// which needs no dd; bit 1 the second).
template <int RHO, int USE = 3>
SFOC_DEV void row_run(const float* p, const float* tg, const float* td, const float* tdd, float og[kRun],
                      float od[kRun], float odd[kRun]) {
    float x[2 * RHO + kRun];
#pragma unroll
    for (int q = 0; q < 2 * RHO + kRun; ++q) x[q] = p[q - RHO];
#pragma unroll
    for (int j = 0; j < kRun; ++j) {
        const float c = x[j + RHO];
        float g = tg[0] * c, dd = USE & 2 ? tdd[0] * c : 0.f, d = 0.f;
#pragma unroll
        for (int k = 1; k <= RHO; ++k) {
            const float l = x[j + RHO - k], r = x[j + RHO + k];
            const float sm = l + r, df = l - r;
            g = fmaf(tg[k], sm, g);
            if (USE & 2) dd = fmaf(tdd[k], sm, dd);
            d = fmaf(td[k], df, d);
        }
        og[j] = g;
        od[j] = d;
        odd[j] = dd;
    }
}

// Even (te) and odd (to) column taps on one map for a vertical run of RUN
// outputs; the first output's centre is element i0 of map s (pitch P).  The
// top element's index is kept opaque to the compiler, so the reads share one
// base register and fold their row offsets into the LDS instructions where
// those fit.
template <int RHO, int RUN = kRun>
SFOC_DEV void col_run(const float* s, int i0, int P, const float* te, const float* to, float ev[RUN],
                      float od[RUN]) {
    int b = i0 - RHO * P;
    asm volatile("" : "+v"(b));
    const float* n = s + b;
    float x[2 * RHO + RUN];
#pragma unroll
    for (int q = 0; q < 2 * RHO + RUN; ++q) x[q] = n[q * P];
#pragma unroll
    for (int j = 0; j < RUN; ++j) {
        const float c = x[j + RHO];
        float e = te ? te[0] * c : 0.f, d = 0.f;
#pragma unroll
        for (int k = 1; k <= RHO; ++k) {
            const float l = x[j + RHO - k], r = x[j + RHO + k];
            if (te) e = fmaf(te[k], l + r, e);
            if (to) d = fmaf(to[k], l - r, d);
        }
        ev[j] = e;
        od[j] = d;
    }
}

// Any radius: the same sums with taps read pairwise from LDS.
SFOC_DEV void row_run_any(const float* p, int rho, const float* tg, const float* td, const float* tdd,
                          float og[kRun], float od[kRun], float odd[kRun]) {
#pragma unroll
    for (int j = 0; j < kRun; ++j) {
        const float c = p[j];
        float g = tg[0] * c, dd = tdd[0] * c, d = 0.f;
        for (int k = 1; k <= rho; ++k) {
            const float l = p[j - k], r = p[j + k];
            g = fmaf(tg[k], l + r, g);
            dd = fmaf(tdd[k], l + r, dd);
            d = fmaf(td[k], l - r, d);
        }
        og[j] = g;
        od[j] = d;
        odd[j] = dd;
    }
}
template <int RUN = kRun>
SFOC_DEV void col_run_any(const float* p, int P, int rho, const float* te, const float* to, float ev[RUN],
                          float od[RUN]) {
#pragma unroll
    for (int j = 0; j < RUN; ++j) {
        const float c = p[j * P];
        float e = te ? te[0] * c : 0.f, d = 0.f;
        for (int k = 1; k <= rho; ++k) {
            const float l = p[(j - k) * P], r = p[(j + k) * P];
            if (te) e = fmaf(te[k], l + r, e);
            if (to) d = fmaf(to[k], l - r, d);
        }
        ev[j] = e;
        od[j] = d;
    }
}

#define SFOC_RADIUS_SWITCH(rho, CALL_T, CALL_ANY) \
    switch (rho) {                                \
        case 1: CALL_T(1); break;                 \
        case 2: CALL_T(2); break;                 \
        case 3: CALL_T(3); break;                 \
        case 4: CALL_T(4); break;                 \
        case 5: CALL_T(5); break;                 \
        case 6: CALL_T(6); break;                 \
        case 7: CALL_T(7); break;                 \
        case 8: CALL_T(8); break;                 \
        case 9: CALL_T(9); break;                 \
        case 10: CALL_T(10); break;               \
        case 11: CALL_T(11); break;               \
        case 12: CALL_T(12); break;               \
        default: CALL_ANY; break;                 \
    }

// The row sums, column sums and total of a tile that is not described, set
// to zero (the layout of the describe kernel's aggregate output).
SFOC_DEV void zero_tile_aggregates(const DescribeJob& J, int ty0, int tx0) {
    const IntegAgg ag = integ_agg(J.H, J.W);
    const int t = threadIdx.x, ta = ty0 / kTS, tb = tx0 / kTS;
    if (t < 2 * kTS) {
        const int q = t / kTS, i = t % kTS;
        if (ty0 + i < J.H) J.agg[(q ? ag.rs2 : ag.rs1) + tb * (int64_t)J.H + ty0 + i] = 0.0;
        if (tx0 + i < J.W) J.agg[(q ? ag.cs2 : ag.cs1) + ta * (int64_t)J.W + tx0 + i] = 0.0;
        if (i == 0) J.agg[(q ? ag.tt2 : ag.tt1) + ta * ag.ntx + tb] = 0.0;
    }
}

// The workgroup's entry {job, tile row origin, tile column origin, what} of the
// table, or of the image's tiles where there is none.  Workgroups are dealt to the
// eight XCDs in turn; renumbered so that each XCD takes a contiguous run of tiles,
// whose overlapping input halos then meet in one L2.
__device__ __forceinline__ int4 tile_entry(const int4* __restrict__ tiles, const uint8_t* __restrict__ tmask) {
    const int nblk = (int)(gridDim.x * gridDim.y), q8 = nblk / 8 * 8;
    const int id = (int)(blockIdx.y * gridDim.x + blockIdx.x);
    const int k = id < q8 ? (id % 8) * (q8 / 8) + id / 8 : id;
    if (tiles) return tiles[k];
    return make_int4(0, (int)(k / gridDim.x) * kTS, (int)(k % gridDim.x) * kTS, tmask ? 2 : 0);
}
// Without a job table every entry is of `single`, and a negative job is an empty
// slot that the whole workgroup skips.  what = 1: a grid tile that nothing reads,
// whose integral-image aggregates are set to zero (the box sums over the tiles that
// are described stay exact); what = 2: a grid tile that is described if the mask
// marks it.
__device__ __forceinline__ bool tile_unread(const DescribeJob& J, const int4& e, const uint8_t* __restrict__ tmask) {
    return e.w == 1 || (e.w == 2 && !tmask[(e.y / kTS) * ((J.W + kTS - 1) / kTS) + e.z / kTS]);
}

// The square input region of a tile (side `side`, top-left pixel (y0, x0),
// reflect-101 borders) into simg (pitch P): kU rows' loads are issued before any
// of their LDS stores.
template <int kU>
__device__ __forceinline__ void load_region(const DescribeJob& J, int y0, int x0, int side, float* simg, int P) {
    const float* __restrict__ img = J.img;
    const int t = threadIdx.x, H = J.H, W = J.W;
    const int64_t ld = J.ld;
    const bool inside = y0 >= 0 && x0 >= 0 && y0 + side <= H && x0 + side <= W;
    constexpr int kRows = kNT / 64;
    for (int b = t % 64; b < side; b += 64) {
        const int gx = inside ? x0 + b : reflect101(x0 + b, W);
        for (int a0 = t / 64; a0 < side; a0 += kRows * kU) {
            float v[kU];
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const int a = a0 + u * kRows;
                v[u] = 0.f;
                if (a < side) {
                    const int gy = inside ? y0 + a : reflect101(y0 + a, H);
                    v[u] = img[(int64_t)gy * ld + gx];
                }
            }
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const int a = a0 + u * kRows;
                if (a < side) simg[a * P + b] = v[u];
            }
        }
    }
}

// What a thread stores: a run of kRun pixels of one row.  Each thread stores
// its run of a channel as one vector (8 threads cover a 128-byte row segment),
// so every store instruction writes whole cache lines; unaligned widths, tiles
// whose column origin is not a multiple of kRun and the right edge fall back
// to scalar stores.  The channel sums for the integral images (d1, d2)
// accumulate in channel order.
struct RunOut {
    int64_t plane, off0;
    int gy, gx0, W;
    bool row, full;    // the run has a pixel in the image; it can be one vector
    double d1[kRun], d2[kRun];
};
__device__ __forceinline__ void init_run(RunOut& O, const DescribeJob& J, const DescribeConsts& C, int ty0, int tx0) {
    const int t = threadIdx.x;
    O.plane = (int64_t)J.H * J.W;
    O.W = J.W;
    O.gy = ty0 + t / (kTS / kRun);
    O.gx0 = tx0 + (t % (kTS / kRun)) * kRun;
    const size_t align = C.dtype == SFOC_DTYPE_F32 ? 15 : 7;
    O.full = (J.W & (kRun - 1)) == 0 && (O.gx0 & (kRun - 1)) == 0 && ((uintptr_t)J.desc & align) == 0 &&
             O.gx0 + kRun <= J.W;
    O.row = O.gy < J.H && O.gx0 < J.W;
    O.off0 = (int64_t)O.gy * J.W + O.gx0;
#pragma unroll
    for (int j = 0; j < kRun; ++j) O.d1[j] = O.d2[j] = 0.0;
}

// Channels [lo, hi) of acc, normalised, rounded to type DT and stored in a form
// (kEdge, kWhole, kVector: the run reaches past the row's end, all of it lies in the
// image, it is one vector), and their channel sums.
enum { kEdge, kWhole, kVector };
template <int Z, int DT, int FORM>
__device__ __forceinline__ void emit_channels(const float (&acc)[Z][kRun], const float (&inv)[kRun], int lo, int hi,
                                              int c0, void* __restrict__ desc, bool sums, RunOut& O) {
#pragma unroll
    for (int c = 0; c < Z; ++c) {
        if (c < lo || c >= hi) continue;
        float v[kRun];
#pragma unroll
        for (int j = 0; j < kRun; ++j) {
            v[j] = acc[c][j] * inv[j];
            // (rounded to float32 first: the compiler would fuse the conversion, for
            // the store or for the sums alone)
            if (DT == SFOC_DTYPE_F16) asm("" : "+v"(v[j]));
        }
        if constexpr (DT == SFOC_DTYPE_F32) {
            float* dst = (float*)desc + (c0 + c) * O.plane + O.off0;
            if constexpr (FORM == kVector) {
                *(float4*)dst = make_float4(v[0], v[1], v[2], v[3]);
            } else {
#pragma unroll
                for (int j = 0; j < kRun; ++j)
                    if (FORM == kWhole || O.gx0 + j < O.W) dst[j] = v[j];
            }
        } else {
            uint16_t q[kRun];
#pragma unroll
            for (int j = 0; j < kRun; ++j) {
                q[j] = DT == SFOC_DTYPE_BF16 ? f32_to_bf16_bits(v[j]) : f32_to_f16_bits(v[j]);
                v[j] = DT == SFOC_DTYPE_BF16 ? bf16_bits_to_f32(q[j]) : f16_bits_to_f32(q[j]);
            }
            uint16_t* dst = (uint16_t*)desc + (c0 + c) * O.plane + O.off0;
            if constexpr (FORM == kVector) {
                *(ushort4*)dst = make_ushort4(q[0], q[1], q[2], q[3]);
            } else {
#pragma unroll
                for (int j = 0; j < kRun; ++j)
                    if (FORM == kWhole || O.gx0 + j < O.W) dst[j] = q[j];
            }
        }
        if (sums) {
#pragma unroll
            for (int j = 0; j < kRun; ++j) {
                const double dv = (double)v[j];
                O.d1[j] += dv;
                O.d2[j] = fma(dv, dv, O.d2[j]);
            }
        }
    }
}

// One order block, channels [lo, hi) of acc: normalisation, rounding, store
// (channel c goes to plane c0 + c), channel sums.  Type and form are chosen once
// and not per channel, where their branches cost more than the stores: 2048 x 2048,
// FP16, without integrals 151 us with them inside, 144 us so; 2045 x 2047, FP32,
// whose runs check every pixel against the row's end there, 176 and 152 us.
template <int Z>
__device__ __forceinline__ void emit_block(const float (&acc)[Z][kRun], int lo, int hi, int c0, void* __restrict__ desc, bool sums,
                         const DescribeConsts& C, RunOut& O) {
    float inv[kRun];
#pragma unroll
    for (int j = 0; j < kRun; ++j) {
        float s2 = 0.f;
#pragma unroll
        for (int c = 0; c < Z; ++c)
            if (c >= lo && c < hi) s2 = fmaf(acc[c][j], acc[c][j], s2);
        inv[j] = rsqrtf(s2 + C.eps);
    }
    if (!O.row) return;
    auto emit = [&](auto dt) {
        constexpr int DT = decltype(dt)::value;
        if (O.full) emit_channels<Z, DT, kVector>(acc, inv, lo, hi, c0, desc, sums, O);
        else if (O.gx0 + kRun <= O.W) emit_channels<Z, DT, kWhole>(acc, inv, lo, hi, c0, desc, sums, O);
        else emit_channels<Z, DT, kEdge>(acc, inv, lo, hi, c0, desc, sums, O);
    };
    if (C.dtype == SFOC_DTYPE_F32) emit(std::integral_constant<int, SFOC_DTYPE_F32>{});
    else if (C.dtype == SFOC_DTYPE_BF16) emit(std::integral_constant<int, SFOC_DTYPE_BF16>{});
    else emit(std::integral_constant<int, SFOC_DTYPE_F16>{});
}

// Per-pixel channel sums of the stored values (zero outside the image) into
// the integral-image buffers, and this tile's aggregates for the prefix pass:
// row sums (the 8 lanes of a row, butterfly), column sums (the 8 rows of a
// wave, butterfly, then the 4 waves in order) and the total (the 32 column
// sums, butterfly).  Every sum is taken in a fixed order, so the integral
// images are reproducible.  cs: 2 KB of LDS that no thread still reads
// ([map][wave][column]).
__device__ __forceinline__ void emit_sums(const DescribeJob& J, RunOut& O, int ty0, int tx0, double* cs) {
    const int t = threadIdx.x, H = J.H, W = J.W, gy = O.gy, gx0 = O.gx0;
    double* __restrict__ integ1 = J.integ1;
    double* __restrict__ integ2 = J.integ2;
    double(&d1)[kRun] = O.d1;
    double(&d2)[kRun] = O.d2;
#pragma unroll
    for (int j = 0; j < kRun; ++j)
        if (gy >= H || gx0 + j >= W) d1[j] = d2[j] = 0.0;
    if (gy < H) {
        const int64_t io = (int64_t)(gy + 1) * (W + 1) + gx0 + 1;
#pragma unroll
        for (int j = 0; j < kRun; ++j)
            if (gx0 + j < W) {
                integ1[io + j] = d1[j];
                integ2[io + j] = d2[j];
            }
    }
    const IntegAgg ag = integ_agg(H, W);
    double* __restrict__ agg = J.agg;
    const int tb = tx0 / kTS, ta = ty0 / kTS;
    double r1 = ((d1[0] + d1[1]) + d1[2]) + d1[3];
    double r2 = ((d2[0] + d2[1]) + d2[2]) + d2[3];
#pragma unroll
    for (int d = 1; d < kTS / kRun; d <<= 1) {
        r1 += __shfl_xor(r1, d, 64);
        r2 += __shfl_xor(r2, d, 64);
    }
    if ((t & (kTS / kRun - 1)) == 0 && gy < H) {
        agg[ag.rs1 + tb * (int64_t)H + gy] = r1;
        agg[ag.rs2 + tb * (int64_t)H + gy] = r2;
    }
#pragma unroll
    for (int j = 0; j < kRun; ++j)
#pragma unroll
        for (int d = kTS / kRun; d < 64; d <<= 1) {
            d1[j] += __shfl_xor(d1[j], d, 64);
            d2[j] += __shfl_xor(d2[j], d, 64);
        }
    const int lane = t & 63, wv = t >> 6;
    if (lane < kTS / kRun) {
#pragma unroll
        for (int j = 0; j < kRun; ++j) {
            cs[(0 * (kNT / 64) + wv) * kTS + lane * kRun + j] = d1[j];
            cs[(1 * (kNT / 64) + wv) * kTS + lane * kRun + j] = d2[j];
        }
    }
    __syncthreads();
    static_assert(2 * kTS == 64, "the column sums of both maps fill one wave");
    if (t < 2 * kTS) {
        // wave 0: lane q * 32 + x sums column x of map q over the four
        // waves in order, then the 32 columns of each map are summed by
        // a butterfly within its half-wave (a fixed order)
        const int q = t / kTS, x = t % kTS;
        double c = 0.0;
#pragma unroll
        for (int w = 0; w < kNT / 64; ++w) c += cs[(q * (kNT / 64) + w) * kTS + x];
        if (tx0 + x < W) agg[(q ? ag.cs2 : ag.cs1) + ta * (int64_t)W + tx0 + x] = c;
#pragma unroll
        for (int d = 1; d < kTS; d <<= 1) c += __shfl_xor(c, d, 64);
        if (x == 0) agg[(q ? ag.tt2 : ag.tt1) + ta * ag.ntx + tb] = c;
    }
}

template <int Z, int CG>
__global__ __launch_bounds__(kNT, Z >= 32 ? 2 : 3) void describe_kernel(const DescribeJob single,
                                                          const DescribeJob* __restrict__ jobs,
                                                          const int4* __restrict__ tiles,
                                                          const uint8_t* __restrict__ tmask, const DescribeConsts C,
                                                          int BSP, int ISX, int BPP, int IPP) {
    extern __shared__ float lds[];
    const int t = threadIdx.x;
    const int4 e = tile_entry(tiles, tmask);
    if (e.x < 0) return;
    const DescribeJob J = jobs ? load_table(jobs, e.x) : single;
    const int ty0 = e.y, tx0 = e.z;
    if (tile_unread(J, e, tmask)) {
        if (J.agg) zero_tile_aggregates(J, ty0, tx0);
        return;
    }
    const int Q = C.Q, R = C.R;
    const int nrun = BSP / kRun;
    float* simg = lds;
    float* srow = simg + ISX * IPP;
    float* sbas = lds;   // written once the image and row-pass maps are dead
    const int BB = BSP * BPP;   // one basis / channel map

    // 1. input region (top-left at tile origin - Q - R)
    load_region<4>(J, ty0 - Q - R, tx0 - Q - R, ISX, simg, IPP);
    __syncthreads();

    // 2. basis responses Gx, Gy, Gxx, Gyy, Gxy * I summed over sigma, held in
    //    registers by the thread that owns each vertical run of kRun pixels.
    // runs: (BSP / kRun) vertical runs in each of the BSr = kTS + 2Q columns
    // that steering reads (the padding columns up to BSP are skipped); BSP at
    // most 48.
    constexpr int kMaxOwn = 3;
    float bas[kMaxOwn][5][kRun];
#pragma unroll
    for (int o = 0; o < kMaxOwn; ++o)
#pragma unroll
        for (int m = 0; m < 5; ++m)
#pragma unroll
            for (int j = 0; j < kRun; ++j) bas[o][m][j] = 0.f;
    const int BSr = kTS + 2 * Q;      // rows / columns of the basis maps that steering reads
    const int ncolrun = nrun * BSr;   // (row-run, column) pairs
    for (int s = 0; s < C.nsig; ++s) {
        const int rho = C.rad[s];
        const float* tg = C.taps + C.off[s];
        const float* td = tg + (rho + 1);
        const float* tdd = td + (rho + 1);
        const float cn = C.cnorm[s];
        const int rows = BSP + 2 * rho;
        // row pass on rows [0, rows) x cols [0, BSP): horizontal runs.  Row a
        // of this pass is image-region row a + R - rho.
        for (int e = t; e < rows * nrun; e += kNT) {
            const int a = e / nrun, b0 = (e - a * nrun) * kRun;
            const float* p = simg + (a + R - rho) * IPP + (b0 + R);
            float og[kRun], od[kRun], odd[kRun];
#define ROW_T(RR) row_run<RR>(p, tg, td, tdd, og, od, odd)
            SFOC_RADIUS_SWITCH(rho, ROW_T, row_run_any(p, rho, tg, td, tdd, og, od, odd))
#undef ROW_T
            float* w = srow + a * BPP + b0;
#pragma unroll
            for (int j = 0; j < kRun; ++j) {
                w[j] = og[j];
                w[rows * BPP + j] = od[j];
                w[2 * rows * BPP + j] = odd[j];
            }
        }
        __syncthreads();
        // column pass on vertical runs; output row a reads pass rows a + rho + k.
        const float* rg = srow;
        const float* rd = srow + rows * BPP;
        const float* rdd = srow + 2 * rows * BPP;
        const int ig = ISX * IPP, id = ig + rows * BPP, idd = ig + 2 * rows * BPP;   // the same, as lds indices
        const int use = C.use[s];
#pragma unroll
        for (int o = 0; o < kMaxOwn; ++o) {
            const int e = t + o * kNT;
            if (e < ncolrun) {
                const int b = e % BSr, a0 = (e / BSr) * kRun;
                float bx[kRun], by[kRun], bxx[kRun], byy[kRun], bxy[kRun], dummy[kRun];
                const int c0 = (a0 + rho) * BPP + b;
                // rg -> By (odd d), Byy (even dd); rd -> Bx (even g), Bxy (odd d);
                // rdd -> Bxx (even g).
#define COL_T(RR)                                                \
    do {                                                         \
        col_run<RR>(lds, ig + c0, BPP, tdd, td, byy, by);        \
        col_run<RR>(lds, id + c0, BPP, tg, td, bx, bxy);         \
        col_run<RR>(lds, idd + c0, BPP, tg, nullptr, bxx, dummy); \
    } while (0)
#define COL_ANY                                                  \
    do {                                                         \
        col_run_any(rg + c0, BPP, rho, tdd, td, byy, by);        \
        col_run_any(rd + c0, BPP, rho, tg, td, bx, bxy);         \
        col_run_any(rdd + c0, BPP, rho, tg, nullptr, bxx, dummy); \
    } while (0)
                SFOC_RADIUS_SWITCH(rho, COL_T, COL_ANY)
#undef COL_T
#undef COL_ANY
                (void)dummy;
#pragma unroll
                for (int j = 0; j < kRun; ++j) {
                    // the 2-D normalisation cn of this sigma, applied as the
                    // response joins the sum over sigma
                    if (use & 1) {
                        bas[o][0][j] = fmaf(cn, bx[j], bas[o][0][j]);
                        bas[o][1][j] = fmaf(cn, by[j], bas[o][1][j]);
                    }
                    if (use & 2) {
                        bas[o][2][j] = fmaf(cn, bxx[j], bas[o][2][j]);
                        bas[o][3][j] = fmaf(cn, byy[j], bas[o][3][j]);
                        bas[o][4][j] = fmaf(cn, bxy[j], bas[o][4][j]);
                    }
                }
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int o = 0; o < kMaxOwn; ++o) {
        const int e = t + o * kNT;
        if (e < ncolrun) {
            const int b = e % BSr, a0 = (e / BSr) * kRun;
#pragma unroll
            for (int m = 0; m < 5; ++m)
#pragma unroll
                for (int j = 0; j < kRun; ++j) sbas[m * BB + (a0 + j) * BPP + b] = bas[o][m][j];
        }
    }
    __syncthreads();

    // 3. steer + rectify per channel group into LDS, then dilated smoothing
    //    of this thread's horizontal run of kRun outputs.
    float acc[Z][kRun];
    float* schan = sbas + 5 * BB;
    const int N = C.N, B = 2 * C.K + 1;
    RunOut O;
    init_run(O, J, C, ty0, tx0);
    // (in a function of its own, by which the compiler addresses the maps with
    // fewer instructions: 1024 x 1024, eight orientations of the first order 190 us
    // without, 172 us with)
    auto steer_smooth = [&](int lo, int hi) {
#pragma unroll
        for (int c0 = lo; c0 < hi; c0 += CG) {
            // thread index laundered per group: keeps the group's LDS addresses
            // from being hoisted (and kept live) across the whole channel loop.
            int tl = t;
            asm volatile("" : "+v"(tl));
            const int obase = (tl / (kTS / kRun) + Q) * BPP + (tl % (kTS / kRun)) * kRun + Q;
            for (int e = tl; e < BSr * BSr; e += kNT) {
                const int a = e / BSr, b = e - a * BSr;
                const int idx = a * BPP + b;
#pragma unroll
                for (int cc = 0; cc < CG; ++cc) {
                    const int c = c0 + cc;
                    if (c < Z) {
                        float v;   // (the order of each sum is spelled out: results do not move with the compiler)
                        if (c < N) {
                            v = fmaf(C.s1[c], sbas[BB + idx], C.c1[c] * sbas[idx]);
                        } else {
                            const int k = c - N;
                            v = fmaf(C.sc2[k], sbas[4 * BB + idx],
                                     fmaf(C.cc[k], sbas[2 * BB + idx], C.ss[k] * sbas[3 * BB + idx]));
                        }
                        if (C.rectify == SFOC_RECTIFY_ABS) v = fabsf(v);
                        else if (C.rectify == SFOC_RECTIFY_RELU) v = fmaxf(v, 0.f);
                        schan[cc * BB + idx] = v;
                    }
                }
            }
            __syncthreads();
#pragma unroll
            for (int cc = 0; cc < CG; ++cc) {
                const int c = c0 + cc;
                if (c < Z) {
                    const float* w = (c < N) ? C.w1 : C.w2;
                    const float* ch = schan + cc * BB + obase;
#pragma unroll
                    for (int j = 0; j < kRun; ++j) {
                        float a = 0.f;
                        for (int di = 0; di < C.ndil; ++di) {
                            const int r = C.dil[di];
                            for (int i = 0; i < B; ++i)
                                for (int jj = 0; jj < B; ++jj)
                                    a = fmaf(w[i * B + jj], ch[(i - C.K) * r * BPP + (jj - C.K) * r + j], a);
                        }
                        acc[c][j] = a;
                    }
                }
            }
            __syncthreads();
        }
    };
    steer_smooth(0, Z);
    emit_block<Z>(acc, 0, N, 0, J.desc, J.integ1 != nullptr, C, O);
    emit_block<Z>(acc, N, Z, 0, J.desc, J.integ1 != nullptr, C, O);
    if (J.integ1) emit_sums(J, O, ty0, tx0, reinterpret_cast<double*>(lds));
}

// ---- K = 1, rates 1, 2, 3, both orders ----------------------------------------
// Row pass, then column pass, of one sigma; the responses join the thread's
// sums over sigma.  RHO = 0: any radius.  Thread t owns the column runs
// t + o kNT of three rows: 494 runs of 38 columns, so that every wave has two
// rounds of three rows (runs of four rows: 380, two rounds for half of the
// waves).  USE: see row_run; what an order does not read is not computed.
template <int RHO, int USE>
__device__ __forceinline__ void sigma_pass(const float* simg, int IPP, float* srow, const DescribeConsts& C, int s,
                         float (&bas)[kCOwn][5][kCRun]) {
    // (the index laundered: what is derived from it is not hoisted out of the
    // sigma loop, for every radius at once)
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    const int rho = RHO ? RHO : C.rad[s], R = C.R;
    const float* tg = C.taps + C.off[s];
    const float* td = tg + (rho + 1);
    const float* tdd = td + (rho + 1);
    const float cn = C.cnorm[s];
    const int use = RHO ? USE : C.use[s];
    const int rows = kB + 2 * rho, map = rows * kRP;
    // Row a of this pass is image-region row a + R - rho.  The lanes run along
    // the rows: with odd pitches their accesses fall on different banks.  (The
    // last run's two columns past the map are never read.)
    constexpr int kRuns = (kB + kRun - 1) / kRun;
    for (int e = t; e < rows * kRuns; e += kNT) {
        const int q = e / rows, a = e - q * rows, b0 = q * kRun;
        const float* p = simg + (a + R - rho) * IPP + (b0 + R);
        float og[kRun], od[kRun], odd[kRun];
        if constexpr (RHO > 0) row_run<RHO, USE>(p, tg, td, tdd, og, od, odd);
        else row_run_any(p, rho, tg, td, tdd, og, od, odd);
        float* w = srow + a * kRP + b0;
#pragma unroll
        for (int j = 0; j < kRun; ++j) {
            w[j] = og[j];
            w[map + j] = od[j];
            if (USE & 2) w[2 * map + j] = odd[j];
        }
    }
    __syncthreads();
    // output row a reads pass rows a + rho + k; g -> By (odd d), Byy (even dd);
    // d -> Bx (even g), Bxy (odd d); dd -> Bxx (even g)
#pragma unroll
    for (int o = 0; o < kCOwn; ++o) {
        __builtin_amdgcn_sched_barrier(0);
        const int e = t + o * kNT;
        if (e < kCRuns * kB) {
            const int c0 = (e / kB * kCRun + rho) * kRP + e % kB;
            float bx[kCRun], by[kCRun], bxx[kCRun], byy[kCRun], bxy[kCRun], none[kCRun];
            const float* t1 = USE & 1 ? tg : nullptr;
            const float* t1d = USE & 1 ? td : nullptr;
            const float* t2dd = USE & 2 ? tdd : nullptr;
            const float* t2d = USE & 2 ? td : nullptr;
            if constexpr (RHO > 0) {
                col_run<RHO, kCRun>(srow, c0, kRP, t2dd, t1d, byy, by);
                col_run<RHO, kCRun>(srow, c0 + map, kRP, t1, t2d, bx, bxy);
                if (USE & 2) col_run<RHO, kCRun>(srow, c0 + 2 * map, kRP, tg, nullptr, bxx, none);
            } else {
                col_run_any<kCRun>(srow + c0, kRP, rho, t2dd, t1d, byy, by);
                col_run_any<kCRun>(srow + c0 + map, kRP, rho, t1, t2d, bx, bxy);
                if (USE & 2) col_run_any<kCRun>(srow + c0 + 2 * map, kRP, rho, tg, nullptr, bxx, none);
            }
            (void)none;
            // the 2-D normalisation cn of this sigma is applied here
#pragma unroll
            for (int j = 0; j < kCRun; ++j) {
                if (use & 1) {
                    bas[o][0][j] = fmaf(cn, bx[j], bas[o][0][j]);
                    bas[o][1][j] = fmaf(cn, by[j], bas[o][1][j]);
                }
                if (use & 2) {
                    bas[o][2][j] = fmaf(cn, bxx[j], bas[o][2][j]);
                    bas[o][3][j] = fmaf(cn, byy[j], bas[o][3][j]);
                    bas[o][4][j] = fmaf(cn, bxy[j], bas[o][4][j]);
                }
            }
        }
    }
    __syncthreads();
}
template <int RHO>
__device__ __forceinline__ void sigma_pass_use(const float* simg, int IPP, float* srow, const DescribeConsts& C, int s,
                                               float (&bas)[kCOwn][5][kCRun]) {
    if (RHO > 0 && C.use[s] == 1) sigma_pass<RHO, RHO ? 1 : 3>(simg, IPP, srow, C, s, bas);
    else if (RHO > 0 && C.use[s] == 2) sigma_pass<RHO, RHO ? 2 : 3>(simg, IPP, srow, C, s, bas);
    else sigma_pass<RHO, 3>(simg, IPP, srow, C, s, bas);
}

// The same method for the parameters in use, z = 2 N channels.  What bounds
// it is instruction issue, so everything is arranged for few instructions a
// pixel: the maps are linear with compile-time pitches; a thread holds the
// basis of its six map elements in registers while an order's channels are
// steered (a multiply-add or two and a store a channel, no address
// arithmetic); steered maps alternate between two buffers, the ones the first
// order's basis came from, with one barrier a channel; and an order is emitted
// before the next is steered, so four workgroups fit a CU (40 KB of LDS for
// R = 9, 128 VGPRs for N <= 8).
// 2048 x 2048, FP32 with integral inputs: 250 us with the basis read from LDS
// by a loop over map elements (23 issue slots a channel and element), runs of
// four rows and two or four row-pass phases a sigma; 185 us so (85.0 M wave
// instructions, three quarters of the issue slots).
// The arguments are read where the launch put them: as a by-value parameter
// with this many readers the compiler would copy them to scratch memory.
struct K1Args {
    DescribeJob single;
    const DescribeJob* jobs;
    const int4* tiles;
    const uint8_t* tmask;
    DescribeConsts C;
};
template <int N>
__global__ __launch_bounds__(kNT, N <= 8 ? 4 : 3) void describe_k1_kernel(const K1Args by_value) {
    extern __shared__ float lds[];
    const K1Args& A = *(const K1Args*)__builtin_amdgcn_kernarg_segment_ptr();
    const DescribeConsts& C = A.C;
    const int4 e = tile_entry(A.tiles, A.tmask);
    if (e.x < 0) return;
    const DescribeJob J = A.jobs ? load_table(A.jobs, e.x) : A.single;
    const int ty0 = e.y, tx0 = e.z;
    if (tile_unread(J, e, A.tmask)) {
        if (J.agg) zero_tile_aggregates(J, ty0, tx0);
        return;
    }
    const int t = threadIdx.x, R = C.R, side = kB + 2 * R, IPP = side | 1;
    float* srow = lds + side * IPP;
    load_region<8>(J, ty0 - 3 - R, tx0 - 3 - R, side, lds, IPP);
    __syncthreads();

    // Gx, Gy, Gxx, Gyy, Gxy * I summed over sigma, held by the threads of the
    // column runs, then laid out as maps over the dead image region
    {
        float bas[kCOwn][5][kCRun];
#pragma unroll
        for (int o = 0; o < kCOwn; ++o)
#pragma unroll
            for (int m = 0; m < 5; ++m)
#pragma unroll
                for (int j = 0; j < kCRun; ++j) bas[o][m][j] = 0.f;
        for (int s = 0; s < C.nsig; ++s) {
#define PASS(RR) sigma_pass_use<RR>(lds, IPP, srow, C, s, bas)
            SFOC_RADIUS_SWITCH(C.rad[s], PASS, PASS(0))
#undef PASS
        }
#pragma unroll
        for (int o = 0; o < kCOwn; ++o) {
            const int e = t + o * kNT;
            if (e < kCRuns * kB) {
                float* d = lds + e / kB * kCRun * kCP + e % kB;
#pragma unroll
                for (int m = 0; m < 5; ++m)
#pragma unroll
                    for (int j = 0; j < kCRun; ++j) d[m * kCM + j * kCP] = bas[o][m][j];
            }
        }
    }
    __syncthreads();

    RunOut O;
    init_run(O, J, C, ty0, tx0);
    const bool sums = J.integ1 != nullptr;
    const int rect = C.rectify;
    // the top-left element of the neighbourhood of the thread's output run
    const int nb = (t / (kTS / kRun)) * kCP + (t % (kTS / kRun)) * kRun + 3 * kCP + 3;
    float acc[N][kRun];
    // Channels of one order: steer(c, k) is channel c at the thread's map
    // element k.  Map elements past the 38 x 38 pixels hold values that no
    // output reads.  A buffer is written again two channels later, when every
    // thread has passed the barrier after it last read it.
    auto channels = [&](auto steer, const float* w) {
#pragma unroll
        for (int c = 0; c < N; ++c) {
            float* buf = lds + (c & 1) * kCM;
            if (rect == SFOC_RECTIFY_ABS) {
#pragma unroll
                for (int k = 0; k < kPix; ++k) buf[t + k * kNT] = fabsf(steer(c, k));
            } else if (rect == SFOC_RECTIFY_RELU) {
#pragma unroll
                for (int k = 0; k < kPix; ++k) buf[t + k * kNT] = fmaxf(steer(c, k), 0.f);
            } else {
#pragma unroll
                for (int k = 0; k < kPix; ++k) buf[t + k * kNT] = steer(c, k);
            }
            __syncthreads();
            smooth_run_k1_123(lds, (c & 1) * kCM + nb, kCP, w[4], w[1], w[0], acc[c]);
            // computed here, with one channel's reads in flight at a time
#pragma unroll
            for (int j = 0; j < kRun; ++j) asm volatile("" : "+v"(acc[c][j]));
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    {
        float b0[kPix], b1[kPix];
#pragma unroll
        for (int k = 0; k < kPix; ++k) {
            b0[k] = lds[t + k * kNT];
            b1[k] = lds[kCM + t + k * kNT];
        }
        __syncthreads();   // the maps become the channel buffers
        channels([&](int c, int k) { return fmaf(C.c1[c], b0[k], C.s1[c] * b1[k]); }, C.w1);
    }
    emit_block<N>(acc, 0, N, 0, J.desc, sums, C, O);
    {
        float b2[kPix], b3[kPix], b4[kPix];
#pragma unroll
        for (int k = 0; k < kPix; ++k) {
            b2[k] = lds[2 * kCM + t + k * kNT];
            b3[k] = lds[3 * kCM + t + k * kNT];
            b4[k] = lds[4 * kCM + t + k * kNT];
        }
        if (N & 1) __syncthreads();   // buffer 0 again, read by the last channel
        channels([&](int c, int k) { return fmaf(C.sc2[c], b4[k], fmaf(C.cc[c], b2[k], C.ss[c] * b3[k])); }, C.w2);
    }
    emit_block<N>(acc, 0, N, N, J.desc, sums, C, O);
    if (sums) {
        // the column sums go where nobody reads any more (map 2)
        emit_sums(J, O, ty0, tx0, reinterpret_cast<double*>(lds + 2 * kCM));
    }
}

// ---- integral images (Eq. 14-16) ------------------------------------------
// The inclusive 2-D prefix sum (Eq. 15) of a per-pixel map s, at a pixel
// (y0 + i, x0 + j) of the tile (a, b) with origin (y0, x0), splits into
//   Corner(a, b)                  the tiles above and to the left,
// + sum_{j' <= j} Above(x0 + j')  the rows above the tile, per column,
// + sum_{i' <= i} [Left(y0 + i') + sum_{j' <= j} s(y0 + i', x0 + j')]
// with Left(y) the sum of row y left of the tile and Above(x) the sum of
// column x above it.  The describe kernel wrote s into the integral buffers
// and each tile's row sums, column sums and total; integral_prefix turns
// these into Left (exclusive prefixes of the row sums over tile columns),
// Above (of the column sums over tile rows) and Corner (the 2-D exclusive
// prefix of the tile totals); integral_tiles then reads s once and writes
// the prefix sums in place.  All sums are in a fixed order.

// In place, for two sequences at once: a[0], a[step], ... and b[0],
// b[step], ... (n entries each) -> their exclusive prefix sums.  Sixteen
// loads of each are in flight before their sums, which run in order.
SFOC_DEV void exclusive_prefix2(double* __restrict__ a, double* __restrict__ b, int64_t n, int64_t step) {
    constexpr int kB = 16;
    double ra = 0.0, rb = 0.0;
    int64_t k = 0;
    for (; k + kB <= n; k += kB) {
        double x[kB], y[kB];
#pragma unroll
        for (int u = 0; u < kB; ++u) {
            x[u] = a[(k + u) * step];
            y[u] = b[(k + u) * step];
        }
#pragma unroll
        for (int u = 0; u < kB; ++u) {
            a[(k + u) * step] = ra;
            b[(k + u) * step] = rb;
            ra += x[u];
            rb += y[u];
        }
    }
    for (; k < n; ++k) {
        const double x = a[k * step], y = b[k * step];
        a[k * step] = ra;
        b[k * step] = rb;
        ra += x;
        rb += y;
    }
}

void integral_prefix_items(int job, int H, int W, std::vector<int4>& out) {
    for (int k = 0; k < (H + kScanNT - 1) / kScanNT; ++k) out.push_back(make_int4(job, 0, k, 0));
    for (int k = 0; k < (W + kScanNT - 1) / kScanNT; ++k) out.push_back(make_int4(job, 1, k, 0));
    out.push_back(make_int4(job, 2, 0, 0));
}

template <bool BATCH>
__global__ __launch_bounds__(kScanNT) void integral_prefix(const IntegJob single, const IntegJob* __restrict__ jobs,
                                                           const int4* __restrict__ items) {
    IntegJob J;
    int kind, blk;
    if (BATCH) {
        const int4 it = items[blockIdx.x];
        J = load_table(jobs, it.x);
        kind = it.y;
        blk = it.z;
    } else {
        J = single;
        const int nbr = (J.H + kScanNT - 1) / kScanNT, nbc = (J.W + kScanNT - 1) / kScanNT;
        const int k = blockIdx.x;
        kind = k < nbr ? 0 : (k < nbr + nbc ? 1 : 2);
        blk = kind == 0 ? k : (kind == 1 ? k - nbr : 0);
    }
    const int H = J.H, W = J.W, t = threadIdx.x;
    const IntegAgg ag = integ_agg(H, W);
    double* __restrict__ agg = J.agg;
    if (kind == 0) {          // Left: per row y, over the tile columns
        const int y = blk * kScanNT + t;
        if (y < H) exclusive_prefix2(agg + ag.rs1 + y, agg + ag.rs2 + y, ag.ntx, H);
    } else if (kind == 1) {   // Above: per column x, over the tile rows
        const int x = blk * kScanNT + t;
        if (x < W) exclusive_prefix2(agg + ag.cs1 + x, agg + ag.cs2 + x, ag.nty, W);
    } else {                  // Corner: tile totals, over tile columns, then over tile rows
        for (int64_t a = t; a < ag.nty; a += kScanNT)
            exclusive_prefix2(agg + ag.tt1 + a * ag.ntx, agg + ag.tt2 + a * ag.ntx, ag.ntx, 1);
        __syncthreads();
        for (int64_t b = t; b < ag.ntx; b += kScanNT)
            exclusive_prefix2(agg + ag.tt1 + b, agg + ag.tt2 + b, ag.nty, ag.ntx);
    }
}

// One 32 x 32 tile per workgroup, in three phases over an LDS copy of the
// tile.  Thread t first holds column t % 32 of rows 4 (t / 32) .. + 3, so a
// wave's loads and stores cover two rows of 32 consecutive pixels: it loads
// s, sums down its four rows, then adds the totals of the row groups above
// (the column prefix C).  Then thread t holds a run of 4 pixels of row t / 8
// and sums C along the row: I = Corner + prefix(Above) + prefix(Left) +
// prefix over the row of C, the decomposition above in another order.  The
// results go back through LDS to the column layout for the stores.  Row 0
// and column 0 of the integral images are set to zero by the tiles that
// border them.
template <bool BATCH>
__global__ __launch_bounds__(kScanNT) void integral_tiles(const IntegJob single, const IntegJob* __restrict__ jobs,
                                                          const int4* __restrict__ tiles,
                                                          uint8_t* __restrict__ tmask) {
    constexpr int kRows = kTS * kTS / kScanNT;   // rows per thread in the column layout
    constexpr int kGroups = kTS / kRows;         // row groups in a tile
    constexpr int kRuns = kTS / kRun;            // runs in a tile row
    static_assert(kRows == 4 && kGroups * kTS == kScanNT && kRuns * kTS == kScanNT, "tile layouts");
    IntegJob J;
    int ta, tb;
    // Workgroups are dealt to the eight XCDs in turn; renumbered so that each
    // XCD takes one contiguous run of tiles (row-major), neighbouring tiles
    // share an L2 and the cache lines on their borders (the images' row
    // pitch W + 1 is not a multiple of a line) are fetched once.
    const int nblk = BATCH ? (int)gridDim.x : (int)(gridDim.x * gridDim.y);
    const int id = BATCH ? (int)blockIdx.x : (int)(blockIdx.y * gridDim.x + blockIdx.x);
    const int q8 = nblk / 8 * 8;
    const int k = id < q8 ? (id % 8) * (q8 / 8) + id / 8 : id;
    if (BATCH) {
        const int4 e = tiles[k];
        J = load_table(jobs, e.x);
        ta = e.y;
        tb = e.z;
    } else {
        J = single;
        ta = k / gridDim.x;
        tb = k - ta * gridDim.x;
        if (tmask) {   // the mask's last reader: the byte is cleared for the next call
            const bool read = tmask[k] != 0;
            __syncthreads();
            if (threadIdx.x == 0) tmask[k] = 0;
            if (!read) return;   // a tile that nothing reads
        }
    }
    __shared__ double T[2][kTS][kTS + 1];   // the tile of both maps
    __shared__ double tot[2][kScanNT];      // row-group totals, then run totals
    __shared__ double pre_left[2][kTS];     // inclusive prefix of Left over the tile rows
    __shared__ double pre_above[2][kTS];    // Corner + inclusive prefix of Above over the tile columns
    const int H = J.H, W = J.W, t = threadIdx.x;
    const IntegAgg ag = integ_agg(H, W);
    const double* __restrict__ agg = J.agg;
    const int64_t P = W + 1;
    const int y0 = ta * kTS, x0 = tb * kTS;
    const int c = t % kTS, gr = t / kTS;    // column layout: column c, rows kRows * gr + k
    // Left (map 1 in lanes 0..31, map 2 in lanes 32..63 of waves 0 and 2)
    // and Above with Corner (waves 1 and 3), loaded before the tile and
    // without branches (waves 2 and 3 repeat 0 and 1; only those store).
    const bool is_above = (t / (2 * kTS)) & 1;
    const int qa = (t / kTS) & 1, ea = t % kTS;
    const int64_t ia = is_above ? (qa ? ag.cs2 : ag.cs1) + ta * (int64_t)W + min(x0 + ea, W - 1)
                                : (qa ? ag.rs2 : ag.rs1) + tb * (int64_t)H + min(y0 + ea, H - 1);
    const double va_in = agg[ia];
    const bool va_ok = is_above ? x0 + ea < W : y0 + ea < H;
    const double corner = agg[(qa ? ag.tt2 : ag.tt1) + ta * ag.ntx + tb];
    // The tile, at clamped addresses (every load in bounds and all of them in
    // flight at once); pixels outside the image count as zero.
    double s[2][kRows];
    bool ok[kRows];
#pragma unroll
    for (int k = 0; k < kRows; ++k) {
        const int y = y0 + kRows * gr + k, x = x0 + c;
        ok[k] = y < H && x < W;
        const int64_t off = (int64_t)(min(y, H - 1) + 1) * P + min(x, W - 1) + 1;
        s[0][k] = J.g1[off];
        s[1][k] = J.g2[off];
    }
    // the prefixes of Left, and of Above with Corner
    double va = va_ok ? va_in : 0.0;
#pragma unroll
    for (int d = 1; d < kTS; d <<= 1) {
        const double u = __shfl_up(va, d, kTS);
        if (ea >= d) va += u;
    }
    if (t < 4 * kTS) {
        if (!is_above) pre_left[qa][ea] = va;
        else pre_above[qa][ea] = corner + va;
    }
    // column prefix: down the thread's rows, then the row groups above
#pragma unroll
    for (int q = 0; q < 2; ++q) {
#pragma unroll
        for (int k = 0; k < kRows; ++k) s[q][k] = ok[k] ? s[q][k] : 0.0;
#pragma unroll
        for (int k = 1; k < kRows; ++k) s[q][k] += s[q][k - 1];
        tot[q][gr * kTS + c] = s[q][kRows - 1];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        double e = 0.0;
        for (int g2 = 0; g2 < gr; ++g2) e += tot[q][g2 * kTS + c];
#pragma unroll
        for (int k = 0; k < kRows; ++k) T[q][kRows * gr + k][c] = s[q][k] + e;
    }
    __syncthreads();
    // row prefix of C: thread t holds the run of row i from column j0
    const int i = t / kRuns, rl = t % kRuns, j0 = rl * kRun;
    double v[2][kRun];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
#pragma unroll
        for (int k = 0; k < kRun; ++k) v[q][k] = T[q][i][j0 + k];
#pragma unroll
        for (int k = 1; k < kRun; ++k) v[q][k] += v[q][k - 1];
        tot[q][i * kRuns + rl] = v[q][kRun - 1];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        double e = pre_left[q][i];
        for (int r2 = 0; r2 < rl; ++r2) e += tot[q][i * kRuns + r2];
#pragma unroll
        for (int k = 0; k < kRun; ++k) T[q][i][j0 + k] = pre_above[q][j0 + k] + (e + v[q][k]);
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        double* __restrict__ g = q ? J.g2 : J.g1;
#pragma unroll
        for (int k = 0; k < kRows; ++k) {
            const int y = y0 + kRows * gr + k, x = x0 + c;
            if (ok[k]) g[(int64_t)(y + 1) * P + x + 1] = T[q][kRows * gr + k][c];
        }
        if (ta == 0 && t < kTS && x0 + t < W) g[x0 + t + 1] = 0.0;
        if (ta == 0 && tb == 0 && t == 0) g[0] = 0.0;
        if (tb == 0 && t < kTS && y0 + t < H) g[(int64_t)(y0 + t + 1) * P] = 0.0;
    }
}

// ---- launch -------------------------------------------------------------
// K = 1 at rates 1, 2, 3 with both orders: compile-time geometry.
static bool describe_k1(const DescribeConsts& c) {
    return c.K == 1 && c.ndil == 3 && c.dil[0] == 1 && c.dil[1] == 2 && c.dil[2] == 3 && c.second &&
           c.N * 2 == c.z;
}

int describe_configs(const DescribeConsts& c) { return describe_k1(c) && c.z <= 16 ? 2 : 1; }

template <int Z>
static hipError_t launch_describe_z(const DescribeJob& job, const DescribeJob* jobs, const int4* tiles, int ntiles,
                                    const uint8_t* tmask, const DescribeConsts& c, hipStream_t st) {
    const dim3 grid = tiles ? dim3(ntiles) : dim3((job.W + kTS - 1) / kTS, (job.H + kTS - 1) / kTS);
    if (grid.x == 0) return hipSuccess;
    if constexpr (Z % 2 == 0)
        if (describe_k1(c)) {
            auto kern = describe_k1_kernel<Z / 2>;
            const size_t bytes = describe_k1_lds(c.R);
            hipError_t e = ensure_dynamic_lds((const void*)kern, (int)bytes);
            if (e != hipSuccess) return e;
            trace_begin(st, SFOC_K_DESCRIBE);
            hipLaunchKernelGGL(kern, grid, dim3(kNT), bytes, st, K1Args{job, jobs, tiles, tmask, c});
            trace_end(st, SFOC_K_DESCRIBE);
            return hipGetLastError();
        }
    constexpr int CG = Z >= 4 ? 4 : Z;
    const DescribeGeom g = describe_geom(c, CG);
    auto kern = describe_kernel<Z, CG>;
    hipError_t e = ensure_dynamic_lds((const void*)kern, (int)g.bytes);
    if (e != hipSuccess) return e;
    trace_begin(st, SFOC_K_DESCRIBE);
    hipLaunchKernelGGL(kern, grid, dim3(kNT), g.bytes, st, job, jobs, tiles, tmask, c, g.BSP, g.ISX, g.BPP, g.IPP);
    trace_end(st, SFOC_K_DESCRIBE);
    return hipGetLastError();
}

static hipError_t launch_describe_any(const DescribeJob& job, const DescribeJob* jobs, const int4* tiles, int ntiles,
                                      const uint8_t* tmask, const DescribeConsts& c, hipStream_t st) {
    switch (c.z) {
        case 2: return launch_describe_z<2>(job, jobs, tiles, ntiles, tmask, c, st);
        case 3: return launch_describe_z<3>(job, jobs, tiles, ntiles, tmask, c, st);
        case 4: return launch_describe_z<4>(job, jobs, tiles, ntiles, tmask, c, st);
        case 6: return launch_describe_z<6>(job, jobs, tiles, ntiles, tmask, c, st);
        case 8: return launch_describe_z<8>(job, jobs, tiles, ntiles, tmask, c, st);
        case 12: return launch_describe_z<12>(job, jobs, tiles, ntiles, tmask, c, st);
        case 16: return launch_describe_z<16>(job, jobs, tiles, ntiles, tmask, c, st);
        case 24: return launch_describe_z<24>(job, jobs, tiles, ntiles, tmask, c, st);
        case 32: return launch_describe_z<32>(job, jobs, tiles, ntiles, tmask, c, st);
        default: return hipErrorInvalidValue;
    }
}

// Several images in one launch: jobs and tiles are device tables.
hipError_t launch_describe_batched(const DescribeJob* jobs, const int4* tiles, int ntiles, const DescribeConsts& c,
                                   hipStream_t st) {
    DescribeJob none{};
    return launch_describe_any(none, jobs, tiles, ntiles, nullptr, c, st);
}

hipError_t launch_describe(const float* img, int H, int W, int64_t ld, void* desc, double* i1, double* i2,
                           double* agg, const DescribeConsts& c, hipStream_t st, const uint8_t* tmask) {
    DescribeJob job{img, desc, i1, i2, agg, ld, H, W};
    return launch_describe_any(job, nullptr, nullptr, 0, tmask, c, st);
}

hipError_t launch_describe_tiles(const float* img, int H, int W, int64_t ld, void* desc, const int4* tiles,
                                 int ntiles, const DescribeConsts& c, hipStream_t st) {
    if (ntiles == 0) return hipSuccess;
    DescribeJob job{img, desc, nullptr, nullptr, nullptr, ld, H, W};
    return launch_describe_any(job, nullptr, tiles, ntiles, nullptr, c, st);
}

// ---- the pair call's describe table ---------------------------------------
// One launch describes both images of a pair.  Entries 0 .. NR - 1 of the
// table are the reference image's grid tiles in row-major order, {0, row
// origin, column origin, 2}: described where the window mask marks the
// tile, else given zero integral-image aggregates.  Slot (i, a, c) after
// them, i < n, a, c < ceil(m / T), is the sensed image's tile of IP i's
// template with rows from the template's row a * T and columns from its
// column c * T ({1, ...}), or an empty slot (job -1) where the IP reads
// nothing (template_tile_range).  Tiles of two IPs may overlap: both
// describe the shared pixels, with equal results (a pixel's descriptor does
// not depend on the tile that computes it).  Thread 0 writes the two jobs;
// thread i < n also marks the reference tiles of IP i's search window
// (window_tile_range, the rule batched plans apply on the host), byte
// stores of 1 in any order.  The mask is not cleared first: the integral
// pass, its last reader, clears every byte it reads, and a byte left set by
// memory that never held a mask only makes a tile be described that
// nothing reads.
__global__ __launch_bounds__(256) void pair_table_kernel(const int32_t* __restrict__ ips,
                                                         const int32_t* __restrict__ prior, int n, int m, int r,
                                                         int Hs, int Ws, int Hr, int Wr, const DescribeJob jref,
                                                         const DescribeJob jsen, DescribeJob* __restrict__ jobs,
                                                         int4* __restrict__ tiles, uint8_t* __restrict__ mask) {
    const int S = template_tile_slots(m, kTS), CT = template_tile_rows(m, kTS);
    const int ntx = (Wr + kTS - 1) / kTS, NR = ntx * ((Hr + kTS - 1) / kTS);
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e == 0) {
        jobs[0] = jref;
        jobs[1] = jsen;
    }
    if (e < n) {
        const int i = (int)e;
        int64_t a0, a1, b0, b1;
        if (window_tile_range(ips[2 * i], ips[2 * i + 1], prior ? prior[2 * i] : 0, prior ? prior[2 * i + 1] : 0, m,
                              r, Hs, Ws, Hr, Wr, kTS, &a0, &a1, &b0, &b1))
            for (int64_t a = a0; a <= a1; ++a)
                for (int64_t b = b0; b <= b1; ++b) mask[a * ntx + b] = 1;
    }
    if (e < NR) {
        const int a = (int)(e / ntx), b = (int)(e - (int64_t)a * ntx);
        tiles[e] = make_int4(0, a * kTS, b * kTS, 2);
    } else if (e < NR + (int64_t)n * S) {
        const int64_t f = e - NR;
        const int i = (int)(f / S), s = (int)(f - (int64_t)i * S), a = s / CT, c = s - a * CT;
        int64_t ty, tx;
        const bool in = template_tile_range(ips[2 * i], ips[2 * i + 1], prior ? prior[2 * i] : 0,
                                            prior ? prior[2 * i + 1] : 0, m, r, Hs, Ws, Hr, Wr, &ty, &tx);
        tiles[e] = in ? make_int4(1, (int)(ty + (int64_t)a * kTS), (int)(tx + (int64_t)c * kTS), 0)
                      : make_int4(-1, 0, 0, 0);
    }
}

int64_t pair_table_entries(int Hr, int Wr, int n, int m) {
    return (int64_t)((Wr + kTS - 1) / kTS) * ((Hr + kTS - 1) / kTS) + (int64_t)n * template_tile_slots(m, kTS);
}

hipError_t launch_describe_pair(const float* ref, int Hr, int Wr, int64_t ldr, void* dref, double* i1, double* i2,
                                double* agg, const float* sen, int Hs, int Ws, int64_t lds, void* dsen,
                                const int32_t* ips, const int32_t* prior, int n, int m, int r, DescribeJob* jobs,
                                int4* tiles, uint8_t* mask, const DescribeConsts& c, hipStream_t st) {
    const DescribeJob jref{ref, dref, i1, i2, agg, ldr, Hr, Wr};
    const DescribeJob jsen{sen, dsen, nullptr, nullptr, nullptr, lds, Hs, Ws};
    const int64_t cnt = pair_table_entries(Hr, Wr, n, m);
    const int64_t nthr = cnt > n ? cnt : n;
    hipLaunchKernelGGL(pair_table_kernel, dim3((unsigned)((nthr + 255) / 256)), dim3(256), 0, st, ips, prior, n, m, r,
                       Hs, Ws, Hr, Wr, jref, jsen, jobs, tiles, mask);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    DescribeJob none{};
    return launch_describe_any(none, jobs, tiles, (int)cnt, mask, c, st);
}

hipError_t launch_integral(double* i1, double* i2, int H, int W, double* agg, hipStream_t st, uint8_t* tmask) {
    const IntegJob J{i1, i2, agg, H, W};
    const IntegJob* none = nullptr;
    const int4* nit = nullptr;
    const int npre = (H + kScanNT - 1) / kScanNT + (W + kScanNT - 1) / kScanNT + 1;
    trace_begin(st, SFOC_K_INTEGRAL);
    hipLaunchKernelGGL(integral_prefix<false>, dim3(npre), dim3(kScanNT), 0, st, J, none, nit);
    hipLaunchKernelGGL(integral_tiles<false>, dim3((W + kTS - 1) / kTS, (H + kTS - 1) / kTS), dim3(kScanNT), 0, st,
                       J, none, nit, tmask);
    trace_end(st, SFOC_K_INTEGRAL);
    return hipGetLastError();
}

hipError_t launch_integral_batched(const IntegJob* jobs, const int4* pre, int npre, const int4* tiles, int ntiles,
                                   hipStream_t st) {
    if (npre == 0) return hipSuccess;
    const IntegJob none{};
    trace_begin(st, SFOC_K_INTEGRAL);
    hipLaunchKernelGGL(integral_prefix<true>, dim3(npre), dim3(kScanNT), 0, st, none, jobs, pre);
    hipLaunchKernelGGL(integral_tiles<true>, dim3(ntiles), dim3(kScanNT), 0, st, none, jobs, tiles,
                       (uint8_t*)nullptr);
    trace_end(st, SFOC_K_INTEGRAL);
    return hipGetLastError();
}

}  // namespace sfoc
