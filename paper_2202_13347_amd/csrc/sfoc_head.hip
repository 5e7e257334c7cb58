// Learned CP-validity / sub-pixel head: features from the NCC surfaces,
// network forward, backward and Adam, and the inference decision.
//
// A launch of one workgroup per sample carries each sample through the whole
// network (and back, in training) in LDS on the FP32 matrix cores; a second
// launch sums the weight gradients over the batch and applies Adam.  Every sum
// is taken in a fixed order, so every result is bit-reproducible.
#include <hip/hip_runtime.h>
#include <math.h>

#include <type_traits>

#include "sfoc_dev.h"
#include "sfoc_launch.h"
#include "sfoc_trace.h"

namespace sfoc {
namespace head {

constexpr int kCrop = SFOC_HEAD_CROP, kHalf = kCrop / 2, kNStat = SFOC_HEAD_NSTAT, kCh = 32;
constexpr int kS0 = 33, kS1 = 33, kS2 = 17, kS3 = 9, kS4 = 5;   // map sides
constexpr int kFlat = kCh * kS4 * kS4;                           // 800
constexpr int kFcIn = kFlat + kNStat;                            // 808
// Parameter offsets (float32 vector, order of the header).
constexpr int kW1 = 0, kB1 = kW1 + kCh * 9;
constexpr int kW2 = kB1 + kCh, kB2 = kW2 + kCh * kCh * 9;
constexpr int kW3 = kB2 + kCh, kB3 = kW3 + kCh * kCh * 9;
constexpr int kW4 = kB3 + kCh, kB4 = kW4 + kCh * kCh * 9;
constexpr int kF1 = kB4 + kCh, kC1 = kF1 + kCh * kFcIn;
constexpr int kF2 = kC1 + kCh, kC2 = kF2 + 3 * kCh;
constexpr int kNParams = kC2 + 3;
static_assert(kNParams == SFOC_HEAD_PARAMS, "parameter layout");
constexpr float kLambda = 4.0f, kBeta = 0.1f, kClip = 1.5f;
constexpr int kMaxN = 65536;

// To bfloat16 (nearest even) and back, by the conversion instruction.
SFOC_DEV float bf16_round(float w) { return static_cast<float>(static_cast<__bf16>(w)); }
// Orders a wave's LDS writes before its following reads.
SFOC_DEV void wave_order() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
// The thread index laundered through an empty asm: what a phase derives from
// it is recomputed there instead of being hoisted out of the sample loop and
// kept in registers across the other phases.
SFOC_DEV int tid_here() {
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

// ---- network: one workgroup per sample ---------------------------------------
// A sample's whole pass runs in LDS: nothing but the crop and the parameters
// is read from HBM, and in training nothing but the sample's weight-gradient
// partials and the small vectors of the fully connected layers is written.
// The convolutions, their data gradients and their weight gradients are
// products on the FP32 matrix cores (16 x 16 x 4: FP32 operands and sums):
//   forward        D[o][pos]  = sum over (c, tap) of W[o][c][tap] in[c][S pos + tap]
//   data gradient  D[c][pos]  = sum over (o, tap) of W[o][c][tap] g[o][(pos - tap) / S],
//                  one product per parity class of the position (its taps)
//   weight grad.   D[o][c]    = sum over pos of g[o][pos] in[c][S pos + tap], per tap
// The input of conv2 (32 x 33 x 33 floats) would fill the LDS, so conv2 works
// in three bands of output rows and conv1 is computed per band, again in the
// backward pass (9 of 290 multiply-adds a sample).  Every sum has a fixed
// order: results are bit-reproducible.
// A 16 x 16 x 4 product adds its four terms to the sum one after the other,
// each as fmaf does.  So a convolution's sum is the plain loop's, from the bias
// over channels and then taps in one chain of fmaf, and fc1's and fc2's are
// such chains: every activation, and with it what the ReLUs let through of a
// gradient, is defined by that loop and does not depend on the tiling.
// What bounds it: with one workgroup a CU, the LDS reads and the barriers
// between phases; the matrix-core instructions alone (10.8 k of 32 cycles a
// sample in training, a quarter of them on each SIMD) are 36 us.  A training
// step of 256 samples took 2043 us with a thread per output pixel (or weight)
// and every activation in HBM, 138 us now (in a kernel trace this launch 134 us
// and the update 10); the forward pass of 400 samples 153 us and 77 us (two
// rounds of 256 CUs; fc1's chain of 808 is 4 us of each).
typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr int kNetNT = 512, kWaves = kNetNT / 64;
constexpr int kWP = 40;                          // LDS pitch of W[(tap, c)][o] (four rows on 32 banks)
constexpr int kBandRows = 6, kBands = 3;         // conv2 output rows per band
constexpr int kBR = 2 * kBandRows + 1;           // a1 rows of a band
// LDS planes (floats per channel) and row pitches, with a border of zeros
// where the next layer reads past the map.  Odd planes: the 16 channels that
// a matrix operand spans fall on different banks.
constexpr int kP1 = kS1 + 2, kL1 = kBR * kP1;    // a1 band: columns -1 .. 33
constexpr int kP2 = kS2 + 2, kL2 = kP2 * kP2;    // a2 (later its gradient), rows and columns -1 .. 17
constexpr int kP3 = kS3 + 2, kL3 = kP3 * kP3;
constexpr int kL4 = kS4 * kS4;
// Weights of 32 outputs are loaded by 16 lanes an output: no division for an
// element's place (256 samples forward: 47 us with one for each and the registers
// it spilled, 38 us so).
constexpr int kLanes = kNetNT / kCh;
// fc1 in three chunks of inputs: a chunk's weights as float4 [k / 4][o], at a
// pitch that spreads the stores of 16 inputs and 4 outputs over all banks.
constexpr int kFcRows = 288, kFcChunks = 3, kFcPitch = kCh + 2, kFcPad = kFcRows * kFcChunks;
constexpr int kFcRegs = kFcRows / kLanes;
static_assert(kFcPad >= kFcIn && kFcRegs * kLanes == kFcRows && kFcRows % 4 == 0, "fc1 chunks");
constexpr int kPC = kS0 + 2;                     // crop, rows and columns -1 .. 33
static_assert(kL1 % 2 == 1 && kL2 % 2 == 1 && kL3 % 2 == 1 && kL4 % 2 == 1, "odd planes");
constexpr int kConvParams = kF1;                 // conv1..conv4 weights and biases: a prefix of the vector
struct NetLds {
    float w[9 * kCh * kWP];     // the layer's rounded weights [(c, tap)][o], o at weight_col
    float a2[kCh * kL2];
    union {
        float a1[kCh * kL1];
        struct {
            float a3[kCh * kL3];
            float a4[kFcPad];   // then the statistics: fc1's input, zeros to the end
            float4 fw[kFcRows / 4 * kFcPitch];
        };
    };
    float crop[kPC * kPC + 3];
    float w1[9 * kCh];          // conv1 weights [tap][o]
    float bias[3 * kCh];        // of conv2, conv3, conv4
    float f2[3 * kCh];          // fc2 weights [q][o]
    float h1[kCh], dh1[kCh], dout[4];
    int job;
};
static_assert(sizeof(NetLds) <= 160 * 1024 && kWaves * kCh * 16 <= kCh * kL1, "LDS of a CU; the wave sums fit a1");
static_assert(kCh * kL3 + kFcPad + kFcRows * kFcPitch <= kCh * kL1 && kCh * kL3 % 4 == 0, "fc1 in the place of a1");

SFOC_DEV f32x4 mfma4(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

// One layer's weights (32 x 32 x 9): loaded into registers ahead of the phase
// before, then rounded to bfloat16 into w[(c, tap)][o].  Within its row an
// output's place is exchanged by channel, so that the data gradient, whose lanes
// run over the channels, reads from sixteen banks and not from four.
SFOC_DEV int weight_swap(int c) { return 2 * ((c >> 2) & 3); }
SFOC_DEV int weight_col(int o, int c) { return o ^ weight_swap(c); }
constexpr int kWRegs = kCh * 9 / kLanes;
static_assert(kWRegs * kLanes == kCh * 9, "whole rounds");
SFOC_DEV void load_weights(const float* __restrict__ th, float (&v)[kWRegs]) {
    const int t = tid_here();
    const float* p = th + t / kLanes * (kCh * 9) + t % kLanes;
#pragma unroll
    for (int k = 0; k < kWRegs; ++k) v[k] = p[k * kLanes];
}
SFOC_DEV void stage_weights(const float (&v)[kWRegs], float* w) {
    const int t = tid_here(), o = t / kLanes;
#pragma unroll
    for (int k = 0; k < kWRegs; ++k) {
        const int ct = t % kLanes + k * kLanes;
        w[ct * kWP + weight_col(o, ct / 9)] = bf16_round(v[k]);
    }
}

// conv1 (+ ReLU) for the a1 rows r0 .. r0 + kBR - 1 into the band; rows and
// columns outside the map are zero.  Lane o of a half-wave owns output channel
// o and slides along a row.
SFOC_DEV void conv1_band(NetLds& S, const float* __restrict__ th, int r0) {
    const int t = tid_here(), o = t % kCh, grp = t / kCh;
    constexpr int kGrps = kNetNT / kCh, kSeg = 11, kSegs = kS1 / kSeg;
    float w[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) w[k] = S.w1[k * kCh + o];
    const float bias = th[kB1 + o];
    for (int q = grp; q < kBR * kSegs; q += kGrps) {
        const int rr = q / kSegs, x0 = (q - rr * kSegs) * kSeg, y = r0 + rr;
        float* dst = S.a1 + o * kL1 + rr * kP1 + 1 + x0;
        if (x0 == 0) dst[-1] = 0.f;
        if (x0 + kSeg == kS1) dst[kSeg] = 0.f;
        if (y < 0 || y >= kS1) {
#pragma unroll
            for (int x = 0; x < kSeg; ++x) dst[x] = 0.f;
            continue;
        }
        const float* src = S.crop + y * kPC + x0;   // rows y - 1 .. y + 1, columns x0 - 1 ..
        float v[3][kSeg + 2];
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int x = 0; x < kSeg + 2; ++x) v[i][x] = src[i * kPC + x];
#pragma unroll
        for (int x = 0; x < kSeg; ++x) {
            float acc = bias;
#pragma unroll
            for (int i = 0; i < 3; ++i)
#pragma unroll
                for (int j = 0; j < 3; ++j) acc = fmaf(w[i * 3 + j], v[i][x + j], acc);
            dst[x] = fmaxf(acc, 0.f);
        }
    }
}

// Stride-2 convolution + bias + ReLU of `rows` output rows from a zero-bordered
// LDS map `in` (plane LI, pitch PI; its first row is the row above output row
// 0's centre) into `out` (plane LO, pitch PO, first pixel at OO).  A wave takes
// tiles of 16 positions and 16 HALVES channels, one chain of products each.
// Product k = 9 c + tap: lane group g holds k = 4 s + g at step s, so that nine
// steps (four channels) on, its operands lie four planes further: nine offsets a
// lane.  The operands are read as many steps ahead as keep the reads under way
// within the fifteen that a wave can count (256 samples forward: 51 us with nine
// steps' reads at once, 46 us so).
template <int HOUT, int LI, int PI, int LO, int PO, int OO, int HALVES>
SFOC_DEV void conv_tiles(const float* in, const float* w, const float* bias, float* out, int rows) {
    const int t = tid_here(), lane = t & 63, wv = t >> 6, n = lane & 15, g = lane >> 4;
    constexpr int kSplit = 2 / HALVES, kS = 9, kGroups = kCh / 4, kAhead = HALVES == 2 ? 4 : 6;
    const int npos = rows * HOUT, jobs = kSplit * ((npos + 15) / 16);
    int off[kS];
#pragma unroll
    for (int r = 0; r < kS; ++r) {
        const int k = 4 * r + g, c = k / 9, tap = k - c * 9;
        off[r] = c * LI + (tap / 3) * PI + tap % 3;
    }
    for (int job = wv; job < jobs; job += kWaves) {
        const int h0 = job % kSplit, p = (job / kSplit) * 16 + n, pc = min(p, npos - 1);
        const int y = pc / HOUT, x = pc - y * HOUT;
        const float* b0 = in + 2 * y * PI + 2 * x;
        const float* a0 = w + g * kWP + h0 * 16;
        f32x4 acc[HALVES];
#pragma unroll
        for (int h = 0; h < HALVES; ++h)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[h][r] = bias[(h0 + h) * 16 + 4 * g + r];
        const float* ax[4];   // the lane's output in the rows of channels 4 q .. 4 q + 3, by q mod 4
#pragma unroll
        for (int q = 0; q < 4; ++q) ax[q] = a0 + (n ^ weight_swap(4 * q));
        float av[kAhead + 1][HALVES], bv[kAhead + 1];
        auto read = [&](int s) {
            const int q = s / kS, r = s % kS, buf = s % (kAhead + 1);
            bv[buf] = b0[off[r] + 4 * q * LI];
#pragma unroll
            for (int h = 0; h < HALVES; ++h) av[buf][h] = ax[q % 4][4 * s * kWP + 16 * h];
        };
#pragma unroll
        for (int s = 0; s < kAhead; ++s) read(s);
#pragma unroll
        for (int s = 0; s < kS * kGroups; ++s) {
            if (s + kAhead < kS * kGroups) read(s + kAhead);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int h = 0; h < HALVES; ++h) acc[h] = mfma4(av[s % (kAhead + 1)][h], bv[s % (kAhead + 1)], acc[h]);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (p < npos) {
#pragma unroll
            for (int h = 0; h < HALVES; ++h)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    out[((h0 + h) * 16 + 4 * g + r) * LO + OO + y * PO + x] = fmaxf(acc[h][r], 0.f);
        }
    }
}

// Gradient of a stride-2 convolution's input at rows [2 ya, R1) of the map
// `act` (plane LI, pitch PI; pixel (y, x) at OI + (y - y0) PI + x), masked by
// act > 0 and written over it; g is the output gradient (plane LG, pitch PG,
// first pixel at OG).  Position (2a + cy, 2b + cx) gets the taps i = 1 - cy (of
// output row a + cy) and, for cy = 1, i = 2 (of row a); columns likewise: T = 1,
// 2 or 4 taps.  Product k = T o + tap: lane group q holds tap q mod T of outputs
// q / T, q / T + 4 / T, ...  The waves draw (class, 16 positions, 16 channels) tiles from a counter, longest
// first; what a tile computes does not depend on who draws it.
template <int HOUT, int LG, int PG, int OG, int LI, int PI, int OI>
SFOC_DEV void dgrad_tiles(const float* g, const float* w, float* act, int y0, int ya, int R1, int* counter) {
    const int lane = tid_here() & 63, n = lane & 15, q = lane >> 4;
    int ntile[4], first[4], total = 0;   // classes cy, cx = 11, 10, 01, 00
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int cy = k < 2, cx = !(k & 1);
        const int ny = max(0, (R1 - 2 * ya - cy + 1) / 2), nx = HOUT - cx;
        ntile[k] = (ny * nx + 15) / 16;
        first[k] = total;
        total += 2 * ntile[k];
    }
    for (;;) {
        int job = 0;
        if (lane == 0) job = atomicAdd(counter, 1);
        job = __builtin_amdgcn_readfirstlane(job);
        if (job >= total) break;
        const int k = job >= first[3] ? 3 : job >= first[2] ? 2 : job >= first[1] ? 1 : 0;
        const int cy = k < 2, cx = !(k & 1), jk = job - first[k], half = jk & 1;
        const int ny = (R1 - 2 * ya - cy + 1) / 2, nx = HOUT - cx, np = ny * nx;
        const int p = (jk >> 1) * 16 + n, pc = min(p, np - 1), a = pc / nx, b = pc - a * nx;
        const int c = half * 16 + n;
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
        auto run = [&](auto taps) {
            constexpr int T = decltype(taps)::value, kO = 4 / T, kAhead = 6;   // (see conv_tiles)
            const int o0 = q / T, ti = q % T;
            // cy = 0: tap row 1 on row a; cy = 1: 0 on row a + 1, then 2 on row a
            const int iy = T == 4 ? ti >> 1 : cy ? ti : 0, ix = T == 4 ? ti & 1 : cx ? ti : 0;
            const int i = cy ? 2 * iy : 1, j = cx ? 2 * ix : 1;
            const float* gp = g + o0 * LG + OG + (ya + a + (cy && !iy)) * PG + b + (cx && !ix);
            const float* wp = w + (c * 9 + i * 3 + j) * kWP;
            const float* wo[2 * T];   // outputs below 8 of this lane
#pragma unroll
            for (int v = 0; v < 2 * T; ++v) wo[v] = wp + weight_col(o0 + kO * v, c);
            float av[kAhead + 1], bv[kAhead + 1];
            auto read = [&](int os) {
                av[os % (kAhead + 1)] = wo[os % (2 * T)][8 * (os / (2 * T))];
                bv[os % (kAhead + 1)] = gp[kO * os * LG];
            };
#pragma unroll
            for (int os = 0; os < kAhead; ++os) read(os);
#pragma unroll
            for (int os = 0; os < 8 * T; ++os) {
                if (os + kAhead < 8 * T) read(os + kAhead);
                __builtin_amdgcn_sched_barrier(0);
                acc = mfma4(av[os % (kAhead + 1)], bv[os % (kAhead + 1)], acc);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        if (k == 0) run(std::integral_constant<int, 4>{});
        else if (k == 3) run(std::integral_constant<int, 1>{});
        else run(std::integral_constant<int, 2>{});
        if (p < np) {
            const int y = 2 * (ya + a) + cy - y0, x = 2 * b + cx;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                float* d = act + (half * 16 + 4 * q + r) * LI + OI + y * PI + x;
                *d = *d > 0.f ? acc[r] : 0.f;
            }
        }
    }
}

// Weight-gradient tiles of a stride-2 convolution over `rows` output rows: the
// 36 tiles (o half, tap, c half) are dealt to the waves, tile wv + 8 k to
// acc[k] (every wave has one o half, so its g operand serves all its tiles).
constexpr int kWTiles = 36, kWPer = (kWTiles + kWaves - 1) / kWaves;
template <int HOUT, int LG, int PG, int LI, int PI>
SFOC_DEV void wgrad_tiles(const float* g, const float* in, int rows, f32x4 (&acc)[kWPer]) {
    const int td = tid_here(), lane = td & 63, wv = td >> 6, n = lane & 15, q = lane >> 4;
    const int npos = rows * HOUT;
    const float* ga = g + ((wv & 1) * 16 + n) * LG;
    const float* ib[kWPer];
#pragma unroll
    for (int k = 0; k < kWPer; ++k) {
        const int t = min(wv + kWaves * k, kWTiles - 1), tc = t >> 1, tap = tc >> 1, ch = tc & 1;
        ib[k] = in + (ch * 16 + n) * LI + (tap / 3) * PI + tap % 3;
    }
    // position p = q, q + 4, ...; the next two positions' operands are read
    // while the matrix instructions of the two before run
    constexpr int kU = 2;
    int y = q / HOUT, x = q - y * HOUT, p = q;
    float av[kU], bv[kU][kWPer], an[kU], bn[kU][kWPer];
    auto read = [&](float(&a_)[kU], float(&b_)[kU][kWPer]) {
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const bool ok = p < npos;
            const int go = ok ? y * PG + x : 0, off = ok ? 2 * y * PI + 2 * x : 0;
            const float v = ga[go];
            a_[u] = ok ? v : 0.f;
#pragma unroll
            for (int k = 0; k < kWPer; ++k) b_[u][k] = ib[k][off];
            p += 4;
            x += 4;
            if (x >= HOUT) {
                x -= HOUT;
                ++y;
            }
        }
    };
    const int steps = (npos + 4 * kU - 1) / (4 * kU);
    read(av, bv);
    for (int s = 0; s < steps; ++s) {
        read(an, bn);   // (past the last position: zero operands at offset 0)
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < kU; ++u)
#pragma unroll
            for (int k = 0; k < kWPer; ++k)
                if (k + 1 < kWPer || wv + kWaves * k < kWTiles) acc[k] = mfma4(av[u], bv[u][k], acc[k]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            av[u] = an[u];
#pragma unroll
            for (int k = 0; k < kWPer; ++k) bv[u][k] = bn[u][k];
        }
    }
}

// The tiles' sums into the workgroup's partials (added to those of its earlier
// samples), in the parameter order [o][c][tap].
SFOC_DEV void store_wgrad(const f32x4 (&acc)[kWPer], float* __restrict__ part, bool add) {
    const int td = tid_here(), lane = td & 63, wv = td >> 6, n = lane & 15, q = lane >> 4;
#pragma unroll
    for (int k = 0; k < kWPer; ++k) {
        const int t = wv + kWaves * k;
        if (t >= kWTiles) continue;
        const int tc = t >> 1, tap = tc >> 1, c = (tc & 1) * 16 + n;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            float* d = part + (((t & 1) * 16 + 4 * q + r) * kCh + c) * 9 + tap;
            *d = add ? *d + acc[k][r] : acc[k][r];
        }
    }
}

// Bias gradient: sums of a gradient map's rows x cols per channel.
template <int LG, int PG>
SFOC_DEV void store_bgrad(const float* g, int rows, int cols, float* __restrict__ part, bool add) {
    const int t = tid_here(), o = t / 16, k = t % 16;
    float s = 0.f;
    for (int p = k; p < rows * cols; p += 16) s += g[o * LG + (p / cols) * PG + p % cols];
#pragma unroll
    for (int d = 1; d < 16; d <<= 1) s += __shfl_xor(s, d, 64);
    if (k == 0) part[o] = add ? part[o] + s : s;
}

// A chunk of fc1's weights: loaded along the inputs into registers, then rounded
// into fw (zero past the last input).
SFOC_DEV void load_fc(const float* __restrict__ th, int chunk, float (&v)[kFcRegs]) {
    const int t = tid_here(), k0 = chunk * kFcRows + t % kLanes;
    const float* p = th + kF1 + t / kLanes * kFcIn;
#pragma unroll
    for (int i = 0; i < kFcRegs; ++i) {
        const int k = k0 + i * kLanes;
        v[i] = p[min(k, kFcIn - 1)];
        v[i] = k < kFcIn ? v[i] : 0.f;
    }
}
SFOC_DEV void stage_fc(const float (&v)[kFcRegs], float4* fw) {
    const int t = tid_here(), k0 = t % kLanes;
    float* p = reinterpret_cast<float*>(fw + k0 / 4 * kFcPitch + t / kLanes) + k0 % 4;
#pragma unroll
    for (int i = 0; i < kFcRegs; ++i) p[i * (kLanes / 4) * (kFcPitch * 4)] = bf16_round(v[i]);
}
// The chunk's inputs x added to h, output o's sum, in order; the operands are read
// as far ahead as a wave can count (see conv_tiles).  The first operands' places
// in LDS are opaque to the compiler, so that the reads of a round share a base
// register each instead of costing an address add.
SFOC_DEV float fc_chunk(const float4* lds, const float4* fw, const float* x, int o, float h) {
    constexpr int kQuads = kFcRows / 4, kSlots = 8;
    static_assert(kQuads % kSlots == 0, "whole rounds");
    int wi = (int)(fw - lds) + o, xi = (int)(reinterpret_cast<const float4*>(x) - lds);
    asm volatile("" : "+v"(wi), "+v"(xi));
    const float4* wq = lds + wi;
    const float4* xq = lds + xi;
    float4 w[kSlots], v[kSlots];
    auto read = [&](int q, int slot) {
        w[slot] = wq[q * kFcPitch];
        v[slot] = xq[q];
    };
    auto add = [&](int slot) {
        __builtin_amdgcn_sched_barrier(0);
        h = fmaf(w[slot].x, v[slot].x, h);
        h = fmaf(w[slot].y, v[slot].y, h);
        h = fmaf(w[slot].z, v[slot].z, h);
        h = fmaf(w[slot].w, v[slot].w, h);
        __builtin_amdgcn_sched_barrier(0);
    };
#pragma unroll
    for (int u = 0; u + 1 < kSlots; ++u) read(u, u);
#pragma unroll 1
    for (int q = 0; q + kSlots < kQuads; q += kSlots)
#pragma unroll
        for (int u = 0; u < kSlots; ++u) {
            read(q + u + kSlots - 1, (u + kSlots - 1) % kSlots);
            add(u);
        }
    read(kQuads - 1, kSlots - 1);
#pragma unroll
    for (int u = 0; u < kSlots; ++u) add(u);
    return h;
}

// ---- loss and its gradient w.r.t. the outputs -------------------------------
SFOC_DEV float sigmoidf_(float l) {
    const float e = __expf(-fabsf(l));
    return l >= 0.f ? 1.f / (1.f + e) : e / (1.f + e);
}
SFOC_DEV float smooth_l1(float d) {
    const float a = fabsf(d);
    return a < kBeta ? 0.5f * d * d / kBeta : a - 0.5f * kBeta;
}
SFOC_DEV float smooth_l1_grad(float d) { return fabsf(d) < kBeta ? d / kBeta : (d > 0.f ? 1.f : -1.f); }

constexpr uint32_t kEligible = SFOC_CP_VALID | SFOC_CP_INCONSISTENT;

// The decision on a CP record (inference).
SFOC_DEV void apply_decision(sfoc_cp* __restrict__ cps, int i, const float* out, float threshold) {
    sfoc_cp c = cps[i];
    if (!(c.flags & kEligible)) return;
    const float p = sigmoidf_(out[0]);
    c.flags = (c.flags & ~kEligible) | SFOC_CP_LEARNED | (p >= threshold ? SFOC_CP_VALID : SFOC_CP_INCONSISTENT);
    c.sub_dy = fminf(kClip, fmaxf(-kClip, out[1]));
    c.sub_dx = fminf(kClip, fmaxf(-kClip, out[2]));
    cps[i] = c;
}

struct NetArgs {
    const float* th;
    const float* crops;
    const float* stats;
    int n;
    float* out;            // n x 3
    sfoc_cp* cps;          // inference: records the decision applies to, or null
    float threshold;
    const float* label;    // training
    const float* target;
    float* x4;             // n x 800: fc1's input
    float* h1;             // n x 32
    float* dh1;            // n x 32
    float* dout;           // n x 3
    float* loss;           // n
    float* part;           // [workgroup][kConvParams]
};

template <bool TRAIN>
__global__ __launch_bounds__(kNetNT, 2) void net_kernel(const NetArgs A) {
    extern __shared__ float4 lds_raw[];
    NetLds& S = *reinterpret_cast<NetLds*>(lds_raw);
    const int t = threadIdx.x, lane = t & 63;
    const float* __restrict__ th = A.th;
    if (t < 9 * kCh) S.w1[(t % 9) * kCh + t / 9] = bf16_round(th[kW1 + t]);
    if (t < kCh) {
        S.bias[t] = th[kB2 + t];
        S.bias[kCh + t] = th[kB3 + t];
        S.bias[2 * kCh + t] = th[kB4 + t];
    }
    if (t < 3 * kCh) S.f2[t] = bf16_round(th[kF2 + t]);
    for (int b = blockIdx.x; b < A.n; b += gridDim.x) {
        const bool add = b != (int)blockIdx.x;   // later samples add to the partials
        __syncthreads();
        const float* crop = A.crops + (size_t)b * kS0 * kS0;
#pragma unroll
        for (int e = t; e < kPC * kPC; e += kNetNT) {
            const int y = e / kPC - 1, x = e % kPC - 1;
            S.crop[e] = y >= 0 && y < kS0 && x >= 0 && x < kS0 ? crop[y * kS0 + x] : 0.f;
        }
        for (int e = t; e < kCh * kL2; e += kNetNT) S.a2[e] = 0.f;
        const float stat = A.stats[(size_t)b * kNStat + min(t, kNStat - 1)];
        float wr[kWRegs], fr[kFcRegs];
        load_weights(th + kW2, wr);
        stage_weights(wr, S.w);
        load_weights(th + kW3, wr);
        __syncthreads();
        // conv1, conv2 by bands of rows
        for (int band = 0; band < kBands; ++band) {
            const int r0 = band * kBandRows, rows = min(kBandRows, kS2 - r0);
            conv1_band(S, th, 2 * r0 - 1);
            __syncthreads();
            conv_tiles<kS2, kL1, kP1, kL2, kP2, kP2 + 1, 2>(S.a1, S.w, S.bias, S.a2 + r0 * kP2, rows);
            __syncthreads();
        }
        for (int e = t; e < kCh * kL3; e += kNetNT) S.a3[e] = 0.f;
        if (t < kFcPad - kFlat) S.a4[kFlat + t] = t < kNStat ? stat : 0.f;
        stage_weights(wr, S.w);
        load_weights(th + kW4, wr);
        load_fc(th, 0, fr);
        __syncthreads();
        conv_tiles<kS3, kL2, kP2, kL3, kP3, kP3 + 1, 1>(S.a2, S.w, S.bias + kCh, S.a3, kS3);
        __syncthreads();
        stage_weights(wr, S.w);
        stage_fc(fr, S.fw);
        if (TRAIN) load_weights(th + kW3, wr);
        load_fc(th, 1, fr);
        __syncthreads();
        conv_tiles<kS4, kL3, kP3, kL4, kS4, 0, 1>(S.a3, S.w, S.bias + 2 * kCh, S.a4, kS4);
        __syncthreads();
        // fc1 (lane o of the first wave output o), then fc2 (lane q output q)
        {
            float h = t < kCh ? th[kC1 + t] : 0.f;
            for (int chunk = 0; chunk < kFcChunks; ++chunk) {
                if (chunk) {
                    stage_fc(fr, S.fw);
                    if (chunk + 1 < kFcChunks) load_fc(th, chunk + 1, fr);
                    __syncthreads();
                }
                if (t < kCh) h = fc_chunk(lds_raw, S.fw, S.a4 + chunk * kFcRows, t, h);
                if (chunk + 1 < kFcChunks) __syncthreads();
            }
            if (t < kCh) S.h1[t] = fmaxf(h, 0.f);
        }
        wave_order();   // fc2 reads what lanes of its own wave wrote
        if (t < 64) {
            const int ql = min(lane, 2);
            float v = th[kC2 + ql];
#pragma unroll
            for (int o = 0; o < kCh; ++o) v = fmaf(S.f2[ql * kCh + o], S.h1[o], v);
            float s[3];
#pragma unroll
            for (int q = 0; q < 3; ++q) s[q] = __shfl(v, q, 64);
            if (lane == 0) {
                float o[3];
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    o[q] = s[q];
                    if (A.out) A.out[(size_t)b * 3 + q] = o[q];
                }
                if constexpr (!TRAIN) {
                    if (A.cps) apply_decision(A.cps, b, o, A.threshold);
                } else {
                    const float inv = 1.0f / (float)A.n;
                    const float l = o[0], y = A.label[b];
                    const float dy = o[1] - A.target[2 * b], dx = o[2] - A.target[2 * b + 1];
                    const float bce = fmaxf(l, 0.f) - l * y + log1pf(__expf(-fabsf(l)));
                    A.loss[b] = bce + kLambda * y * (smooth_l1(dy) + smooth_l1(dx));
                    S.dout[0] = (sigmoidf_(l) - y) * inv;
                    S.dout[1] = kLambda * y * smooth_l1_grad(dy) * inv;
                    S.dout[2] = kLambda * y * smooth_l1_grad(dx) * inv;
#pragma unroll
                    for (int q = 0; q < 3; ++q) A.dout[(size_t)b * 3 + q] = S.dout[q];
                    S.job = 0;
                }
            }
        }
        if constexpr (TRAIN) {
            float* __restrict__ part = A.part + (size_t)blockIdx.x * kConvParams;
            __syncthreads();
            if (t < kCh) {
                float g = 0.f;
#pragma unroll
                for (int q = 0; q < 3; ++q) g = fmaf(S.f2[q * kCh + t], S.dout[q], g);
                const float h = S.h1[t], d = h > 0.f ? g : 0.f;
                S.dh1[t] = d;
                A.h1[(size_t)b * kCh + t] = h;
                A.dh1[(size_t)b * kCh + t] = d;
            }
            __syncthreads();
            // gradient of conv4's output over a4 (kept in HBM as fc1's input)
            for (int k = t; k < kFlat; k += kNetNT) {
                float g = 0.f;
#pragma unroll
                for (int o = 0; o < kCh; ++o) g = fmaf(bf16_round(th[kF1 + o * kFcIn + k]), S.dh1[o], g);
                const float a = S.a4[k];
                A.x4[(size_t)b * kFlat + k] = a;
                S.a4[k] = a > 0.f ? g : 0.f;
            }
            __syncthreads();
            f32x4 acc[kWPer];
            auto clear = [&]() {
#pragma unroll
                for (int k = 0; k < kWPer; ++k) acc[k] = f32x4{0.f, 0.f, 0.f, 0.f};
            };
            // conv4: weight and bias gradients, then the gradient over a3
            clear();
            wgrad_tiles<kS4, kL4, kS4, kL3, kP3>(S.a4, S.a3, kS4, acc);
            store_wgrad(acc, part + kW4, add);
            store_bgrad<kL4, kS4>(S.a4, kS4, kS4, part + kB4, add);
            __syncthreads();
            dgrad_tiles<kS4, kL4, kS4, 0, kL3, kP3, kP3 + 1>(S.a4, S.w, S.a3, 0, 0, kS3, &S.job);
            __syncthreads();
            // conv3
            stage_weights(wr, S.w);
            load_weights(th + kW2, wr);
            if (t == 0) S.job = 0;
            clear();
            wgrad_tiles<kS3, kL3, kP3, kL2, kP2>(S.a3 + kP3 + 1, S.a2, kS3, acc);
            store_wgrad(acc, part + kW3, add);
            store_bgrad<kL3, kP3>(S.a3 + kP3 + 1, kS3, kS3, part + kB3, add);
            __syncthreads();
            dgrad_tiles<kS3, kL3, kP3, kP3 + 1, kL2, kP2, kP2 + 1>(S.a3, S.w, S.a2, 0, 0, kS2, &S.job);
            __syncthreads();
            // conv2 and conv1 by the same bands: a1 again, conv2's weight
            // gradient, the gradient over the band's own a1 rows, and conv1's
            // weight gradient D[o][tap] = sum da1[o][pos] crop[pos + tap] with
            // a constant one as tap 9 (the bias)
            stage_weights(wr, S.w);
            store_bgrad<kL2, kP2>(S.a2 + kP2 + 1, kS2, kS2, part + kB2, add);
            clear();
            f32x4 acc1[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
            const int n = lane & 15, q = lane >> 4, wv = t >> 6;
            for (int band = 0; band < kBands; ++band) {
                const int r0 = band * kBandRows, rows = min(kBandRows, kS2 - r0);
                const int a0 = 2 * r0, a1 = min(2 * (r0 + rows), kS1);   // the band's own a1 rows
                conv1_band(S, th, a0 - 1);
                if (t == 0) S.job = 0;
                __syncthreads();
                wgrad_tiles<kS2, kL2, kP2, kL1, kP1>(S.a2 + (r0 + 1) * kP2 + 1, S.a1, rows, acc);
                __syncthreads();
                dgrad_tiles<kS2, kL2, kP2, kP2 + 1, kL1, kP1, 1>(S.a2, S.w, S.a1, a0 - 1, r0, a1, &S.job);
                __syncthreads();
                const int npos = (a1 - a0) * kS1;
                const int tap = min(n, 8);
                const float* cr = S.crop + (a0 + tap / 3) * kPC + tap % 3;
                for (int p0 = 4 * wv; p0 < npos; p0 += 4 * kWaves) {
                    const int p = p0 + q, pc = min(p, npos - 1), y = pc / kS1, x = pc - y * kS1;
                    const bool ok = p < npos;
                    const float bv = n < 9 ? cr[y * kPC + x] : (n == 9 ? 1.f : 0.f);
                    const float* ap = S.a1 + n * kL1 + (y + 1) * kP1 + x + 1;
#pragma unroll
                    for (int h = 0; h < 2; ++h) acc1[h] = mfma4(ok ? ap[h * 16 * kL1] : 0.f, bv, acc1[h]);
                }
                __syncthreads();
            }
            store_wgrad(acc, part + kW2, add);
            // conv1: the waves' sums in wave order (a1 is dead)
            float* red = S.a1;
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int r = 0; r < 4; ++r) red[(wv * kCh + h * 16 + 4 * q + r) * 16 + n] = acc1[h][r];
            __syncthreads();
            for (int e = t; e < kCh * 10; e += kNetNT) {
                const int o = e / 10, tap = e - o * 10;
                float s = 0.f;
                for (int w = 0; w < kWaves; ++w) s += red[(w * kCh + o) * 16 + tap];
                float* d = part + (tap < 9 ? kW1 + o * 9 + tap : kB1 + o);
                *d = add ? *d + s : s;
            }
        }
    }
}

// ---- gradients over the batch and Adam ------------------------------------------
struct UpdateArgs {
    float* th;
    float* m;
    float* v;
    float* grad;           // kNParams
    float* loss;           // one float, or null
    const float* part;     // [parts][kConvParams]
    const float* x4;
    const float* stats;
    const float* h1;
    const float* dh1;
    const float* dout;
    const float* sloss;    // per sample
    int n, parts;
    float lr, c1, c2;
};

SFOC_DEV void adam_step(const UpdateArgs& A, int e, float g) {
    A.grad[e] = g;
    const float mm = 0.9f * A.m[e] + 0.1f * g;
    const float vv = 0.999f * A.v[e] + 0.001f * g * g;
    A.m[e] = mm;
    A.v[e] = vv;
    A.th[e] -= A.lr * (mm * A.c1) / (sqrtf(vv * A.c2) + 1e-8f);
}

// Workgroups of 64 entries x 4 slices of the sum (over the partials, or over
// the batch); the slices are added in order.  First the convolutions, then
// fc1's weights (eight groups of four outputs x 64 inputs), the other vectors
// (a wave an entry) and the loss.
constexpr int kUpNT = 256, kUpE = 64, kUpS = kUpNT / kUpE;
constexpr int kUpConv = (kConvParams + kUpE - 1) / kUpE;
constexpr int kUpK = (kFcIn + kUpE - 1) / kUpE, kUpO = 4, kUpFc = (kCh / kUpO) * kUpK;
constexpr int kUpVecN = 4 * kCh + 3, kUpVec = (kUpVecN + kUpNT / 64 - 1) / (kUpNT / 64);
__global__ __launch_bounds__(kUpNT) void update_kernel(const UpdateArgs A) {
    __shared__ float red[kUpS][kUpO][kUpE];
    __shared__ double redl[kUpNT];
    const int t = threadIdx.x, i = t % kUpE, s = t / kUpE;
    int blk = blockIdx.x;
    if (blk < kUpConv) {
        const int e = blk * kUpE + i, ec = min(e, kConvParams - 1);
        const int per = (A.parts + kUpS - 1) / kUpS, k0 = s * per, k1 = min(A.parts, k0 + per);
        float a = 0.f;
#pragma unroll 16
        for (int k = k0; k < k1; ++k) a += A.part[(size_t)k * kConvParams + ec];
        red[s][0][i] = a;
        __syncthreads();
        if (s == 0 && e < kConvParams) {
            for (int q = 1; q < kUpS; ++q) a += red[q][0][i];
            adam_step(A, e, a);
        }
        return;
    }
    blk -= kUpConv;
    const int per = (A.n + kUpS - 1) / kUpS, b0 = s * per, b1 = min(A.n, b0 + per);
    if (blk < kUpFc) {
        const int o0 = (blk / kUpK) * kUpO, k = (blk % kUpK) * kUpE + i;
        const float* x = k < kFlat ? A.x4 + k : A.stats + min(k - kFlat, kNStat - 1);
        const size_t pitch = k < kFlat ? kFlat : kNStat;
        float a[kUpO] = {};
#pragma unroll 8
        for (int b = b0; b < b1; ++b) {
            const float xv = x[b * pitch];
            const float4 d = *reinterpret_cast<const float4*>(A.dh1 + (size_t)b * kCh + o0);
            a[0] = fmaf(d.x, xv, a[0]);
            a[1] = fmaf(d.y, xv, a[1]);
            a[2] = fmaf(d.z, xv, a[2]);
            a[3] = fmaf(d.w, xv, a[3]);
        }
#pragma unroll
        for (int o = 0; o < kUpO; ++o) red[s][o][i] = a[o];
        __syncthreads();
        // slice s finishes output o0 + s
        float g = 0.f;
        for (int q = 0; q < kUpS; ++q) g += red[q][s][i];
        if (k < kFcIn) adam_step(A, kF1 + (o0 + s) * kFcIn + k, g);
        return;
    }
    blk -= kUpFc;
    if (blk < kUpVec) {   // fc1 biases (0..31), fc2 weights (32..127), fc2 biases (128..130): a wave each
        const int r = blk * (kUpNT / 64) + t / 64, lane = t % 64;
        if (r >= kUpVecN) return;
        float g = 0.f;
        for (int b = lane; b < A.n; b += 64) {
            if (r < kCh) g += A.dh1[(size_t)b * kCh + r];
            else if (r < 4 * kCh) g = fmaf(A.dout[(size_t)b * 3 + r / kCh - 1], A.h1[(size_t)b * kCh + r % kCh], g);
            else g += A.dout[(size_t)b * 3 + r - 4 * kCh];
        }
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) g += __shfl_xor(g, d, 64);
        if (lane == 0) adam_step(A, r < kCh ? kC1 + r : r < 4 * kCh ? kF2 + r - kCh : kC2 + r - 4 * kCh, g);
        return;
    }
    double a = 0.0;
    for (int b = t; b < A.n; b += kUpNT) a += (double)A.sloss[b];
    redl[t] = a;
    __syncthreads();
    for (int d = kUpNT / 2; d > 0; d >>= 1) {
        if (t < d) redl[t] += redl[t + d];
        __syncthreads();
    }
    if (t == 0) A.loss[0] = (float)(redl[0] / A.n);
}

// ---- features -------------------------------------------------------------
template <int DT>
SFOC_DEV float ld_desc(const void* p, int64_t i) {
    if (DT == SFOC_DTYPE_F32) return ((const float*)p)[i];
    if (DT == SFOC_DTYPE_BF16) return bf16_bits_to_f32(((const uint16_t*)p)[i]);
    return f16_bits_to_f32(((const uint16_t*)p)[i]);
}

struct FeatArgs {
    const void* desc_sen;
    const double* integ1;
    const double* integ2;
    const int32_t* ips;
    const int32_t* prior;
    const float* ncc;
    const sfoc_cp* cps;
    float* crops;
    float* stats;
    int64_t Hs, Ws, Wr;
    int z, m, r;
};

constexpr int kFeatNT = 1024;
template <int DT>
__global__ __launch_bounds__(kFeatNT) void features_kernel(const FeatArgs A) {
    __shared__ double rd[4][kFeatNT];
    __shared__ float rmax[kFeatNT];
    const int i = blockIdx.x, t = threadIdx.x;
    const sfoc_cp cp = A.cps[i];
    float* crop = A.crops + (size_t)i * kCrop * kCrop;
    float* st = A.stats + (size_t)i * kNStat;
    if (!(cp.flags & kEligible)) {
        for (int e = t; e < kCrop * kCrop; e += kFeatNT) crop[e] = 0.f;
        if (t < kNStat) st[t] = 0.f;
        return;
    }
    const int r = A.r, m = A.m, V = 2 * r + 1;
    const int u = cp.dy + r, v = cp.dx + r;
    const float* S = A.ncc + (size_t)i * V * V;
    for (int e = t; e < kCrop * kCrop; e += kFeatNT) {
        const int a = e / kCrop, b = e - a * kCrop;
        const int y = u - kHalf + a, x = v - kHalf + b;
        crop[e] = (y >= 0 && y < V && x >= 0 && x < V) ? S[y * V + x] : -1.f;
    }
    // surface sums and the best value outside the 3 x 3 block
    double s1 = 0.0, s2 = 0.0;
    float best = -1.f;
    for (int e = t; e < V * V; e += kFeatNT) {
        const int y = e / V, x = e - y * V;
        const float s = S[e];
        s1 += s;
        s2 += (double)s * s;
        if ((abs(y - u) > 1 || abs(x - v) > 1) && s > best) best = s;
    }
    // template sums (Eq. 12)
    const int py = A.ips[2 * i], px = A.ips[2 * i + 1];
    const int64_t ty = (int64_t)py - m / 2, tx = (int64_t)px - m / 2;
    const int64_t plane = A.Hs * A.Ws;
    double t1 = 0.0, t2 = 0.0;
    const int mm = m * m;
    // A thread takes template positions q = t, t + kFeatNT, ... and, for each,
    // all channels: one division per position instead of two per element,
    // eight channels' loads in flight per step.  The summation order is
    // fixed (position, then channel), so the sums are reproducible.
    for (int q = t; q < mm; q += kFeatNT) {
        const int yy = q / m, xx = q - yy * m;
        const int64_t pos = (ty + yy) * A.Ws + tx + xx;
        for (int h0 = 0; h0 < A.z; h0 += 8) {
            double d[8];
#pragma unroll
            for (int k = 0; k < 8; ++k)
                d[k] = h0 + k < A.z ? (double)ld_desc<DT>(A.desc_sen, (h0 + k) * plane + pos) : 0.0;
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                t1 += d[k];
                t2 += d[k] * d[k];
            }
        }
    }
    rd[0][t] = s1;
    rd[1][t] = s2;
    rd[2][t] = t1;
    rd[3][t] = t2;
    rmax[t] = best;
    __syncthreads();
    for (int s = kFeatNT / 2; s > 0; s >>= 1) {
        if (t < s) {
#pragma unroll
            for (int k = 0; k < 4; ++k) rd[k][t] += rd[k][t + s];
            rmax[t] = fmaxf(rmax[t], rmax[t + s]);
        }
        __syncthreads();
    }
    if (t == 0) {
        const double n = (double)V * V;
        const double mean = rd[0][0] / n;
        const double var = fmax(rd[1][0] / n - mean * mean, 0.0);
        const double mnz = (double)m * m * A.z;
        const double RT = rd[2][0], RTT = rd[3][0];
        const double varT = RTT - RT * RT / mnz;
        const int pry = A.prior ? A.prior[2 * i] : 0, prx = A.prior ? A.prior[2 * i + 1] : 0;
        const int64_t y = ty - r + pry + u, x = tx - r + prx + v;   // search window at the peak
        const int64_t IW = A.Wr + 1;
        const int64_t a00 = y * IW + x, a01 = a00 + m, a10 = a00 + (int64_t)m * IW, a11 = a10 + m;
        const double RS = A.integ1[a11] - A.integ1[a10] - A.integ1[a01] + A.integ1[a00];
        const double RSS = A.integ2[a11] - A.integ2[a10] - A.integ2[a01] + A.integ2[a00];
        const double varS = RSS - RS * RS / mnz;
        const float c0 = S[u * V + v];
        const double d0 = c0;
        const double curv = 0.5 * (((double)S[(u - 1) * V + v] - 2.0 * d0 + S[(u + 1) * V + v]) +
                                   ((double)S[u * V + v - 1] - 2.0 * d0 + S[u * V + v + 1]));
        st[0] = c0;
        st[1] = rmax[0];
        st[2] = (float)mean;
        st[3] = (float)sqrt(var);
        st[4] = (float)sqrt(fmax(varT, 0.0) / mnz);
        st[5] = (float)sqrt(fmax(varS, 0.0) / mnz);
        st[6] = (float)(RT / mnz);
        st[7] = (float)curv;
    }
}

// ---- workspace ------------------------------------------------------------
struct Layout {
    size_t out;   // (not used: an inference's workspace keeps its size, and a short or null one is refused)
    size_t x4, h1, dh1, dout, loss, part, grad, total;       // training
    int parts;
};

static size_t take(size_t& off, size_t floats) {
    const size_t o = off;
    off = align_up(off + floats * sizeof(float), 256);
    return o;
}

// Workgroups of a training launch: one a sample up to one a CU (a workgroup
// fills a CU's LDS), so that the partials stay within 29 MB.
constexpr int kMaxParts = 256;

static Layout layout(int n, bool train) {
    Layout L{};
    size_t off = 0;
    L.out = take(off, (size_t)n * 3);
    L.parts = n < kMaxParts ? n : kMaxParts;
    if (train) {
        L.x4 = take(off, (size_t)n * kFlat);
        L.h1 = take(off, (size_t)n * kCh);
        L.dh1 = take(off, (size_t)n * kCh);
        L.dout = take(off, (size_t)n * 3);
        L.loss = take(off, (size_t)n);
        L.part = take(off, (size_t)L.parts * kConvParams);
        L.grad = take(off, kNParams);
    }
    L.total = off;
    return L;
}

template <bool TRAIN>
static hipError_t launch_net(const NetArgs& a, int blocks, int trace, hipStream_t st) {
    auto kern = net_kernel<TRAIN>;
    hipError_t e = ensure_dynamic_lds((const void*)kern, (int)sizeof(NetLds));
    if (e != hipSuccess) return e;
    trace_begin(st, trace);
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(kNetNT), sizeof(NetLds), st, a);
    trace_end(st, trace);
    return hipGetLastError();
}

static hipError_t forward(const float* th, const float* crops, const float* stats, int n, float* out, sfoc_cp* cps,
                          float threshold, hipStream_t st) {
    NetArgs a{};
    a.th = th;
    a.crops = crops;
    a.stats = stats;
    a.n = n;
    a.out = out;
    a.cps = cps;
    a.threshold = threshold;
    return launch_net<false>(a, n, SFOC_K_HEAD_FWD, st);
}

}  // namespace head
}  // namespace sfoc

using namespace sfoc;
using namespace sfoc::head;

extern "C" {

int sfoc_head_workspace(int32_t n, int32_t train, size_t* bytes) {
    if (!bytes || n < 0) return SFOC_E_INVALID_ARG;
    if (n > kMaxN) return SFOC_E_UNSUPPORTED;
    *bytes = layout(n, train != 0).total;
    return SFOC_OK;
}

int sfoc_head_features(const void* desc_sen, int64_t Hs, int64_t Ws, const double* integ1, const double* integ2,
                       int64_t Hr, int64_t Wr, int32_t z, int32_t dtype, const int32_t* ips, const int32_t* prior,
                       int32_t n, int32_t m, int32_t r, const float* ncc, const sfoc_cp* cps, float* crops,
                       float* stats, void* stream) {
    int rc = check_match_shape(n, m, r);
    if (rc) return rc;
    if (z < 1 || dtype_size(dtype) == 0 || Hs < 1 || Ws < 1 || Hr < 1 || Wr < 1) return SFOC_E_INVALID_ARG;
    if (Hs > kMaxSide || Ws > kMaxSide || Hr > kMaxSide || Wr > kMaxSide) return SFOC_E_UNSUPPORTED;
    if (n == 0) return SFOC_OK;
    if (!desc_sen || !integ1 || !integ2 || !ips || !ncc || !cps || !crops || !stats) return SFOC_E_INVALID_ARG;
    FeatArgs A{desc_sen, integ1, integ2, ips, prior, ncc, cps, crops, stats, Hs, Ws, Wr, z, m, r};
    hipStream_t st = (hipStream_t)stream;
    trace_begin(st, SFOC_K_HEAD_FEAT);
    if (dtype == SFOC_DTYPE_F32) hipLaunchKernelGGL(features_kernel<SFOC_DTYPE_F32>, dim3(n), dim3(kFeatNT), 0, st, A);
    else if (dtype == SFOC_DTYPE_BF16) hipLaunchKernelGGL(features_kernel<SFOC_DTYPE_BF16>, dim3(n), dim3(kFeatNT), 0, st, A);
    else hipLaunchKernelGGL(features_kernel<SFOC_DTYPE_F16>, dim3(n), dim3(kFeatNT), 0, st, A);
    trace_end(st, SFOC_K_HEAD_FEAT);
    return hip_status(hipGetLastError());
}

int sfoc_head_forward(const float* params, const float* crops, const float* stats, int32_t n, float* out, void* ws,
                      size_t ws_bytes, void* stream) {
    if (n < 0) return SFOC_E_INVALID_ARG;
    if (n > kMaxN) return SFOC_E_UNSUPPORTED;
    if (n == 0) return SFOC_OK;
    if (!params || !crops || !stats || !out || !ws) return SFOC_E_INVALID_ARG;
    const Layout L = layout(n, false);
    if (ws_bytes < L.total) return SFOC_E_WORKSPACE;
    return hip_status(forward(params, crops, stats, n, out, nullptr, 0.f, (hipStream_t)stream));
}

int sfoc_head_infer(const float* params, const float* crops, const float* stats, int32_t n, float threshold,
                    sfoc_cp* cps, float* out, void* ws, size_t ws_bytes, void* stream) {
    if (n < 0 || !(threshold >= 0.f && threshold <= 1.f)) return SFOC_E_INVALID_ARG;
    if (n > kMaxN) return SFOC_E_UNSUPPORTED;
    if (n == 0) return SFOC_OK;
    if (!params || !crops || !stats || !cps || !ws) return SFOC_E_INVALID_ARG;
    const Layout L = layout(n, false);
    if (ws_bytes < L.total) return SFOC_E_WORKSPACE;
    return hip_status(forward(params, crops, stats, n, out, cps, threshold, (hipStream_t)stream));
}

int sfoc_head_train_step(float* params, float* adam_m, float* adam_v, int32_t t, float lr, const float* crops,
                         const float* stats, const float* label, const float* target, int32_t n, float* grad,
                         float* loss, void* ws, size_t ws_bytes, void* stream) {
    if (n < 0 || t < 1 || !(lr >= 0.f)) return SFOC_E_INVALID_ARG;
    if (n > kMaxN) return SFOC_E_UNSUPPORTED;
    if (n == 0) return SFOC_OK;
    if (!params || !adam_m || !adam_v || !crops || !stats || !label || !target || !ws) return SFOC_E_INVALID_ARG;
    const Layout L = layout(n, true);
    if (ws_bytes < L.total) return SFOC_E_WORKSPACE;
    char* w = (char*)ws;
    hipStream_t st = (hipStream_t)stream;
    NetArgs a{};
    a.th = params;
    a.crops = crops;
    a.stats = stats;
    a.n = n;
    a.label = label;
    a.target = target;
    a.x4 = (float*)(w + L.x4);
    a.h1 = (float*)(w + L.h1);
    a.dh1 = (float*)(w + L.dh1);
    a.dout = (float*)(w + L.dout);
    a.loss = (float*)(w + L.loss);
    a.part = (float*)(w + L.part);
    hipError_t e = launch_net<true>(a, L.parts, SFOC_K_HEAD_BWD, st);
    if (e != hipSuccess) return hip_status(e);
    UpdateArgs u{};
    u.th = params;
    u.m = adam_m;
    u.v = adam_v;
    u.grad = grad ? grad : (float*)(w + L.grad);
    u.loss = loss;
    u.part = a.part;
    u.x4 = a.x4;
    u.stats = stats;
    u.h1 = a.h1;
    u.dh1 = a.dh1;
    u.dout = a.dout;
    u.sloss = a.loss;
    u.n = n;
    u.parts = L.parts;
    u.lr = lr;
    // bias corrections in double on the host
    u.c1 = (float)(1.0 / (1.0 - pow(0.9, (double)t)));
    u.c2 = (float)(1.0 / (1.0 - pow(0.999, (double)t)));
    trace_begin(st, SFOC_K_HEAD_ADAM);
    hipLaunchKernelGGL(update_kernel, dim3(kUpConv + kUpFc + kUpVec + (loss ? 1 : 0)), dim3(kUpNT), 0, st, u);
    trace_end(st, SFOC_K_HEAD_ADAM);
    return hip_status(hipGetLastError());
}

}  // extern "C"
