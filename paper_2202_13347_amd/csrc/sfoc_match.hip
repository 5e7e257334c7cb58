// Fast-NCC_SFOC CP detection (Section 2.2, Eq. 9-16; Section 3.2.2) on gfx950.
//
// One workgroup per interest point.  For each descriptor channel h the
// template T_h (m x m, zero padded) and the search window S_h (M x M) get a
// real 2-D FFT of side L >= M, with the spectrum product F(S_h) conj(F(T_h))
// summed over channels in registers; summing in the spectrum is exact by
// linearity, so one inverse transform gives R_ST (Eq. 10, 13).
//
// Each length-L transform is a two-pass Cooley-Tukey with L = NA * NB:
//   pass A: a thread holds x[n1 + NB*n2], n2 = 0..NA-1, does an NA-point
//           DFT in registers and applies the twiddle W_L^(n1*k2);
//   pass B: a thread holds those results for two mirrored columns k2 and
//           NA - k2 and does NB-point DFTs, so it ends with the bins k and
//           L - k together.
// Rows of the window are real: two rows form one complex row, and the two
// half spectra are separated in the thread that holds k and L - k.  Of the
// column transforms, the DC and Nyquist columns (both real) are packed into
// one complex column and separated the same way.  The spectrum of T_h and
// the running sum over channels stay in registers; one LDS buffer of
// L x (L/2 + 1) complex values (padded) carries each 2-D transform.
//
// R_S and R_SS come from four lookups in the float64 integral images of the
// reference descriptor (Eq. 16); R_T and R_TT are accumulated in float64
// while the template is read.  NCC (Eq. 9) is assembled with the variance
// subtraction in float64, then the argmax, the parabola refinement and the
// per-CP flags are written.
#include <type_traits>

#include "sfoc_dev.h"
#include "sfoc_launch.h"
#include "sfoc_trace.h"

namespace sfoc {

// Per-block flags of a split surface.
constexpr int kBlkNonflat = 1, kBlkNonfin = 2, kBlkFlatT = 4, kBlkBadT = 8, kBlkOOB = 16;

// Keeps the scheduler from moving work across stage boundaries (it would
// otherwise hoist the next stage's global loads and raise register pressure).
SFOC_DEV void stage_fence() { __builtin_amdgcn_sched_barrier(0); }
// The thread index laundered through an empty asm: index arithmetic derived
// from it is recomputed inside each stage instead of being hoisted out of
// the channel loop and kept live (which costs registers, then spills).
SFOC_DEV int tid_local() {
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

// Complex products.  Each part is a sum of two products of which one is
// rounded before the fused multiply-add; which one is spelled out here and in
// the tables of the DFT codelets below instead of being left to the compiler.
// So every kernel built from these pieces rounds alike (the pair call, its
// split and spread forms, the plan's kernels), and a change of the code around
// them does not move a result.  The choices are those that the compiler had made
// before they were written out, so the bits are the same at every side.  At
// side 64 that takes two forms, by the half of its pass that a task lies in
// (dft8's hi): 64-side matches from bfloat16 take 0.5 % longer for it (4000 IPs,
// m 32, r 16: 471 to 473 us), others as long.
//   form & 2: the real part fuses the imaginary product, form & 1: the
//   imaginary part fuses a.x * b.y.
SFOC_DEV float2 cmulf(float2 a, float2 b, int form) {
    const float re = form & 2 ? fmaf(a.y, -b.y, a.x * b.x) : fmaf(a.x, b.x, -(a.y * b.y));
    const float im = form & 1 ? fmaf(a.x, b.y, a.y * b.x) : fmaf(a.y, b.x, a.x * b.y);
    return make_float2(re, im);
}
// Twiddle products: row passes, forward column pass, inverse passes (a * conj(w)).
SFOC_DEV float2 cmul_row(float2 a, float2 w) { return cmulf(a, w, 0); }
SFOC_DEV float2 cmul_col(float2 a, float2 w) { return cmulf(a, w, 1); }
SFOC_DEV float2 cmul_inv(float2 a, float2 w) { return cmulf(a, make_float2(w.x, -w.y), 0); }
SFOC_DEV float2 cmulc(float2 a, float2 b) {  // a * conj(b), the spectrum product
    return make_float2(fmaf(a.y, b.y, a.x * b.x), fmaf(a.y, b.x, -(a.x * b.y)));
}
// a * b, every product rounded before the sum.
SFOC_DEV float2 cmulr(float2 a, float2 b) {
#pragma clang fp contract(off)
    return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
// The passes a codelet serves: forward rows and columns, inverse columns,
// inverse rows; by themselves, pass A of the rows from float16 descriptors
// and, with an 8-point codelet, pass A of the inverse columns and of the rows
// from bfloat16 descriptors.
constexpr int kFwd = 0, kInvCol = 1, kInvRow = 2, kFwdF16 = 3, kInvColA8 = 4, kFwdBf16A8 = 5;
SFOC_DEV float2 cconj(float2 a) { return make_float2(a.x, -a.y); }
// c ? a : b per component (a select of two array elements written this way
// stays in registers; as one conditional expression the compiler may turn
// it into a select of the arrays' addresses, which puts both in scratch).
SFOC_DEV float2 pick(bool c, float2 a, float2 b) { return make_float2(c ? a.x : b.x, c ? a.y : b.y); }
SFOC_DEV float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
SFOC_DEV float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
SFOC_DEV float2 cscale(float2 a, float s) { return make_float2(a.x * s, a.y * s); }
// multiply by -i (forward) or +i (inverse)
template <bool INV>
SFOC_DEV float2 mul_mi(float2 a) { return INV ? make_float2(-a.y, a.x) : make_float2(a.y, -a.x); }

// Descriptor element of type DT (0 f32, 1 bf16, 2 f16) at p[i].
template <int DT>
SFOC_DEV float ldd(const void* p, int i) {
    if constexpr (DT == 0) return ((const float*)p)[i];
    else if constexpr (DT == 1) return bf16_bits_to_f32(((const uint16_t*)p)[i]);
    else return f16_bits_to_f32(((const uint16_t*)p)[i]);
}
template <int DT>
SFOC_DEV const void* elem_ptr(const void* base, int64_t idx) {
    return (const char*)base + idx * (DT == 0 ? 4 : 2);
}

// Orders one wave's LDS reads before its following writes.  Enough where
// every location a lane writes is read only by lanes of its own wave in the
// same round (the row-pair passes: a pair's tasks are consecutive lanes);
// LDS instructions of one wave execute in order.
SFOC_DEV void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Orders the reads of a row pair's tasks before their in-place writes.  A
// pair's TPP tasks are consecutive task indices; when TPP divides the wave
// size they are lanes of one wave and wave_sync suffices, otherwise a pair
// can straddle two waves and the whole workgroup synchronises (every
// thread runs the same number of rounds, so all of them reach it).
template <int TPP>
SFOC_DEV void pair_sync() {
    if constexpr (64 % TPP == 0) wave_sync();
    else __syncthreads();
}

// ---- small DFTs in registers -------------------------------------------
// 4-point DFT of which only the first K samples are given (the others are
// zero and not read).
template <bool INV, int K = 4>
SFOC_DEV void dft4(float2& a0, float2& a1, float2& a2, float2& a3) {
    static_assert(K >= 1 && K <= 4, "at least one sample");
    if constexpr (K == 1) {
        a1 = a2 = a3 = a0;
    } else if constexpr (K == 2) {
        const float2 t0 = a0, t2 = a1, t3 = mul_mi<INV>(a1);
        a0 = cadd(t0, t2);
        a2 = csub(t0, t2);
        a1 = cadd(t0, t3);
        a3 = csub(t0, t3);
    } else {
        const float2 t0 = cadd(a0, a2), t1 = csub(a0, a2);
        const float2 t2 = K == 4 ? cadd(a1, a3) : a1, t3 = mul_mi<INV>(K == 4 ? csub(a1, a3) : a1);
        a0 = cadd(t0, t2);
        a2 = csub(t0, t2);
        a1 = cadd(t1, t3);
        a3 = csub(t1, t3);
    }
}

// x[k] <- sum_n x[n] W_8^(nk), W_8 = exp(-+2 pi i / 8); 2 x 4 split.  Only
// the samples n < NV are read, the others count as zero.  hi: the task is of
// the upper half of pass A's row pairs or columns (kFwdBf16A8, kInvColA8 only;
// the same over a wave).
template <int CTX, int NV = 8>
SFOC_DEV void dft8(float2 (&x)[8], bool hi = false) {
    static_assert(NV >= 2 && NV <= 8, "both halves have a sample");
    constexpr bool INV = CTX == kInvCol || CTX == kInvRow || CTX == kInvColA8;
    constexpr int kF[6][2] = {{2, 2}, {2, 1}, {2, 1}, {2, 2}, {1, 1}, {2, 2}};   // product forms of b1 and b3
    float2 a0 = x[0], a1 = x[2], a2 = x[4], a3 = x[6];
    float2 b0 = x[1], b1 = x[3], b2 = x[5], b3 = x[7];
    dft4<INV, (NV + 1) / 2>(a0, a1, a2, a3);
    dft4<INV, NV / 2>(b0, b1, b2, b3);
    const float h = 0.70710678118654752f;
    const float sg = INV ? 1.f : -1.f;
    const float2 w1 = make_float2(h, sg * h), w3 = make_float2(-h, sg * h);
    b2 = mul_mi<INV>(b2);
    if (CTX == kFwdBf16A8 && hi) {
        b1 = cmulr(b1, w1);
        b3 = cmulr(b3, w3);
    } else {
        b1 = CTX == kInvColA8 && hi ? cmulf(b1, w1, 2) : cmulf(b1, w1, kF[CTX][0]);
        b3 = cmulf(b3, w3, kF[CTX][1]);
    }
    x[0] = cadd(a0, b0);
    x[4] = csub(a0, b0);
    x[1] = cadd(a1, b1);
    x[5] = csub(a1, b1);
    x[2] = cadd(a2, b2);
    x[6] = csub(a2, b2);
    x[3] = cadd(a3, b3);
    x[7] = csub(a3, b3);
}

// 16-point DFT, 4 x 4 split: n = n1 + 4 n2, k = 4 k1 + k2.  Only the samples
// n < NV are read, the others count as zero.
template <int CTX, int NV = 16>
SFOC_DEV void dft16(float2 (&x)[16]) {
    static_assert(NV >= 4 && NV <= 16, "every column has a sample");
    constexpr bool INV = CTX == kInvCol || CTX == kInvRow;
    // product forms of y[n1][k2], n1, k2 = 1..3 (W_16^4 is a swap)
    constexpr int kF[4][3][3] = {{{2, 2, 2}, {2, 0, 2}, {2, 1, 1}},
                                 {{1, 2, 1}, {1, 0, 1}, {1, 1, 2}},
                                 {{0, 1, 0}, {2, 0, 1}, {0, 1, 2}},
                                 {{2, 2, 2}, {2, 0, 2}, {2, 2, 1}}};
    const float sg = INV ? 1.f : -1.f;
    const float c1 = 0.92387953251128676f, s1 = 0.38268343236508977f, h = 0.70710678118654752f;
    // twiddles W_16^e for e = 0..9
    const float2 w[10] = {make_float2(1.f, 0.f),  make_float2(c1, sg * s1), make_float2(h, sg * h),
                          make_float2(s1, sg * c1), make_float2(0.f, sg * 1.f), make_float2(-s1, sg * c1),
                          make_float2(-h, sg * h), make_float2(-c1, sg * s1), make_float2(-1.f, 0.f),
                          make_float2(-c1, -sg * s1)};
    float2 y[4][4];
    auto column = [&](auto n1c) {
        constexpr int n1 = decltype(n1c)::value, K = (NV - n1 + 3) / 4;
        float2 a0 = x[n1], a1 = x[n1 + 4], a2 = x[n1 + 8], a3 = x[n1 + 12];
        dft4<INV, K>(a0, a1, a2, a3);
        y[n1][0] = a0;
        y[n1][1] = a1;
        y[n1][2] = a2;
        y[n1][3] = a3;
    };
    column(std::integral_constant<int, 0>{});
    column(std::integral_constant<int, 1>{});
    column(std::integral_constant<int, 2>{});
    column(std::integral_constant<int, 3>{});
#pragma unroll
    for (int n1 = 1; n1 < 4; ++n1)
#pragma unroll
        for (int k2 = 1; k2 < 4; ++k2)
            y[n1][k2] = n1 * k2 == 4 ? mul_mi<INV>(y[n1][k2])
                                     : cmulf(y[n1][k2], w[n1 * k2], kF[CTX][n1 - 1][k2 - 1]);
#pragma unroll
    for (int k2 = 0; k2 < 4; ++k2) {
        float2 a0 = y[0][k2], a1 = y[1][k2], a2 = y[2][k2], a3 = y[3][k2];
        dft4<INV>(a0, a1, a2, a3);
        x[k2] = a0;
        x[4 + k2] = a1;
        x[8 + k2] = a2;
        x[12 + k2] = a3;
    }
}

// 3-point DFT: with W = exp(-+2 pi i / 3) = -1/2 -+ i sqrt(3)/2,
// X1, X2 = a0 - (a1 + a2)/2 +- i s (a1 - a2), s = -+sqrt(3)/2 (the product
// rounded first in the inverse columns, fused elsewhere).
template <int CTX>
SFOC_DEV void dft3(float2& a0, float2& a1, float2& a2) {
    const float s = (CTX != kFwd ? 1.f : -1.f) * 0.86602540378443865f;
    const float2 t1 = cadd(a1, a2), t2 = csub(a1, a2);
    const float2 m = make_float2(fmaf(-0.5f, t1.x, a0.x), fmaf(-0.5f, t1.y, a0.y));
    a0 = cadd(a0, t1);
    if constexpr (CTX == kInvCol) {
        const float2 q = make_float2(__fmul_rn(-s, t2.y), __fmul_rn(s, t2.x));   // i s t2
        a1 = make_float2(__fadd_rn(m.x, q.x), __fadd_rn(m.y, q.y));
        a2 = make_float2(__fsub_rn(m.x, q.x), __fsub_rn(m.y, q.y));
    } else {
        a1 = make_float2(fmaf(-s, t2.y, m.x), fmaf(s, t2.x, m.y));
        a2 = make_float2(fmaf(s, t2.y, m.x), fmaf(-s, t2.x, m.y));
    }
}

// 5-point DFT from the conjugate-symmetric pairs (a1, a4) and (a2, a3):
// with c_k = cos(2 pi k / 5), s_k = sin(2 pi k / 5) and sigma = -+1,
// X1,4 = a0 + c1 t1 + c2 t2 +- sigma i (s1 d1 + s2 d2),
// X2,3 = a0 + c2 t1 + c1 t2 +- sigma i (s2 d1 - s1 d2),
// t1 = a1 + a4, t2 = a2 + a3, d1 = a1 - a4, d2 = a2 - a3.
template <bool INV>
SFOC_DEV void dft5(float2 (&a)[5]) {
    const float sg = INV ? 1.f : -1.f;
    const float c1 = 0.30901699437494742f, c2 = -0.80901699437494742f;
    const float s1 = 0.95105651629515357f, s2 = 0.58778525229247313f;
    const float2 t1 = cadd(a[1], a[4]), t2 = cadd(a[2], a[3]);
    const float2 d1 = csub(a[1], a[4]), d2 = csub(a[2], a[3]);
    const float2 p1 = make_float2(fmaf(c2, t2.x, fmaf(c1, t1.x, a[0].x)), fmaf(c2, t2.y, fmaf(c1, t1.y, a[0].y)));
    const float2 p2 = make_float2(fmaf(c1, t2.x, fmaf(c2, t1.x, a[0].x)), fmaf(c1, t2.y, fmaf(c2, t1.y, a[0].y)));
    const float2 e1 = make_float2(fmaf(s2, d2.x, s1 * d1.x), fmaf(s2, d2.y, s1 * d1.y));
    const float2 e2 = make_float2(fmaf(s2, d1.x, -s1 * d2.x), fmaf(s2, d1.y, -s1 * d2.y));
    const float2 q1 = make_float2(-sg * e1.y, sg * e1.x);   // sigma i e1
    const float2 q2 = make_float2(-sg * e2.y, sg * e2.x);
    a[0] = cadd(a[0], cadd(t1, t2));
    a[1] = cadd(p1, q1);
    a[4] = csub(p1, q1);
    a[2] = cadd(p2, q2);
    a[3] = csub(p2, q2);
}

// 10-point DFT, 2 x 5: the even and odd samples each get a 5-point DFT,
// the odd ones then W_10^k, and X[k], X[k+5] = E[k] +- W_10^k O[k].
template <int CTX>
SFOC_DEV void dft10(float2 (&x)[10]) {
    constexpr bool INV = CTX != kFwd;
    constexpr int kF[2][5] = {{0, 0, 0, 3, 3}, {0, 1, 1, 1, 1}};   // product forms of o[1..4]
    const float sg = INV ? 1.f : -1.f;
    float2 e[5], o[5];
#pragma unroll
    for (int k = 0; k < 5; ++k) {
        e[k] = x[2 * k];
        o[k] = x[2 * k + 1];
    }
    dft5<INV>(e);
    dft5<INV>(o);
    // W_10^k = cos(pi k / 5) + sigma i sin(pi k / 5), k = 1..4
    const float ca = 0.80901699437494742f, sa = 0.58778525229247313f;   // 36 degrees
    const float cb = 0.30901699437494742f, sb = 0.95105651629515357f;   // 72 degrees
    o[1] = cmulf(o[1], make_float2(ca, sg * sa), kF[INV][1]);
    o[2] = cmulf(o[2], make_float2(cb, sg * sb), kF[INV][2]);
    o[3] = cmulf(o[3], make_float2(-cb, sg * sb), kF[INV][3]);
    o[4] = cmulf(o[4], make_float2(-ca, sg * sa), kF[INV][4]);
#pragma unroll
    for (int k = 0; k < 5; ++k) {
        x[k] = cadd(e[k], o[k]);
        x[k + 5] = csub(e[k], o[k]);
    }
}

// 12-point DFT, 3 x 4: n = n1 + 3 n2, k = 4 k1 + k2; 4-point DFTs over n2,
// twiddles W_12^(n1 k2), 3-point DFTs over n1.
template <int CTX>
SFOC_DEV void dft12(float2 (&x)[12]) {
    constexpr bool INV = CTX != kFwd;
    // product forms of y[n1][k2], n1 = 1, 2, k2 = 1..3
    constexpr int kF[2][2][3] = {{{2, 0, 2}, {2, 3, 2}}, {{0, 1, 2}, {0, 1, 2}}};
    const float sg = INV ? 1.f : -1.f;
    const float h = 0.86602540378443865f;   // cos 30 degrees
    float2 y[3][4];
#pragma unroll
    for (int n1 = 0; n1 < 3; ++n1) {
        float2 a0 = x[n1], a1 = x[n1 + 3], a2 = x[n1 + 6], a3 = x[n1 + 9];
        dft4<INV>(a0, a1, a2, a3);
        y[n1][0] = a0;
        y[n1][1] = a1;
        y[n1][2] = a2;
        y[n1][3] = a3;
    }
    // W_12^e, e = n1 k2 in 1..6: angles 30 e degrees
    const float2 w[7] = {make_float2(1.f, 0.f),     make_float2(h, sg * 0.5f), make_float2(0.5f, sg * h),
                         make_float2(0.f, sg * 1.f), make_float2(-0.5f, sg * h), make_float2(-h, sg * 0.5f),
                         make_float2(-1.f, 0.f)};
#pragma unroll
    for (int n1 = 1; n1 < 3; ++n1)
#pragma unroll
        for (int k2 = 1; k2 < 4; ++k2) y[n1][k2] = cmulf(y[n1][k2], w[n1 * k2], kF[INV][n1 - 1][k2 - 1]);
#pragma unroll
    for (int k2 = 0; k2 < 4; ++k2) {
        float2 a0 = y[0][k2], a1 = y[1][k2], a2 = y[2][k2];
        dft3<CTX>(a0, a1, a2);
        x[k2] = a0;
        x[4 + k2] = a1;
        x[8 + k2] = a2;
    }
}

// N-point DFT of which only the samples n < NV are read (N = 8, 16); hi as in
// dft8.
template <int N, int CTX, int NV = N>
SFOC_DEV void dftn(float2 (&x)[N], bool hi = false) {
    static_assert(NV == N || N == 8 || N == 16, "leading samples");
    if constexpr (N == 8) dft8<CTX, NV>(x, hi);
    else if constexpr (N == 10) dft10<CTX>(x);
    else if constexpr (N == 12) dft12<CTX>(x);
    else dft16<CTX, NV>(x);
}

// ---- geometry ----------------------------------------------------------
// A side L = NA * NB transform: pass A are NA-point DFTs, pass B NB-point
// ones.  NT threads per workgroup and MINB workgroups per CU (the LDS
// buffer of the larger sides leaves room for one); the kernels' launch
// bounds ask for the waves per SIMD that MINB workgroups need, which caps
// their registers accordingly.
//
// LDS layout of the transform buffer: row r starts at r * PITCH + (r / NB) *
// SKEW complex values; the pass-A output k2 of element n1 of a row pair sits
// at slot k2 * (NB + PAD) + n1 (ROT: k2 * NB + (n1 + k2) mod NB) of the pair's
// two rows.  The LDS serves 16 lanes of a 64-bit access per cycle from 32
// banks, so 16 consecutive lanes should touch 16 complex addresses that
// differ mod 16.  With PM_A / PM_B (below) the 16 lanes of the row passes
// hold two pairs (four at side 64) whose starts differ by 8 (4, 8, 12) mod
// 16; the column passes' rows n1 + NB k and the pass-B slots then fall on
// distinct residues too (side 128: 5120 LDS cycles per channel in that model,
// 9984 with pitch 68, skew 8 and consecutive pairs).
//
// What bounds the transforms: their VALU and LDS instructions, and the chain
// of stages a workgroup waits for.  Branches around single elements, address
// arithmetic per twiddle, LDS conflicts and eight barriers a channel are what
// this form takes out; measured per launch (float32 unless said): side 128,
// 400 IPs 310 -> 225 us; one IP per CU (119 IPs, float16, z = 12) 209 -> 110 us;
// side 160, 5000 IPs, bfloat16 9.98 -> 6.05 ms; side 64, 16 IPs 162 -> 118 us;
// side 192, 209 blocks 453 -> 350 us.
template <int L>
struct Fft;
template <>
struct Fft<128> {
    static constexpr int NA = 16, NB = 8, NT = 512, PITCH = 74, SKEW = 2, PAD = 1, ROT = 0, MINB = 2;
};
template <>
struct Fft<64> {
    static constexpr int NA = 8, NB = 8, NT = 128, PITCH = 38, SKEW = 4, PAD = 1, ROT = 0, MINB = 7;
};
template <>
struct Fft<160> {
    static constexpr int NA = 16, NB = 10, NT = 640, PITCH = 93, SKEW = 0, PAD = 1, ROT = 0, MINB = 1;
};
template <>
struct Fft<192> {
    static constexpr int NA = 16, NB = 12, NT = 768, PITCH = 102, SKEW = 2, PAD = 0, ROT = 1, MINB = 1;
};

template <int L>
struct MatchCfg {
    using F = Fft<L>;
    static constexpr int NA = F::NA, NB = F::NB, NT = F::NT, P = F::PITCH, SKEW = F::SKEW, MINB = F::MINB;
    static constexpr int WAVES_PER_SIMD = (MINB * NT + 255) / 256;   // 4 SIMDs of 64 lanes per CU
    static constexpr int HA = NA / 2;
    static constexpr int COLS = L / 2;                     // column transforms (DC+Nyquist packed)
    static constexpr int RB = COLS * HA / NT;              // pass-B tasks per thread
    static constexpr int BINS = 2 * NB;                    // bins per pass-B task
    static constexpr int PW = 64 / HA;                     // row pairs / columns of a wave's pass-B tasks
    // Where a wave's pairs or columns are also a whole number of pass-A
    // rounds, the wave does both passes of them and only orders its own LDS
    // accesses in between; otherwise the workgroup synchronises.
    static constexpr bool WL = PW * NB % 64 == 0;
    static constexpr int AR = WL ? PW * NB / 64 : (COLS * NB + NT - 1) / NT;   // pass-A rounds
    static_assert(L == NA * NB && NB % 2 == 0 && NA % 2 == 0, "even radices");
    static_assert(COLS * HA == NT, "one pass-B task per thread and stage");
    static_assert(2 * P >= (NA - 1) * (NB + F::PAD) + NB && 2 * P >= L,
                  "a row pair holds its pass-A outputs, or one real row of L values per row");
    static constexpr size_t buf_elems = (size_t)L * P + (size_t)(L / NB) * SKEW;   // complex
    static SFOC_DEV int row(int r) { return r * P + (r / NB) * SKEW; }
    // row n1 + NB * k with n1 < NB: its NB-row group is k
    static SFOC_DEV int rowg(int n1, int k) { return n1 * P + k * (NB * P + SKEW); }
    // Slot of element n1 of pass-A output column k2 inside a row pair.
    static SFOC_DEV int slot(int n1, int k2) {
        if constexpr (F::ROT) return k2 * NB + (n1 + k2) % NB;
        else return k2 * (NB + F::PAD) + n1;
    }
    // Pair of a wave (or, in pass A without WL, the pair itself) that holds
    // the lanes of index q: neighbouring indices take pairs whose LDS starts
    // differ by 8 mod 16 (2 PITCH = 4 mod 8: two apart; 10 mod 16: four).
    static SFOC_DEV int pm_swap(int q) { return (q & ~3) | ((q & 1) << 1) | ((q >> 1) & 1); }
    static SFOC_DEV int pm_a(int q) { return WL ? pm_swap(q) : q; }
    static SFOC_DEV int pm_b(int q) {
        if constexpr (HA == 4) return q;                              // four consecutive pairs
        else if constexpr (2 * P % 8 == 4) return pm_swap(q);
        else return (q & ~7) | ((q >> 1) & 3) | ((q & 1) << 2);
    }
    static constexpr size_t lds_bytes = sizeof(float2) * (buf_elems + L) + 1024;
};

// Bin index (within the transform) of value q of a pass-B task with j.
template <int L>
SFOC_DEV int bin_of(int j, int q) {
    using C = MatchCfg<L>;
    const int k1 = q % C::NB;
    const int kk = q < C::NB ? j : (j == 0 ? C::HA : C::NA - j);
    return C::NA * k1 + kk;
}
// Packed DC / Nyquist column (C = F_dc + i F_nyq, both Hermitian): replace
// each mirrored pair of slots (k, L-k) by (F_dc[k], F_nyq[k]).  Self-mirrored
// slots (k = 0, L/2) already hold (F_dc, F_nyq) as (re, im).
SFOC_DEV void sep_pair(float2& x, float2& y) {
    const float2 a = x, b = cconj(y);
    x = cscale(cadd(a, b), 0.5f);
    y = cscale(mul_mi<false>(csub(a, b)), 0.5f);
}
template <int NB>
SFOC_DEV void separate_packed(float2 (&u)[NB], float2 (&v)[NB], int j) {
    if (j == 0) {
#pragma unroll
        for (int k1 = 1; k1 < NB / 2; ++k1) sep_pair(u[k1], u[NB - k1]);
#pragma unroll
        for (int k1 = 0; k1 < NB / 2; ++k1) sep_pair(v[k1], v[NB - 1 - k1]);
    } else {
#pragma unroll
        for (int k1 = 0; k1 < NB; ++k1) sep_pair(u[k1], v[NB - 1 - k1]);
    }
}
// Inverse of the above on the accumulated products (Q_dc, Q_nyq) -> the
// packed spectrum P = Q_dc + i Q_nyq at both bins of each pair.
SFOC_DEV void join_pair(float2& x, float2& y) {
    const float2 q0 = x, qn = y;
    x = make_float2(q0.x - qn.y, q0.y + qn.x);
    y = make_float2(q0.x + qn.y, -q0.y + qn.x);
}
template <int NB>
SFOC_DEV void join_packed(float2 (&u)[NB], float2 (&v)[NB], int j) {
    if (j == 0) {
#pragma unroll
        for (int k1 = 1; k1 < NB / 2; ++k1) join_pair(u[k1], u[NB - k1]);
#pragma unroll
        for (int k1 = 0; k1 < NB / 2; ++k1) join_pair(v[k1], v[NB - 1 - k1]);
    } else {
#pragma unroll
        for (int k1 = 0; k1 < NB; ++k1) join_pair(u[k1], v[NB - 1 - k1]);
    }
}

// ---- row stage: real rows -> half spectra -------------------------------
// Samples n1 + NB n2, n2 < NV, of row pair p, taken as one complex row, of an
// nrows x ncols window of one descriptor plane.  Loads at 32-bit byte offsets
// from the plane (a plane holds < 2^30 elements); sample n2 lies NB * n2
// elements further on, a constant offset the load instruction encodes.  The
// window lies inside the image; a missing second row re-reads the first (then
// zeroed).  Where the samples end inside the NV blocks, columns are clamped into
// the window and the samples beyond it zeroed.
template <int L, int DT, int NV>
SFOC_DEV void load_pair(const void* __restrict__ plane, int pitch, int y0, int x0, int nrows, int ncols, int p, int n1,
                        float2 (&x)[MatchCfg<L>::NA]) {
    using C = MatchCfg<L>;
    constexpr int ES = DT == 0 ? 4 : 2;
    const bool full = ncols == NV * C::NB, odd = nrows & 1;
    const char* base = static_cast<const char*>(plane);
    const bool two = 2 * p + 1 < nrows;
    const uint32_t oa = (uint32_t)((y0 + 2 * p) * pitch + x0);
    const uint32_t ob = oa + (two ? (uint32_t)pitch : 0u);
    if (full) {
        const char* ra = base + (size_t)(oa + n1) * ES;
        const char* rb = base + (size_t)(ob + n1) * ES;
#pragma unroll
        for (int n2 = 0; n2 < NV; ++n2) x[n2] = make_float2(ldd<DT>(ra, C::NB * n2), ldd<DT>(rb, C::NB * n2));
    } else {
#pragma unroll
        for (int n2 = 0; n2 < NV; ++n2) {
            const uint32_t c = (uint32_t)min(n1 + C::NB * n2, ncols - 1);
            x[n2] = make_float2(ldd<DT>(base + (size_t)(oa + c) * ES, 0), ldd<DT>(base + (size_t)(ob + c) * ES, 0));
        }
#pragma unroll
        for (int n2 = 0; n2 < NV; ++n2)
            if (n1 + C::NB * n2 >= ncols) x[n2] = make_float2(0.f, 0.f);
    }
    if (odd) {
#pragma unroll
        for (int n2 = 0; n2 < NV; ++n2) x[n2].y = two ? x[n2].y : 0.f;
    }
}

// The sum and sum of squares of a pair's samples join s1, s2.
template <int NV, int NA>
SFOC_DEV void add_pair(const float2 (&x)[NA], double& s1, double& s2) {
    double a = 0.0, q = 0.0;
#pragma unroll
    for (int n2 = 0; n2 < NV; ++n2) {
        const double dr = x[n2].x, di = x[n2].y;
        a += dr + di;
        q += dr * dr + di * di;
    }
    s1 += a;
    s2 += q;
}

// Pass A of rows [0, nrows) x columns [0, ncols) of one descriptor plane,
// zero padded to L: of each row pair, taken as one complex row, element n1's
// samples n1 + NB n2, n2 < NV, are transformed (ncols <= NV * NB; the others
// are zero) and stored with their twiddles.  s1 / s2 (SUMS) accumulate the
// sum and sum of squares of the values.
template <int L, int DT, int NV, bool SUMS>
SFOC_DEV void row_pass_a(const void* __restrict__ plane, int pitch, int y0, int x0, int nrows, int ncols,
                         float2* buf, const float2* tw, double& s1, double& s2) {
    using C = MatchCfg<L>;
    const int tid = tid_local();
    const int npair = (nrows + 1) / 2;
    auto load = [&](int p, int n1, float2(&x)[C::NA]) {
        load_pair<L, DT, NV>(plane, pitch, y0, x0, nrows, ncols, p, n1, x);
    };
    auto finish = [&](int p, int n1, float2(&x)[C::NA]) {
        if constexpr (SUMS) add_pair<NV>(x, s1, s2);
        constexpr int CTX = DT == 2 ? kFwdF16 : DT == 1 && C::NA == 8 && !SUMS ? kFwdBf16A8 : kFwd;
        dftn<C::NA, CTX, NV>(x, tid >= C::NT / 2);
        float2* reg = buf + C::row(2 * p);
        const float2* w = tw + n1;
#pragma unroll
        for (int k2 = 0; k2 < C::NA; ++k2)
            reg[C::slot(n1, k2)] = k2 == 0 ? x[0] : cmul_row(x[k2], w[k2 * C::NB]);
    };
    if constexpr (C::WL) {   // every round's loads first
        const int wp = (tid >> 6) * C::PW, lane = tid & 63;
        float2 x[C::AR][C::NA];
#pragma unroll
        for (int rd = 0; rd < C::AR; ++rd) {
            const int q = rd * 64 + lane, p = wp + C::pm_a(q / C::NB);
            if (p < npair) load(p, q % C::NB, x[rd]);
        }
#pragma unroll
        for (int rd = 0; rd < C::AR; ++rd) {
            const int q = rd * 64 + lane, p = wp + C::pm_a(q / C::NB);
            if (p < npair) finish(p, q % C::NB, x[rd]);
        }
        wave_sync();
    } else {
#pragma unroll 1
        for (int task = tid; task < npair * C::NB; task += C::NT) {
            const int p = task / C::NB, n1 = task - p * C::NB;
            float2 x[C::NA];
            load(p, n1, x);
            finish(p, n1, x);
        }
        __syncthreads();
    }
}

// Pass B: buf row a then holds the half spectrum of row a, times two (the
// halving of the separation is left to the inverse's scale: exact, a power of
// two): bins 1..L/2 - 1, and the real DC and Nyquist bins packed in bin 0.
// A pair's pass-B tasks are lanes of one wave, so the reads of a pair are
// ordered before its in-place writes within the wave.
template <int L>
SFOC_DEV void row_pass_b(int nrows, float2* buf) {
    using C = MatchCfg<L>;
    const int tid = tid_local();
    const int j = tid % C::HA, p = (tid >> 6) * C::PW + C::pm_b((tid & 63) / C::HA);
    const bool act = p < (nrows + 1) / 2;
    const int ka = j, kb = j == 0 ? C::HA : C::NA - j;
    float2* ra = buf + C::row(2 * p);
    float2 u[C::NB], v[C::NB];
    if (act) {
#pragma unroll
        for (int n1 = 0; n1 < C::NB; ++n1) {
            u[n1] = ra[C::slot(n1, ka)];
            v[n1] = ra[C::slot(n1, kb)];
        }
        dftn<C::NB, kFwd>(u);
        dftn<C::NB, kFwd>(v);
    }
    wave_sync();
    if (act) {
        // twice the half spectra of the two real rows: 2A = X + conj X~, 2B = -i (X - conj X~)
        float2* rb = ra + C::P;
#pragma unroll
        for (int k1 = 0; k1 < C::NB / 2; ++k1) {
            const float2 za = u[k1];
            const float2 zb = cconj(pick(j == 0, u[(C::NB - k1) % C::NB], v[C::NB - 1 - k1]));
            float2 A = cadd(za, zb), B = mul_mi<false>(csub(za, zb));
            if (k1 == 0) {   // j == 0: bin 0, with the Nyquist bin
                A.y = j == 0 ? u[C::NB / 2].x + u[C::NB / 2].x : A.y;
                B.y = j == 0 ? u[C::NB / 2].y + u[C::NB / 2].y : B.y;
            }
            ra[C::NA * k1 + ka] = A;
            rb[C::NA * k1 + ka] = B;
        }
#pragma unroll
        for (int k1 = 0; k1 < C::NB / 2; ++k1) {
            const float2 za = v[k1];
            const float2 zb = cconj(pick(j == 0, v[C::NB - 1 - k1], u[C::NB - 1 - k1]));
            ra[C::NA * k1 + kb] = cadd(za, zb);
            rb[C::NA * k1 + kb] = mul_mi<false>(csub(za, zb));
        }
    }
    __syncthreads();
}

// ---- column stage: buf columns -> spectrum bins in registers --------------
// Pass A of the column transforms over columns 1..L/2-1 and the packed column
// 0 (DC + i Nyquist), in place.  Rows >= nvalid (at most NV * NB of them are
// valid) count as zero and are not used.
template <int L, bool INV, int NV>
SFOC_DEV void col_pass_a(float2* buf, const float2* tw, int nvalid) {
    using C = MatchCfg<L>;
    const int tid = tid_local();
    const bool full = nvalid == NV * C::NB;
    // task (cc, n1) reads and rewrites rows n1 + NB m of column cc only
    auto load = [&](int cc, int n1, float2(&x)[C::NA]) {
        const float2* b = buf + C::rowg(n1, 0) + cc;
#pragma unroll
        for (int n2 = 0; n2 < NV; ++n2) x[n2] = b[C::rowg(0, n2)];
        if (!full) {
#pragma unroll
            for (int n2 = 0; n2 < NV; ++n2)
                if (n1 + C::NB * n2 >= nvalid) x[n2] = make_float2(0.f, 0.f);
        }
    };
    auto finish = [&](int cc, int n1, float2(&x)[C::NA]) {
        dftn<C::NA, INV ? (C::NA == 8 ? kInvColA8 : kInvCol) : kFwd, NV>(x, tid >= C::NT / 2);
        float2* b = buf + C::rowg(n1, 0) + cc;
        const float2* tb = tw + n1;
#pragma unroll
        for (int k2 = 0; k2 < C::NA; ++k2) {
            const float2 w = tb[k2 * C::NB];
            b[C::rowg(0, k2)] = k2 == 0 ? x[0] : INV ? cmul_inv(x[k2], w) : cmul_col(x[k2], w);
        }
    };
    if constexpr (C::WL) {
        const int wc = (tid >> 6) * C::PW, lane = tid & 63;
        float2 x[C::AR][C::NA];
#pragma unroll
        for (int rd = 0; rd < C::AR; ++rd) {
            const int q = rd * 64 + lane;
            load(wc + q / C::NB, q % C::NB, x[rd]);
        }
#pragma unroll
        for (int rd = 0; rd < C::AR; ++rd) {
            const int q = rd * 64 + lane;
            finish(wc + q / C::NB, q % C::NB, x[rd]);
        }
        wave_sync();
    } else {   // consecutive lanes take consecutive columns
#pragma unroll 1
        for (int task = tid; task < C::COLS * C::NB; task += C::NT) {
            const int n1 = task / C::COLS, cc = task - n1 * C::COLS;
            float2 x[C::NA];
            load(cc, n1, x);
            finish(cc, n1, x);
        }
        __syncthreads();
    }
}

// Pass B: this thread's bins bin_of(j, q) of column cc (thread = cc * HA +
// j), values q < NB in u and q >= NB in v.
template <int L, bool INV>
SFOC_DEV void col_pass_b(const float2* buf, float2 (&u)[MatchCfg<L>::NB], float2 (&v)[MatchCfg<L>::NB]) {
    using C = MatchCfg<L>;
    const int tid = tid_local();
    const int cc = tid / C::HA, j = tid - cc * C::HA;
    const int ka = j, kb = j == 0 ? C::HA : C::NA - j;
    const float2* ba = buf + C::rowg(0, ka) + cc;
    const float2* bb = buf + C::rowg(0, kb) + cc;
#pragma unroll
    for (int n1 = 0; n1 < C::NB; ++n1) {
        u[n1] = ba[C::rowg(n1, 0)];
        v[n1] = bb[C::rowg(n1, 0)];
    }
    dftn<C::NB, INV ? kInvCol : kFwd>(u);
    dftn<C::NB, INV ? kInvCol : kFwd>(v);
}

// f(integral_constant NV) for the blocks of NB samples that a window of `side`
// rows or columns has: half, three quarters or all of the NA (HALF: half is one
// of the choices).
template <int L, bool HALF, typename F>
SFOC_DEV void by_extent(int side, F f) {
    using C = MatchCfg<L>;
    constexpr std::integral_constant<int, C::NA / 2> half{};
    constexpr std::integral_constant<int, C::NA * 3 / 4> most{};
    constexpr std::integral_constant<int, C::NA> all{};
    if (HALF && side <= half.value * C::NB) f(half);
    else if (side <= most.value * C::NB) f(most);
    else f(all);
}

// Forward 2-D transform of an nrows x ncols window of one plane into buf and
// this thread's bins (u, v).  Windows of at most half or three quarters of
// the side skip the samples that are zero by their extent.
template <int L, int DT, bool HALF, bool SUMS>
SFOC_DEV void forward_2d(const void* plane, int pitch, int y0, int x0, int nrows, int ncols, float2* buf,
                         const float2* tw, double& s1, double& s2, float2 (&u)[MatchCfg<L>::NB],
                         float2 (&v)[MatchCfg<L>::NB]) {
    using C = MatchCfg<L>;
    const int nvalid = 2 * ((nrows + 1) / 2);
    auto stages = [&](auto nv) {
        constexpr int NV = decltype(nv)::value;
        row_pass_a<L, DT, NV, SUMS>(plane, pitch, y0, x0, nrows, ncols, buf, tw, s1, s2);
    };
    auto columns = [&](auto nv) { col_pass_a<L, false, decltype(nv)::value>(buf, tw, nvalid); };
    stage_fence();
    by_extent<L, HALF>(max(nrows, ncols), stages);
    stage_fence();
    row_pass_b<L>(nrows, buf);
    stage_fence();
    by_extent<L, HALF>(max(nrows, ncols), columns);
    col_pass_b<L, false>(buf, u, v);
}

SFOC_DEV bool in_image(int64_t y, int64_t x, int h, int w, int64_t H, int64_t W) {
    return y >= 0 && x >= 0 && y + h <= H && x + w <= W;
}

// Twiddles W_L^(n1 k2), n1 < NB, k2 < NA, at tw[k2 * NB + n1] in LDS (once
// per workgroup): a thread's n1 fixes its base address and k2 an offset that
// the LDS instruction encodes.
template <int L>
SFOC_DEV void init_twiddles(float2* tw) {
    using C = MatchCfg<L>;
    for (int e = threadIdx.x; e < L; e += C::NT) {
        const int k = (e % C::NB) * (e / C::NB);
        float sn, cs;
        sincospif(-2.0f * (float)k / (float)L, &sn, &cs);
        tw[e] = make_float2(cs, sn);
    }
}

// Template sums R_T, R_TT (Eq. 12): a block reduction in float64 of every
// thread's partial sums, left in red[64] and red[65] (red holds at least 66
// doubles); returns with the workgroup synchronised.
template <int NT>
SFOC_DEV void block_sum2(double s1, double s2, double* red) {
    const int t = threadIdx.x;
    const int lane = t & 63, wv = t >> 6;
    for (int d = 32; d >= 1; d >>= 1) {
        s1 += __shfl_down(s1, d, 64);
        s2 += __shfl_down(s2, d, 64);
    }
    if (lane == 0) {
        red[2 * wv] = s1;
        red[2 * wv + 1] = s2;
    }
    __syncthreads();
    if (t == 0) {
        double a = 0.0, b = 0.0;
        for (int w = 0; w < NT / 64; ++w) {
            a += red[2 * w];
            b += red[2 * w + 1];
        }
        red[64] = a;
        red[65] = b;
    }
    __syncthreads();
}

// NCC (Eq. 9), the argmax, the parabola refinement and the CP record of one
// work item, from its correlation surface R_ST: rst_at(u, v) for offsets
// (u, v) of the block [u0, u0 + Vu) x [v0, v0 + Vv), readable by every
// thread.  RT, RTT are the template sums; red is workgroup scratch of at
// least 66 doubles.  Every thread of the workgroup calls it.
template <int NT, typename Rst>
SFOC_DEV void ncc_peak(const MatchArgs& A, int i, int slot, int u0, int v0, int Vu, int Vv, double RT, double RTT,
                       double* red, Rst rst_at) {
    const int nblk = A.nbu * A.nbv;
    const int t = threadIdx.x;
    const int m = A.m, r = A.r, M = m + 2 * r, V = 2 * r + 1;
    const int py = A.ips[2 * i], px = A.ips[2 * i + 1];
    const int pry = A.prior ? A.prior[2 * i] : 0, prx = A.prior ? A.prior[2 * i + 1] : 0;
    const int64_t sy = (int64_t)py - m / 2 - r + pry, sx = (int64_t)px - m / 2 - r + prx;
    float* nout = A.ncc ? A.ncc + (int64_t)i * V * V : (nblk > 1 ? A.surf + (int64_t)i * V * V : nullptr);
    sfoc_cp out;
    out.sen_row = py;
    out.sen_col = px;
    out.dy = out.dx = 0;
    out.sub_dy = out.sub_dx = 0.f;
    out.score = 0.f;
    out.flags = 0;
    const double mnz = (double)m * m * A.z;
    const double tau = 1e-12 * mnz;
    const double varT = RTT - RT * RT / mnz;
    // NCC (Eq. 9) with integral-image box sums (Eq. 16), float64 variance.
    // The integral images are the reference image's, or this IP's own over
    // its search window (origin (sy, sx), side M + 1).
    const int64_t IW = A.integ_win ? (int64_t)M + 1 : A.Wr + 1;
    const double* __restrict__ I1 = A.integ_win ? A.integ1 + (int64_t)i * IW * IW : A.integ1;
    const double* __restrict__ I2 = A.integ_win ? A.integ2 + (int64_t)i * IW * IW : A.integ2;
    const int64_t oy = A.integ_win ? 0 : sy, ox = A.integ_win ? 0 : sx;
    const bool flatT = !(varT > tau);
    const bool badT = !isfinite(RT) || !isfinite(RTT);
    // NCC at offset (u, v); flags: bit 0 non-flat search window, bit 1 non-finite.
    // (u, v) are offsets within this block; the surface offset is (u0 + u, v0 + v).
    auto ncc_at = [&](int u, int v, int& fl) -> float {
        const float rst = rst_at(u, v);
        const int64_t y = oy + u0 + u, x = ox + v0 + v;
        const int64_t a00 = y * IW + x, a01 = a00 + m, a10 = a00 + (int64_t)m * IW, a11 = a10 + m;
        const double RS = I1[a11] - I1[a10] - I1[a01] + I1[a00];
        const double RSS = I2[a11] - I2[a10] - I2[a01] + I2[a00];
        const double varS = RSS - RS * RS / mnz;
        float val = 0.f;
        fl = 0;
        if (!isfinite(rst) || !isfinite(RS) || !isfinite(varS)) fl |= 2;
        if (varS > tau && !flatT) {
            fl |= 1;
            const double num = (double)rst - RS * RT / mnz;
            val = (float)(num / sqrt(varS * varT));
        }
        return val;
    };
    int nonflat = 0, nonfin = 0;
    float best = -INFINITY;
    int bidx = 0x7fffffff;
    for (int e = t; e < Vu * Vv; e += NT) {
        const int u = e / Vv, v = e - u * Vv;
        int fl;
        const float val = ncc_at(u, v, fl);
        nonflat |= fl & 1;
        nonfin |= fl >> 1;
        const int eg = (u0 + u) * V + v0 + v;   // row-major index on the whole surface
        if (nout) nout[eg] = val;
        if (val > best) {   // strictly greater: the first index wins ties
            best = val;
            bidx = eg;
        }
    }
    // block reduce (max value, min index), and the flags.
    {
        const int lane = t & 63, wv = t >> 6;
        for (int d = 32; d >= 1; d >>= 1) {
            const float ob = __shfl_down(best, d, 64);
            const int oi = __shfl_down(bidx, d, 64);
            if (ob > best || (ob == best && oi < bidx)) {
                best = ob;
                bidx = oi;
            }
            nonflat |= __shfl_down(nonflat, d, 64);
            nonfin |= __shfl_down(nonfin, d, 64);
        }
        __syncthreads();
        float* rf = reinterpret_cast<float*>(red);
        int* ri = reinterpret_cast<int*>(red) + 64;
        if (lane == 0) {
            rf[wv] = best;
            ri[wv] = bidx;
            ri[16 + wv] = nonflat;
            ri[32 + wv] = nonfin;
        }
        __syncthreads();
        if (t == 0) {
            for (int w = 1; w < NT / 64; ++w) {
                if (rf[w] > rf[0] || (rf[w] == rf[0] && ri[w] < ri[0])) {
                    rf[0] = rf[w];
                    ri[0] = ri[w];
                }
                ri[16] |= ri[16 + w];
                ri[32] |= ri[32 + w];
            }
        }
        __syncthreads();
        best = rf[0];
        bidx = ri[0];
        nonflat = ri[16];
        nonfin = ri[32];
    }
    if (nblk > 1) {
        if (t == 0) {
            const int fl = (nonflat ? kBlkNonflat : 0) | (nonfin ? kBlkNonfin : 0) | (flatT ? kBlkFlatT : 0) |
                           (badT ? kBlkBadT : 0);
            A.blk[slot] = make_float4(best, __int_as_float(bidx), __int_as_float(fl), 0.f);
        }
        return;
    }
    if (t == 0) {
        if (badT || (nonfin && !flatT)) {
            out.flags = SFOC_CP_NONFINITE;
        } else if (flatT) {
            out.flags = SFOC_CP_FLAT_T;
        } else if (!nonflat || bidx >= V * V) {
            out.flags = SFOC_CP_FLAT_S;
        } else {
            const int u = bidx / V, v = bidx - u * V;
            out.dy = u - r;
            out.dx = v - r;
            out.score = best;
            if (u == 0 || v == 0 || u == V - 1 || v == V - 1) {
                out.flags = SFOC_CP_EDGE_PEAK;
            } else {
                int fl;
                const float c0 = best;
                const float cu = ncc_at(u - 1, v, fl), cd = ncc_at(u + 1, v, fl);
                const float cl = ncc_at(u, v - 1, fl), cr = ncc_at(u, v + 1, fl);
                float den = cu - 2.f * c0 + cd;
                float d = 0.f;
                if (den < 0.f) d = fminf(0.5f, fmaxf(-0.5f, (cu - cd) / (2.f * den)));
                out.sub_dy = d;
                den = cl - 2.f * c0 + cr;
                d = 0.f;
                if (den < 0.f) d = fminf(0.5f, fmaxf(-0.5f, (cl - cr) / (2.f * den)));
                out.sub_dx = d;
            }
        }
        A.cps[i] = out;
    }
}

// The spectra of channel h: the search window's (rows sy.., columns sx.., Mu x
// Mv) into xsp, then the template's into yt; the template's sums join s1, s2
// (SUMS).
// The search window comes first (only the running sum is live during its
// larger row stage), its spectrum kept in registers.
template <int L, int DT, bool SUMS>
SFOC_DEV void channel_spectra(const MatchArgs& A, int h, int64_t sy, int64_t sx, int Mu, int Mv, int64_t ty,
                              int64_t tx, const float2* tw, float2* buf, double& s1, double& s2,
                              float2 (&xsp)[MatchCfg<L>::BINS], float2 (&u)[MatchCfg<L>::NB],
                              float2 (&v)[MatchCfg<L>::NB]) {
    using C = MatchCfg<L>;
    const int64_t plane_s = A.Hs * A.Ws, plane_r = A.Hr * A.Wr;
    const int m = A.m;
    forward_2d<L, DT, false, false>(elem_ptr<DT>(A.desc_ref, h * plane_r), (int)A.Wr, (int)sy, (int)sx, Mu, Mv, buf,
                                    tw, s1, s2, u, v);
    const int tl = tid_local(), cc = tl / C::HA, j = tl - cc * C::HA;
    if (cc == 0) separate_packed<C::NB>(u, v, j);
#pragma unroll
    for (int q = 0; q < C::NB; ++q) {
        xsp[q] = u[q];
        xsp[C::NB + q] = v[q];
    }
    __syncthreads();
    forward_2d<L, DT, true, SUMS>(elem_ptr<DT>(A.desc_sen, h * plane_s), (int)A.Ws, (int)ty, (int)tx, m, m, buf, tw,
                                  s1, s2, u, v);
    if (cc == 0) separate_packed<C::NB>(u, v, j);
}

// R_ST of rows u < Vu from the summed spectrum: real rows in buf, row pair
// (u, u + 1) at C::row(u).
template <int L>
SFOC_DEV void inverse_2d(const float2 (&acc)[MatchCfg<L>::BINS], int Vu, const float2* tw, float2* buf) {
    using C = MatchCfg<L>;
    const int t = threadIdx.x;
    // inverse, columns first: spectrum bins back to LDS (natural order), then
    // column transforms k1 -> u.
    {
        const int cc = t / C::HA, j = t - cc * C::HA;
        float2 u[C::NB], v[C::NB];
#pragma unroll
        for (int q = 0; q < C::NB; ++q) {
            u[q] = acc[q];
            v[q] = acc[C::NB + q];
        }
        if (cc == 0) join_packed<C::NB>(u, v, j);
        const int kb = j == 0 ? C::HA : C::NA - j;
#pragma unroll
        for (int q = 0; q < C::NB; ++q) {
            buf[C::row(C::NA * q + j) + cc] = u[q];
            buf[C::row(C::NA * q + kb) + cc] = v[q];
        }
        __syncthreads();
        col_pass_a<L, true, C::NA>(buf, tw, L);
        col_pass_b<L, true>(buf, u, v);
        __syncthreads();
#pragma unroll
        for (int q = 0; q < C::NB; ++q) {
            const int ra = C::NA * q + j, rb = C::NA * q + kb;
            if (ra < Vu) buf[C::row(ra) + cc] = u[q];
            if (rb < Vu) buf[C::row(rb) + cc] = v[q];
        }
    }
    __syncthreads();
    // rows: pairs (u, u+1) of Hermitian half spectra -> one complex inverse;
    // real part row u, imaginary part row u+1.
    {
        const int vpair = (Vu + 1) / 2;
        // pass A of pair p, element n1: bins k = n1 + NB n2, of which those
        // above L/2 are the conjugates of L - k and bin 0 of the buffer packs
        // the real bins 0 and L/2
        auto pass_a = [&](bool act, int p, int n1) {
            float2 x[C::NA];
            float2* reg = buf + C::row(2 * p);
            if (act) {
                const float2* ra = reg;
                const float2* rb = ra + C::P;
#pragma unroll
                for (int n2 = 0; n2 < C::NA; ++n2) {
                    const int k2 = n1 + C::NB * n2;
                    int e = n2 < C::HA ? k2 : L - k2;
                    if (n2 == C::HA) e = n1 == 0 ? 0 : e;
                    float2 ha = ra[e], hb = rb[e];
                    if (n2 >= C::HA) {
                        ha = cconj(ha);
                        hb = cconj(hb);
                    }
                    if (n2 == 0) {
                        ha.y = n1 == 0 ? 0.f : ha.y;
                        hb.y = n1 == 0 ? 0.f : hb.y;
                    }
                    if (n2 == C::HA) {   // the packed bin's imaginary parts (negated above)
                        ha = n1 == 0 ? make_float2(-ha.y, 0.f) : ha;
                        hb = n1 == 0 ? make_float2(-hb.y, 0.f) : hb;
                    }
                    x[n2] = make_float2(ha.x - hb.y, ha.y + hb.x);
                }
                dftn<C::NA, kInvRow>(x);
            }
            pair_sync<C::WL ? 1 : C::NB>();   // this pair's reads before its in-place writes
            if (act) {
#pragma unroll
                for (int k2 = 0; k2 < C::NA; ++k2)
                    reg[C::slot(n1, k2)] = k2 == 0 ? x[0] : cmul_inv(x[k2], tw[k2 * C::NB + n1]);
            }
        };
        if constexpr (C::WL) {
#pragma unroll 1
            for (int rd = 0; rd < C::AR; ++rd) {
                const int q = rd * 64 + (t & 63), p = (t >> 6) * C::PW + C::pm_a(q / C::NB);
                pass_a(p < vpair, p, q % C::NB);
            }
            wave_sync();
        } else {
            const int rounds = (vpair * C::NB + C::NT - 1) / C::NT;
#pragma unroll 1
            for (int rd = 0; rd < rounds; ++rd) {
                const int task = rd * C::NT + t, p = task / C::NB;
                pass_a(p < vpair, p, task - p * C::NB);
            }
            __syncthreads();
        }
        // (the forward row passes leave twice each half spectrum)
        const float inv = 0.25f * (1.0f / ((float)L * (float)L));
        const int j = t % C::HA, p = (t >> 6) * C::PW + C::pm_b((t & 63) / C::HA);
        const int ka = j, kb = j == 0 ? C::HA : C::NA - j;
        const bool act = p < vpair;
        float2 u[C::NB], v[C::NB];
        float2* reg = buf + C::row(2 * p);
        if (act) {
#pragma unroll
            for (int n1 = 0; n1 < C::NB; ++n1) {
                u[n1] = reg[C::slot(n1, ka)];
                v[n1] = reg[C::slot(n1, kb)];
            }
            dftn<C::NB, kInvRow>(u);
            dftn<C::NB, kInvRow>(v);
        }
        wave_sync();   // this pair's reads before its in-place writes
        if (act) {
            float* rr = reinterpret_cast<float*>(reg);   // R[2p][v] at rr[v], R[2p+1][v] at rr[L + v]
#pragma unroll
            for (int k1 = 0; k1 < C::NB; ++k1) {
                const int va = C::NA * k1 + ka, vb = C::NA * k1 + kb;
                rr[va] = u[k1].x * inv;
                rr[L + va] = u[k1].y * inv;
                rr[vb] = v[k1].x * inv;
                rr[L + vb] = v[k1].y * inv;
            }
        }
        __syncthreads();
    }
}

// The record of an IP whose template or search window leaves its image.
SFOC_DEV sfoc_cp oob_record(int py, int px) {
    sfoc_cp out;
    out.sen_row = py;
    out.sen_col = px;
    out.dy = out.dx = 0;
    out.sub_dy = out.sub_dx = 0.f;
    out.score = 0.f;
    out.flags = SFOC_CP_OOB;
    return out;
}

// One work item: interest point i, offset block bq (record slot `slot`).
// With M <= L there is one block and this workgroup finishes the CP;
// otherwise each block covers offsets [u0, u0 + Vu) x [v0, v0 + Vv) with a
// search window of (m + Vu - 1) x (m + Vv - 1) <= L x L, writes its part of
// the surface and its best score, and peak_kernel combines the blocks.
// Every thread of the workgroup calls it with the same item; it returns
// with the workgroup synchronised.
template <int L, int DT, bool SPLIT = false>
SFOC_DEV void match_item(const MatchArgs& A, int i, int bq, int slot, const float2* tw, float2* buf, double* red) {
    using C = MatchCfg<L>;
    const int nblk = A.nbu * A.nbv;
    const int bu = bq / A.nbv, bv = bq - bu * A.nbv;
    const int t = threadIdx.x;
    const int m = A.m, r = A.r, M = m + 2 * r, V = 2 * r + 1;
    const int u0 = bu * A.Vb, v0 = bv * A.Vb;
    const int Vu = min(A.Vb, V - u0), Vv = min(A.Vb, V - v0);
    const int Mu = m + Vu - 1, Mv = m + Vv - 1;
    const int py = A.ips[2 * i], px = A.ips[2 * i + 1];
    const int pry = A.prior ? A.prior[2 * i] : 0, prx = A.prior ? A.prior[2 * i + 1] : 0;
    const int64_t ty = (int64_t)py - m / 2, tx = (int64_t)px - m / 2;
    const int64_t sy = ty - r + pry, sx = tx - r + prx;
    float* nout = A.ncc ? A.ncc + (int64_t)i * V * V : (nblk > 1 ? A.surf + (int64_t)i * V * V : nullptr);
    if (!in_image(ty, tx, m, m, A.Hs, A.Ws) || !in_image(sy, sx, M, M, A.Hr, A.Wr)) {
        if (t == 0) {
            if (nblk == 1) {
                A.cps[i] = oob_record(py, px);
            } else {
                A.blk[slot] = make_float4(0.f, __int_as_float(0), __int_as_float(kBlkOOB), 0.f);
            }
        }
        if (nout)
            for (int e = t; e < Vu * Vv; e += C::NT) {
                const int u = e / Vv, v = e - u * Vv;
                nout[(u0 + u) * V + v0 + v] = 0.f;
            }
        return;
    }

    float2 acc[C::BINS];   // sum over channels of F(S_h) conj(F(T_h))
#pragma unroll
    for (int q = 0; q < C::BINS; ++q) acc[q] = make_float2(0.f, 0.f);
    double s1 = 0.0, s2 = 0.0;
    float2 xsp[C::BINS];   // search-window spectrum of the current channel
    for (int h = 0; h < A.z; ++h) {
        float2 u[C::NB], v[C::NB];
        channel_spectra<L, DT, true>(A, h, sy + u0, sx + v0, Mu, Mv, ty, tx, tw, buf, s1, s2, xsp, u, v);
        const bool self = tid_local() == 0;   // cc = j = 0: slots 0 and NB/2 hold (F_dc, F_nyq) as reals
#pragma unroll
        for (int q = 0; q < C::BINS; ++q) {
            const float2 xs = xsp[q];
            const float2 yt = q < C::NB ? u[q] : v[q - C::NB];
            const float2 a = acc[q];
            acc[q] = cadd(a, cmulc(xs, yt));
            if (q == 0 || q == C::NB / 2)
                acc[q] = pick(self, make_float2(fmaf(xs.x, yt.x, a.x), fmaf(xs.y, yt.y, a.y)), acc[q]);
        }
        __syncthreads();
    }

    block_sum2<C::NT>(s1, s2, red);
    inverse_2d<L>(acc, Vu, tw, buf);

    if constexpr (SPLIT) {   // split form: R_ST and the template sums for ncc_finish_kernel
        float* __restrict__ o = A.rst + (int64_t)i * V * V;
        for (int e = t; e < Vu * Vv; e += C::NT) {
            const int u = e / Vv, v = e - u * Vv;
            const float* rr = reinterpret_cast<const float*>(buf + C::row((u >> 1) * 2));
            o[(u0 + u) * V + v0 + v] = rr[(u & 1) * L + v];
        }
        if (t == 0) {
            A.tsum[2 * i] = red[64];
            A.tsum[2 * i + 1] = red[65];
        }
    } else {
        ncc_peak<C::NT>(A, i, slot, u0, v0, Vu, Vv, red[64], red[65], red, [&](int u, int v) {
            const float* rr = reinterpret_cast<const float*>(buf + C::row((u >> 1) * 2));
            return rr[(u & 1) * L + v];
        });
    }
}

// Few interest points leave most CUs idle while a workgroup takes a point's
// channels one after the other.  Spread form: a workgroup per (point, channel)
// leaves the spectrum product, and a second launch sums the products in
// channel order, as the fused form does.  The products of the two packed self
// bins are fused into that sum, so their factors are left instead.  A further
// workgroup per point takes the template sums, as the fused form's threads do
// over all channels: both forms give the same bits.
template <int L>
struct Spread {
    using C = MatchCfg<L>;
    static constexpr size_t bins = (size_t)C::BINS * C::NT;   // complex values of a product
    // (two sums an item are more than the two a point that are used)
    static constexpr size_t item_bytes = bins * sizeof(float2) + 4 * sizeof(float2) + 2 * sizeof(double);
};

constexpr int kTemplateRegs = 64;   // registers of loads in flight
// This thread's part of the template sums over all channels, in the order of
// the row passes of match_item: steps of a channel's rounds.  Several steps' loads
// are issued first.
template <int L, int DT>
SFOC_DEV void template_sums(const MatchArgs& A, int64_t ty, int64_t tx, double& s1, double& s2) {
    using C = MatchCfg<L>;
    const int m = A.m, npair = (m + 1) / 2, steps = A.z * C::AR;
    by_extent<L, true>(m, [&](auto nv) {
        constexpr int NV = decltype(nv)::value, kU = kTemplateRegs / (2 * NV) > 1 ? kTemplateRegs / (2 * NV) : 1;
        auto pair = [&](int e, int& n1) {   // the row pair and element of a step, as in row_pass_a
            const int tid = tid_local(), rd = e % C::AR, q = C::WL ? rd * 64 + (tid & 63) : rd * C::NT + tid;
            n1 = q % C::NB;
            return C::WL ? (tid >> 6) * C::PW + C::pm_a(q / C::NB) : q / C::NB;
        };
#pragma unroll 1
        for (int e0 = 0; e0 < steps; e0 += kU) {
            float2 x[kU][C::NA];
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const int e = min(e0 + u, steps - 1);
                int n1;
                const int p = pair(e, n1);
                if (p < npair)
                    load_pair<L, DT, NV>(elem_ptr<DT>(A.desc_sen, e / C::AR * (A.Hs * A.Ws)), (int)A.Ws, (int)ty,
                                         (int)tx, m, m, p, n1, x[u]);
            }
            stage_fence();
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                int n1;
                if (e0 + u < steps && pair(e0 + u, n1) < npair) add_pair<NV>(x[u], s1, s2);
            }
        }
    });
}

template <int L, int DT>
__global__ __launch_bounds__(MatchCfg<L>::NT, MatchCfg<L>::WAVES_PER_SIMD) void match_spectra_kernel(const MatchArgs A) {
    using C = MatchCfg<L>;
    extern __shared__ float4 lds_raw[];
    float2* tw = reinterpret_cast<float2*>(lds_raw);
    float2* buf = tw + L;
    double* red = reinterpret_cast<double*>(buf + C::buf_elems);
    // the template sums' workgroups come first; of the others each XCD takes a
    // contiguous run of points (see match_kernel)
    const int items = A.n * A.z, q8 = items / 8 * 8, id = (int)blockIdx.x - A.n;
    const bool sums = id < 0;
    const int k = sums ? -1 : id < q8 ? (id % 8) * (q8 / 8) + id / 8 : id;
    const int i = sums ? (int)blockIdx.x : k / A.z, h = k - i * A.z;
    const int m = A.m, r = A.r, M = m + 2 * r, t = threadIdx.x;
    const int64_t ty = (int64_t)A.ips[2 * i] - m / 2, tx = (int64_t)A.ips[2 * i + 1] - m / 2;
    const int64_t sy = ty - r + (A.prior ? A.prior[2 * i] : 0), sx = tx - r + (A.prior ? A.prior[2 * i + 1] : 0);
    if (!in_image(ty, tx, m, m, A.Hs, A.Ws) || !in_image(sy, sx, M, M, A.Hr, A.Wr)) return;
    double s1 = 0.0, s2 = 0.0;
    if (sums) {
        template_sums<L, DT>(A, ty, tx, s1, s2);
        block_sum2<C::NT>(s1, s2, red);
        if (t < 2) A.spec_sum[2 * i + t] = red[64 + t];
        return;
    }
    init_twiddles<L>(tw);
    __syncthreads();
    float2 xsp[C::BINS], u[C::NB], v[C::NB];
    channel_spectra<L, DT, false>(A, h, sy, sx, M, M, ty, tx, tw, buf, s1, s2, xsp, u, v);
    float2* __restrict__ o = A.spec + (size_t)k * Spread<L>::bins + t;
    float2* __restrict__ f = A.spec_self + (size_t)k * 4;
#pragma unroll
    for (int q = 0; q < C::BINS; ++q) {
        const float2 yt = q < C::NB ? u[q] : v[q - C::NB];
        o[q * C::NT] = cmulc(xsp[q], yt);
        if ((q == 0 || q == C::NB / 2) && t == 0) {
            f[q ? 2 : 0] = xsp[q];
            f[q ? 3 : 1] = yt;
        }
    }
}

// The second launch: a workgroup per point, for its latency: registers for up to
// four channels' loads in flight rather than for several workgroups a CU.  Above
// side 64 it comes after the integral images and takes the NCC and the peak too
// (119 points, side 128: 161 -> 156 us a call; 64 points, side 160: 231 -> 214);
// at side 64 its 128 threads would be slower at it than ncc_finish_kernel's 256
// (16 points: 80 us a call with that, 89 without), so there it leaves R_ST.
template <int L>
constexpr bool spread_peak() { return L > 64; }
template <int L>
__global__ __launch_bounds__(MatchCfg<L>::NT, (MatchCfg<L>::NT + 255) / 256) void match_combine_kernel(const MatchArgs A) {
    using C = MatchCfg<L>;
    extern __shared__ float4 lds_raw[];
    float2* tw = reinterpret_cast<float2*>(lds_raw);
    float2* buf = tw + L;
    double* red = reinterpret_cast<double*>(buf + C::buf_elems);
    const int i = (int)blockIdx.x, m = A.m, r = A.r, M = m + 2 * r, V = 2 * r + 1, t = threadIdx.x;
    const int py = A.ips[2 * i], px = A.ips[2 * i + 1];
    const int64_t ty = (int64_t)py - m / 2, tx = (int64_t)px - m / 2;
    const int64_t sy = ty - r + (A.prior ? A.prior[2 * i] : 0), sx = tx - r + (A.prior ? A.prior[2 * i + 1] : 0);
    if (!in_image(ty, tx, m, m, A.Hs, A.Ws) || !in_image(sy, sx, M, M, A.Hr, A.Wr)) {
        if (t == 0) A.cps[i] = oob_record(py, px);
        if (A.ncc)
            for (int e = t; e < V * V; e += C::NT) A.ncc[(int64_t)i * V * V + e] = 0.f;
        return;
    }
    init_twiddles<L>(tw);
    float2 acc[C::BINS];
#pragma unroll
    for (int q = 0; q < C::BINS; ++q) acc[q] = make_float2(0.f, 0.f);
    const float2* __restrict__ o = A.spec + (size_t)i * A.z * Spread<L>::bins + t;
    const float2* __restrict__ f = A.spec_self + (size_t)i * A.z * 4;
    constexpr int kU = L <= 64 ? 4 : L <= 128 ? 3 : 2;
    for (int h0 = 0; h0 < A.z; h0 += kU) {
        float2 p[kU][C::BINS], fs[kU][4];
#pragma unroll
        for (int k = 0; k < kU; ++k) {
            const int h = min(h0 + k, A.z - 1);
#pragma unroll
            for (int q = 0; q < C::BINS; ++q) p[k][q] = o[h * Spread<L>::bins + q * C::NT];
#pragma unroll
            for (int q = 0; q < 4; ++q) fs[k][q] = f[4 * h + q];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < kU; ++k) {
            if (h0 + k >= A.z) break;
#pragma unroll
            for (int q = 0; q < C::BINS; ++q) {
                const float2 a = acc[q];
                acc[q] = cadd(a, p[k][q]);
                if (q == 0 || q == C::NB / 2) {
                    const float2 xs = fs[k][q ? 2 : 0], yt = fs[k][q ? 3 : 1];
                    acc[q] = pick(t == 0, make_float2(fmaf(xs.x, yt.x, a.x), fmaf(xs.y, yt.y, a.y)), acc[q]);
                }
            }
        }
    }
    if (t < 2) {
        const double s = A.spec_sum[2 * i + t];
        if constexpr (spread_peak<L>()) red[64 + t] = s;
        else A.tsum[2 * i + t] = s;
    }
    __syncthreads();
    inverse_2d<L>(acc, V, tw, buf);
    auto rst_at = [&](int u, int v) {
        const float* rr = reinterpret_cast<const float*>(buf + C::row((u >> 1) * 2));
        return rr[(u & 1) * L + v];
    };
    if constexpr (spread_peak<L>()) {
        ncc_peak<C::NT>(A, i, i, 0, 0, V, V, red[64], red[65], red, rst_at);
    } else {
        float* __restrict__ R = A.rst + (int64_t)i * V * V;
        for (int e = t; e < V * V; e += C::NT) R[e] = rst_at(e / V, e % V);
    }
}

// Split form, second launch: one workgroup per IP assembles the NCC surface
// (Eq. 9 with the box sums of Eq. 16) from the R_ST and template sums the
// transforms left, and takes its peak, as the fused form does.  IPs whose
// template or search window leaves its image got their record from the
// transforms' launch.
constexpr int kFinishNT = 256;
__global__ __launch_bounds__(kFinishNT) void ncc_finish_kernel(const MatchArgs A) {
    __shared__ double red[66];
    const int i = (int)blockIdx.x;
    const int m = A.m, r = A.r, M = m + 2 * r, V = 2 * r + 1;
    const int py = A.ips[2 * i], px = A.ips[2 * i + 1];
    const int pry = A.prior ? A.prior[2 * i] : 0, prx = A.prior ? A.prior[2 * i + 1] : 0;
    const int64_t ty = (int64_t)py - m / 2, tx = (int64_t)px - m / 2;
    const int64_t sy = ty - r + pry, sx = tx - r + prx;
    if (!in_image(ty, tx, m, m, A.Hs, A.Ws) || !in_image(sy, sx, M, M, A.Hr, A.Wr)) return;
    const float* __restrict__ R = A.rst + (int64_t)i * V * V;
    ncc_peak<kFinishNT>(A, i, i, 0, 0, V, V, A.tsum[2 * i], A.tsum[2 * i + 1], red,
                        [&](int u, int v) { return R[u * V + v]; });
}

template <int L, int DT, bool BATCH, bool SPLIT = false>
__global__ __launch_bounds__(MatchCfg<L>::NT, MatchCfg<L>::WAVES_PER_SIMD) void match_kernel(const MatchArgs single,
                                                                   const MatchArgs* __restrict__ pairs,
                                                                   const int4* __restrict__ items) {
    using C = MatchCfg<L>;
    extern __shared__ float4 lds_raw[];
    float2* tw = reinterpret_cast<float2*>(lds_raw);
    float2* buf = tw + L;
    double* red = reinterpret_cast<double*>(buf + C::buf_elems);   // 1 KB scratch
    // One pair per launch (blockIdx.x -> IP, block), or (BATCH) a table of
    // (pair, IP, block) items over several pairs.
    init_twiddles<L>(tw);
    __syncthreads();
    if (BATCH) {
        const int4 it = items[blockIdx.x];
        const MatchArgs A = load_table(pairs, it.x);
        match_item<L, DT>(A, it.y, it.z, it.y * A.nbu * A.nbv + it.z, tw, buf, red);
    } else {
        // Workgroups are dealt to the eight XCDs in turn; renumbered so that
        // each XCD takes a contiguous run of IPs, whose overlapping search
        // windows then meet in one L2.
        const int n = (int)gridDim.x, q8 = n / 8 * 8, id = (int)blockIdx.x;
        const int k = id < q8 ? (id % 8) * (q8 / 8) + id / 8 : id;
        const int nblk = single.nbu * single.nbv;
        const int i = k / nblk;
        match_item<L, DT, SPLIT>(single, i, k - i * nblk, k, tw, buf, red);
    }
}

// Persistent form for batched plans: a grid of about two workgroups per CU
// takes items in order from a counter (zeroed before the launch) until the
// table is exhausted; every workgroup then exits.
template <int L, int DT>
__global__ __launch_bounds__(MatchCfg<L>::NT, MatchCfg<L>::WAVES_PER_SIMD) void match_persistent_kernel(const MatchArgs* __restrict__ pairs,
                                                                              const int4* __restrict__ items,
                                                                              int nitems, int* __restrict__ counter) {
    using C = MatchCfg<L>;
    extern __shared__ float4 lds_raw[];
    float2* tw = reinterpret_cast<float2*>(lds_raw);
    float2* buf = tw + L;
    double* red = reinterpret_cast<double*>(buf + C::buf_elems);
    __shared__ int next;
    init_twiddles<L>(tw);
    for (;;) {
        if (threadIdx.x == 0) next = atomicAdd(counter, 1);
        __syncthreads();
        const int k = next;
        __syncthreads();   // every thread has read `next` before it is replaced
        if (k >= nitems) break;
        const int4 it = items[k];
        const MatchArgs A = load_table(pairs, it.x);
        match_item<L, DT>(A, it.y, it.z, it.y * A.nbu * A.nbv + it.z, tw, buf, red);
        __syncthreads();
    }
}

__global__ void zero_counter_kernel(int* counter) { *counter = 0; }

// ---- direct correlation on the matrix cores -----------------------------
// R_ST(u, v) = sum_h sum_i sum_k S_h(i + u, k) T_h(i, k - v): Eq. 10 summed in
// space, with T_h(i, j) = 0 outside 0 <= j < m, for 16-bit descriptors and at
// most 32 offsets per axis.  For each channel h and template row i this is
// the product of the 32 window rows i .. i + 31 (32 x K; K = 16 ceil(M / 16)
// columns, zero beyond M) with the banded Toeplitz matrix of template row i
// (K x 32, B[k][v] = T_h(i, k - v)): K / 16 MFMAs of 32 x 32 x 16 with
// float32 accumulation.  The stored 16-bit values are exact operands; only
// the order of the float32 sums differs from the FFT path.
//
// MFMA 32 x 32 x 16 operands (lane l, c = 0..7): A[l % 32][8 (l / 32) + c],
// B[8 (l / 32) + c][l % 32]; result register q of lane l holds
// D[8 (q / 4) + 4 (l / 32) + q % 4][l % 32].
//
// LDS per channel: the window (m + 31 rows, pitch PW; rows and columns from
// M on stay zero), then two copies of the zero-padded template rows, with
// Tz(q) = T_h(i, q - 32): E[q] = Tz(q), O[q] = Tz(q + 1).  Lane (v, g) of
// chunk kb needs Tz(16 kb + 8 g - v + 32 + c), c = 0..7; it reads E when v is
// even and O one element earlier when v is odd, so that every read starts on
// a 4-byte boundary.  Wave w takes the template rows i = w (mod 4); the four
// partial surfaces are summed in wave order.
constexpr int kDirNT = 256;
constexpr int kDirMaxKB = (kDirectMaxM + kDirectMaxV - 1 + 15) / 16;   // chunks of the widest window (94): 6

// Chunks of a window of M = m + 2r columns; a launch runs a fixed chunk
// count NKB >= that of each of its IPs (further chunks multiply zeros).
inline SFOC_HOST_DEVICE int dir_nkb(int m, int r) { return (m + 2 * r + 15) / 16; }
struct DirGeom {
    int PW;      // window row pitch (elements): 16 NKB + 8
    int WR;      // window rows staged: m + 31
    int PT;      // template row pitch (elements): 16 NKB + 40
    int OE;      // offset of the O copy from E (elements): m PT, padded to 17 dwords mod 32
    int bytes;   // dynamic LDS: the operands, or the four 32 x 32 float partial surfaces
};
// A B-operand read by lanes v = 0..31 of one half-wave touches the E dwords
// d + 1 .. d + 16 (even v) and the O dwords d .. d + 15 (odd v), d = 8 kb +
// 4 g plus the row's offset, and one dword later for the second dword read.
// With O 17 dwords (mod 32) after E the two sets fall on disjoint banks of
// the 32-bank LDS.
inline SFOC_HOST_DEVICE DirGeom dir_geom(int m, int nkb) {
    DirGeom g;
    g.PW = 16 * nkb + 8;
    g.WR = m + 31;
    g.PT = 16 * nkb + 40;
    g.OE = m * g.PT + 2 * ((17 - (m * g.PT / 2) % 32 + 32) % 32);
    const int b = 2 * (g.WR * g.PW + g.OE + m * g.PT);
    g.bytes = b > 4 * 1024 * 4 ? b : 4 * 1024 * 4;
    return g;
}

typedef __bf16 dir_bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 dir_f16x8 __attribute__((ext_vector_type(8)));
typedef float dir_f32x16 __attribute__((ext_vector_type(16)));

template <int DT>
SFOC_DEV dir_f32x16 dir_mfma(uint4 a, uint4 b, dir_f32x16 c) {
    if constexpr (DT == 1)
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(dir_bf16x8, a),
                                                       __builtin_bit_cast(dir_bf16x8, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(dir_f16x8, a),
                                                      __builtin_bit_cast(dir_f16x8, b), c, 0, 0, 0);
}

// One interest point of the direct form (A.nbu = A.nbv = 1, V <= 32, m <= 64,
// dir_nkb(m, r) <= NKB).
template <int DT, int NKB>
SFOC_DEV void direct_item(const MatchArgs& A, int i, char* lds, double* red) {
    const int t = threadIdx.x, lane = t & 63, w = t >> 6, ul = lane & 31, gl = lane >> 5;
    const int m = A.m, r = A.r, M = m + 2 * r, V = 2 * r + 1;
    const DirGeom g = dir_geom(m, NKB);
    const int py = A.ips[2 * i], px = A.ips[2 * i + 1];
    const int pry = A.prior ? A.prior[2 * i] : 0, prx = A.prior ? A.prior[2 * i + 1] : 0;
    const int64_t ty = (int64_t)py - m / 2, tx = (int64_t)px - m / 2;
    const int64_t sy = ty - r + pry, sx = tx - r + prx;
    if (!in_image(ty, tx, m, m, A.Hs, A.Ws) || !in_image(sy, sx, M, M, A.Hr, A.Wr)) {
        if (t == 0) {
            sfoc_cp out;
            out.sen_row = py;
            out.sen_col = px;
            out.dy = out.dx = 0;
            out.sub_dy = out.sub_dx = 0.f;
            out.score = 0.f;
            out.flags = SFOC_CP_OOB;
            A.cps[i] = out;
        }
        if (A.ncc)
            for (int e = t; e < V * V; e += kDirNT) A.ncc[(int64_t)i * V * V + e] = 0.f;
        return;
    }
    uint16_t* Wl = reinterpret_cast<uint16_t*>(lds);
    uint16_t* E = Wl + g.WR * g.PW;
    uint16_t* O = E + g.OE;
    {   // the zero bands of both operands stay zero for every channel
        uint32_t* zp = reinterpret_cast<uint32_t*>(lds);
        const int nz = (g.WR * g.PW + g.OE + m * g.PT) / 2;
        for (int e = t; e < nz; e += kDirNT) zp[e] = 0u;
    }
    __syncthreads();
    dir_f32x16 acc0 = {}, acc1 = {};   // even and odd chunks: two independent chains
    double s1 = 0.0, s2 = 0.0;
    const int64_t plane_s = A.Hs * A.Ws, plane_r = A.Hr * A.Wr;
    const uint16_t* refp = static_cast<const uint16_t*>(A.desc_ref) + sy * A.Wr + sx;
    const uint16_t* senp = static_cast<const uint16_t*>(A.desc_sen) + ty * A.Ws + tx;
    // A channel's operands go global -> registers -> LDS.  Wave w takes the
    // rows w, w + 4, ... (at most KR window and KT template rows: M <= 16 NKB,
    // m <= min(64, 16 NKB)); a lane the columns lane and, when the window is
    // wider than 64, lane + 64.  Rows and columns are clamped into the window,
    // so that every load is in bounds and unconditional; only the stores are
    // masked.  Up to NKB = 4 the next channel's loads are issued before this
    // channel's MFMAs and land while they run; wider windows (more registers
    // per lane) load each channel in one batch before its MFMAs.
    constexpr int KR = 4 * NKB, KC = 16 * NKB > 64 ? 2 : 1, KT = 4 * NKB < 16 ? 4 * NKB : 16;
    constexpr bool kPrefetch = NKB <= 4;
    uint16_t wv[KC][KR], tv[KT];
    auto load = [&](int h) {
        // (a laundered thread index: the address arithmetic is redone per
        // channel rather than hoisted out of the loop and kept live)
        const int tl = tid_local(), ln = tl & 63, wl = __builtin_amdgcn_readfirstlane(tl >> 6);
        const uint16_t* rp = refp + h * plane_r + (int64_t)wl * A.Wr;   // wave-uniform bases
        const int wt = min(wl, m - 1);   // (m = 3: the fourth wave has no template row of its own)
        const uint16_t* sp = senp + h * plane_s + (int64_t)wt * A.Ws;
#pragma unroll
        for (int c = 0; c < KC; ++c) {
            const uint32_t x = (uint32_t)min(ln + 64 * c, M - 1);
#pragma unroll
            for (int j = 0; j < KR; ++j)
                wv[c][j] = rp[(uint32_t)(min(wl + 4 * j, M - 1) - wl) * (uint32_t)A.Wr + x];
        }
        const uint32_t xt = (uint32_t)min(ln, m - 1);
#pragma unroll
        for (int j = 0; j < KT; ++j) tv[j] = sp[(uint32_t)(min(wl + 4 * j, m - 1) - wt) * (uint32_t)A.Ws + xt];
    };
    auto store = [&]() {
        const int tl = tid_local(), ln = tl & 63, wl = __builtin_amdgcn_readfirstlane(tl >> 6);
        uint16_t* wrow = Wl + wl * g.PW + ln;
#pragma unroll
        for (int c = 0; c < KC; ++c)
#pragma unroll
            for (int j = 0; j < KR; ++j)
                if (wl + 4 * j < M && ln + 64 * c < M) wrow[4 * j * g.PW + 64 * c] = wv[c][j];
        uint16_t* erow = E + wl * g.PT + 32 + ln;
#pragma unroll
        for (int j = 0; j < KT; ++j)
            if (wl + 4 * j < m && ln < m) {
                erow[4 * j * g.PT] = tv[j];
                erow[4 * j * g.PT + g.OE - 1] = tv[j];   // O[y][31 + x]
                const double f = (double)(DT == 1 ? bf16_bits_to_f32(tv[j]) : f16_bits_to_f32(tv[j]));
                s1 += f;
                s2 += f * f;
            }
    };
    // per template row: every chunk's operands read first, then the MFMAs
    auto compute = [&]() {
        const int tl = tid_local(), ln = tl & 63, wl = __builtin_amdgcn_readfirstlane(tl >> 6), u = ln & 31,
                  gq = ln >> 5;
        for (int ii = wl; ii < m; ii += 4) {
            const uint16_t* arow = Wl + (ii + u) * g.PW + 8 * gq;
            const uint16_t* brow = ((u & 1) ? O : E) + ii * g.PT + 8 * gq + 32 - u - (u & 1);
            uint4 a[NKB], b[NKB];
#pragma unroll
            for (int kb = 0; kb < NKB; ++kb) {
                a[kb] = *reinterpret_cast<const uint4*>(arow + 16 * kb);
                const uint32_t* bp = reinterpret_cast<const uint32_t*>(brow + 16 * kb);
                b[kb] = make_uint4(bp[0], bp[1], bp[2], bp[3]);
            }
#pragma unroll
            for (int kb = 0; kb < NKB; ++kb) {
                if (kb & 1)
                    acc1 = dir_mfma<DT>(a[kb], b[kb], acc1);
                else
                    acc0 = dir_mfma<DT>(a[kb], b[kb], acc0);
            }
        }
    };
    if constexpr (kPrefetch) {
        load(0);
        for (int h = 0; h < A.z; ++h) {
            store();
            __syncthreads();
            if (h + 1 < A.z) load(h + 1);
            compute();
            __syncthreads();
        }
    } else {
        for (int h = 0; h < A.z; ++h) {
            load(h);
            store();
            __syncthreads();
            compute();
            __syncthreads();
        }
    }
    float* P = reinterpret_cast<float*>(lds);   // wave w's partial surface at P + 1024 w
#pragma unroll
    for (int q = 0; q < 16; ++q) P[1024 * w + (8 * (q >> 2) + 4 * gl + (q & 3)) * 32 + ul] = acc0[q] + acc1[q];
    __syncthreads();
    for (int e = t; e < V * V; e += kDirNT) {
        const int u = e / V, o = u * 32 + (e - u * V);
        P[o] = ((P[o] + P[1024 + o]) + P[2048 + o]) + P[3072 + o];
    }
    block_sum2<kDirNT>(s1, s2, red);
    ncc_peak<kDirNT>(A, i, i, 0, 0, V, V, red[64], red[65], red, [&](int u, int v) { return P[u * 32 + v]; });
}

// One pair (blockIdx.x -> IP, dealt to the XCDs in contiguous runs), or
// (BATCH) a table of (pair, IP) items.
template <int DT, int NKB, bool BATCH>
__global__ __launch_bounds__(kDirNT, 4) void match_direct_kernel(const MatchArgs single,
                                                               const MatchArgs* __restrict__ pairs,
                                                               const int4* __restrict__ items) {
    extern __shared__ float4 lds_raw[];
    __shared__ double red[66];
    char* lds = reinterpret_cast<char*>(lds_raw);
    if (BATCH) {
        const int4 it = items[blockIdx.x];
        const MatchArgs A = load_table(pairs, it.x);
        direct_item<DT, NKB>(A, it.y, lds, red);
    } else {
        const int n = (int)gridDim.x, q8 = n / 8 * 8, id = (int)blockIdx.x;
        direct_item<DT, NKB>(single, id < q8 ? (id % 8) * (q8 / 8) + id / 8 : id, lds, red);
    }
}

// ---- combining offset blocks --------------------------------------------
// One thread per interest point: the best score over its blocks (ties: the
// smallest row-major surface index), the flags, and the parabola from the
// surface the blocks wrote.  Same decisions as the single-block path.
template <bool BATCH>
__global__ __launch_bounds__(256) void peak_kernel(const MatchArgs single, const MatchArgs* __restrict__ pairs,
                                                   const int4* __restrict__ items) {
    const MatchArgs A = BATCH ? load_table(pairs, items[blockIdx.x].x) : single;
    const int i = (BATCH ? items[blockIdx.x].y : (int)(blockIdx.x * blockDim.x)) + (int)threadIdx.x;
    if (i >= A.n) return;
    const int nblk = A.nbu * A.nbv;
    const int r = A.r, V = 2 * r + 1;
    sfoc_cp out;
    out.sen_row = A.ips[2 * i];
    out.sen_col = A.ips[2 * i + 1];
    out.dy = out.dx = 0;
    out.sub_dy = out.sub_dx = 0.f;
    out.score = 0.f;
    out.flags = 0;
    float best = -INFINITY;
    int bidx = 0x7fffffff, fl = 0;
    for (int b = 0; b < nblk; ++b) {
        const float4 q = A.blk[(int64_t)i * nblk + b];
        const int qi = __float_as_int(q.y);
        fl |= __float_as_int(q.z);
        if (q.x > best || (q.x == best && qi < bidx)) {
            best = q.x;
            bidx = qi;
        }
    }
    const float* surf = (A.ncc ? A.ncc : A.surf) + (int64_t)i * V * V;
    if (fl & kBlkOOB) {
        out.flags = SFOC_CP_OOB;
    } else if ((fl & kBlkBadT) || ((fl & kBlkNonfin) && !(fl & kBlkFlatT))) {
        out.flags = SFOC_CP_NONFINITE;
    } else if (fl & kBlkFlatT) {
        out.flags = SFOC_CP_FLAT_T;
    } else if (!(fl & kBlkNonflat) || bidx >= V * V) {
        out.flags = SFOC_CP_FLAT_S;
    } else {
        const int u = bidx / V, v = bidx - u * V;
        out.dy = u - r;
        out.dx = v - r;
        out.score = best;
        if (u == 0 || v == 0 || u == V - 1 || v == V - 1) {
            out.flags = SFOC_CP_EDGE_PEAK;
        } else {
            const float c0 = best;
            const float cu = surf[bidx - V], cd = surf[bidx + V], cl = surf[bidx - 1], cr = surf[bidx + 1];
            float den = cu - 2.f * c0 + cd;
            float d = 0.f;
            if (den < 0.f) d = fminf(0.5f, fmaxf(-0.5f, (cu - cd) / (2.f * den)));
            out.sub_dy = d;
            den = cl - 2.f * c0 + cr;
            d = 0.f;
            if (den < 0.f) d = fminf(0.5f, fmaxf(-0.5f, (cl - cr) / (2.f * den)));
            out.sub_dx = d;
        }
    }
    A.cps[i] = out;
}

// ---- consistency: median displacement, 1.5 px (Section 4.1) ------------
// One workgroup; exact k-th smallest by 8-bit radix selection on
// order-preserving keys, so any n works without a sort buffer.
constexpr int kConsNT = 256;
constexpr uint32_t kBad = SFOC_CP_OOB | SFOC_CP_FLAT_T | SFOC_CP_FLAT_S | SFOC_CP_EDGE_PEAK | SFOC_CP_NONFINITE;

SFOC_DEV uint32_t fkey(float f) {
    const uint32_t u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
SFOC_DEV float fkey_inv(uint32_t k) {
    return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}
SFOC_DEV float cp_disp(const sfoc_cp& c, const int32_t* prior, int i, int axis) {
    const int pr = prior ? prior[2 * i + axis] : 0;
    return axis == 0 ? (float)(pr + c.dy) + c.sub_dy : (float)(pr + c.dx) + c.sub_dx;
}

// Keys of the eligible CPs' displacements are cached in LDS up to this many
// CPs (both axes); larger pairs read them from the records on every pass.
constexpr int kConsCache = 6144;

// The k-th smallest (0-based) key among the eligible CPs for four (axis,
// rank) targets at once: four 8-bit radix passes, each building the four
// targets' histograms in one sweep over the keys; wave q then scans
// histogram q (four bins per lane) for the bin holding its rank.
static_assert(kConsNT == 256, "one scanning wave per target");
SFOC_DEV void select_kth4(const sfoc_cp* cps, const int32_t* prior, int n, const int (&axis)[4], int (&k)[4],
                          const uint32_t* const (&cache)[2], int ncache, uint32_t (*hist)[256], uint32_t* sel,
                          uint32_t (&prefix)[4]) {
    uint32_t mask = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) prefix[q] = 0;
    for (int shift = 24; shift >= 0; shift -= 8) {
        for (int b = threadIdx.x; b < 4 * 256; b += kConsNT) hist[b >> 8][b & 255] = 0;
        __syncthreads();
        const int cnt = cache[0] ? ncache : n;
        for (int i = threadIdx.x; i < cnt; i += kConsNT) {
            uint32_t key[2];
            if (cache[0]) {
                key[0] = cache[0][i];
                key[1] = cache[1][i];
            } else {
                const sfoc_cp c = cps[i];
                if (c.flags & kBad) continue;
                key[0] = fkey(cp_disp(c, prior, i, 0));
                key[1] = fkey(cp_disp(c, prior, i, 1));
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t kq = key[axis[q]];
                if ((kq & mask) == prefix[q]) atomicAdd(&hist[q][(kq >> shift) & 255u], 1u);
            }
        }
        __syncthreads();
        {
            const int q = threadIdx.x >> 6, lane = threadIdx.x & 63;
            const uint32_t* h = hist[q];
            const uint32_t h0 = h[4 * lane], h1 = h[4 * lane + 1], h2 = h[4 * lane + 2], h3 = h[4 * lane + 3];
            const uint32_t own = h0 + h1 + h2 + h3;
            uint32_t incl = own;   // inclusive prefix over lanes
            for (int d = 1; d < 64; d <<= 1) {
                const uint32_t u = __shfl_up(incl, d, 64);
                if (lane >= d) incl += u;
            }
            const uint32_t before = incl - own;   // keys in bins below this lane's four
            uint32_t kq = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (j == q) kq = (uint32_t)k[j];
            if (before <= kq && kq < incl) {   // exactly one lane per target
                uint32_t cum = before;
                int b = 4 * lane;
                const uint32_t hs[4] = {h0, h1, h2, h3};
                for (int j = 0; j < 4; ++j, ++b) {
                    if (cum + hs[j] > kq) break;
                    cum += hs[j];
                }
                sel[2 * q] = (uint32_t)b;
                sel[2 * q + 1] = cum;
            }
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            prefix[q] |= sel[2 * q] << shift;
            k[q] -= (int)sel[2 * q + 1];
        }
        mask |= 255u << shift;
        __syncthreads();
    }
}

__global__ __launch_bounds__(kConsNT) void consistency_kernel(sfoc_cp* cps, const int32_t* prior, int n,
                                                              const MatchArgs* __restrict__ pairs) {
    if (pairs) {   // one workgroup per pair of a batched plan
        const MatchArgs P = load_table(pairs, (int)blockIdx.x);
        cps = P.cps;
        prior = P.prior;
        n = P.n;
    }
    __shared__ uint32_t hist[4][256];
    __shared__ uint32_t sel[8];
    __shared__ int cnt;
    __shared__ uint32_t keys[2][kConsCache];
    if (threadIdx.x == 0) cnt = 0;
    __syncthreads();
    // eligible CPs: count, and (for small pairs) their keys, compacted in
    // any order (the selection does not depend on it)
    const bool cached = n <= kConsCache;
    for (int i = threadIdx.x; i < n; i += kConsNT) {
        const sfoc_cp c = cps[i];
        if (c.flags & kBad) continue;
        const int slot = atomicAdd(&cnt, 1);
        if (cached) {
            keys[0][slot] = fkey(cp_disp(c, prior, i, 0));
            keys[1][slot] = fkey(cp_disp(c, prior, i, 1));
        }
    }
    __syncthreads();
    const int ne = cnt;
    if (ne == 0) return;
    // the median per axis: the middle key, or the mean of the two middle
    // ones (ranks ne/2 - 1 and ne/2) when ne is even
    const int axis[4] = {0, 0, 1, 1};
    int k[4] = {(ne - 1) / 2, ne / 2, (ne - 1) / 2, ne / 2};
    const uint32_t* const cache[2] = {cached ? keys[0] : nullptr, cached ? keys[1] : nullptr};
    uint32_t sk[4];
    select_kth4(cps, prior, n, axis, k, cache, ne, hist, sel, sk);
    float med[2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
        med[a] = (ne & 1) ? fkey_inv(sk[2 * a + 1]) : 0.5f * (fkey_inv(sk[2 * a]) + fkey_inv(sk[2 * a + 1]));
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += kConsNT) {
        sfoc_cp c = cps[i];
        if (c.flags & kBad) continue;
        const float ey = cp_disp(c, prior, i, 0) - med[0];
        const float ex = cp_disp(c, prior, i, 1) - med[1];
        c.flags |= (sqrtf(ey * ey + ex * ex) > 1.5f) ? SFOC_CP_INCONSISTENT : SFOC_CP_VALID;
        cps[i].flags = c.flags;
    }
}

// ---- per-window integral images (Eq. 14-16 over one search window) --------
// One workgroup per IP: G1 / G2 are the (M+1) x (M+1) exclusive prefix sums
// of sum_c g and sum_c g^2 (float64, of the stored values) over the IP's
// M x M search window, zero first row and column.  The window is taken in
// bands of rows that fit LDS: a wave takes a row, 64 columns at a time (a
// lane sums its pixel's channels in order, sixteen channels' loads in flight;
// a scan over the lanes and the carry of the columns before give the row
// prefix), then a thread per column and map adds the band's rows to the
// column's running sum and stores them.  Every sum is taken in a fixed order,
// so results are reproducible.  An IP whose windows leave the images is
// skipped (the match flags it and reads nothing).
// Bound by the windows' cache lines (a row of 52 bfloat16 values is 104 bytes
// of one or two 128-byte lines: 85 MB for 400 IPs at z = 16, 17 us at the rate
// of a large copy): 92 us with rows and columns walked one element at a time
// through global memory by one thread each, 24 us in this form (1024 threads:
// 27 us; eight channels in flight: 25 us).
constexpr int kWinNT = 512, kWinU = 16;   // threads; channels whose loads are in flight
constexpr int kWinLds = 48 << 10;   // LDS of a band: three workgroups per CU

// Rows of a band for windows of side M: what fits kWinLds (two float64 maps),
// at least one row per two waves (at the widest window, M = 1213, 78 KB).
static int window_band_rows(int M) {
    const int r = kWinLds / (16 * M);
    return r < 4 ? 4 : (r > M ? M : r);
}

template <int DT>
__global__ __launch_bounds__(kWinNT) void window_integral_kernel(const MatchArgs A, int R) {
    extern __shared__ double band[];   // [map][row][column]
    const int i = blockIdx.x, t = threadIdx.x, lane = t & 63, wv = t >> 6;
    const int m = A.m, r = A.r, M = m + 2 * r, P = M + 1;
    const int py = A.ips[2 * i], px = A.ips[2 * i + 1];
    const int pry = A.prior ? A.prior[2 * i] : 0, prx = A.prior ? A.prior[2 * i + 1] : 0;
    const int64_t ty = (int64_t)py - m / 2, tx = (int64_t)px - m / 2;
    const int64_t sy = ty - r + pry, sx = tx - r + prx;
    if (!in_image(ty, tx, m, m, A.Hs, A.Ws) || !in_image(sy, sx, M, M, A.Hr, A.Wr)) return;
    double* __restrict__ G1 = const_cast<double*>(A.integ1) + (int64_t)i * P * P;
    double* __restrict__ G2 = const_cast<double*>(A.integ2) + (int64_t)i * P * P;
    const int64_t plane = A.Hr * A.Wr;
    for (int e = t; e < P; e += kWinNT) {
        G1[e] = G2[e] = 0.0;
        G1[(int64_t)e * P] = G2[(int64_t)e * P] = 0.0;
    }
    // column work item: map q, column x; its running sum (one item per thread
    // up to M = 256, up to five for the widest window)
    constexpr int kItems = 5;
    double run[kItems];
#pragma unroll
    for (int k = 0; k < kItems; ++k) run[k] = 0.0;
    for (int y0 = 0; y0 < M; y0 += R) {
        const int rows = min(R, M - y0);
        for (int y = wv; y < rows; y += kWinNT / 64) {
            double c1 = 0.0, c2 = 0.0;   // sums of the columns before this chunk
            for (int x0 = 0; x0 < M; x0 += 64) {
                const int x = x0 + lane;
                const bool ok = x < M;
                const int o = (int)((sy + y0 + y) * A.Wr + sx + min(x, M - 1));   // within one plane (< 2^30)
                double s1 = 0.0, s2 = 0.0;
                for (int h0 = 0; h0 < A.z; h0 += kWinU) {
                    float g[kWinU];
#pragma unroll
                    for (int k = 0; k < kWinU; ++k)
                        g[k] = ldd<DT>(elem_ptr<DT>(A.desc_ref, (int64_t)min(h0 + k, A.z - 1) * plane), o);
#pragma unroll
                    for (int k = 0; k < kWinU; ++k)
                        if (h0 + k < A.z) {
                            const double d = (double)g[k];
                            s1 += d;
                            s2 = fma(d, d, s2);
                        }
                }
                s1 = ok ? s1 : 0.0;
                s2 = ok ? s2 : 0.0;
#pragma unroll
                for (int d = 1; d < 64; d <<= 1) {
                    const double u1 = __shfl_up(s1, d, 64), u2 = __shfl_up(s2, d, 64);
                    if (lane >= d) {
                        s1 += u1;
                        s2 += u2;
                    }
                }
                s1 += c1;
                s2 += c2;
                if (ok) {
                    band[y * M + x] = s1;
                    band[(R + y) * M + x] = s2;
                }
                c1 = __shfl(s1, 63, 64);
                c2 = __shfl(s2, 63, 64);
            }
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kItems; ++k) {
            const int e = t + k * kWinNT;
            if (e < 2 * M) {
                const int q = e >= M, x = e - q * M;
                const double* b = band + q * R * M + x;
                double* g = (q ? G2 : G1) + (int64_t)(y0 + 1) * P + x + 1;
                double a = run[k];
#pragma unroll 4
                for (int y = 0; y < rows; ++y) {
                    a += b[y * M];
                    g[(int64_t)y * P] = a;
                }
                run[k] = a;
            }
        }
        __syncthreads();
    }
}

template <int DT>
static hipError_t launch_window_integral(const MatchArgs& a, hipStream_t st) {
    const int M = a.m + 2 * a.r, R = window_band_rows(M);
    static_assert(5 * kWinNT >= 2 * (kMaxTemplate + 2 * kMaxRadiusMatch), "a column item for every column");
    const int lds = 2 * R * M * (int)sizeof(double);
    auto kern = window_integral_kernel<DT>;
    hipError_t e = ensure_dynamic_lds((const void*)kern, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(a.n), dim3(kWinNT), lds, st, a, R);
    return hipGetLastError();
}

// ---- launch -------------------------------------------------------------
void match_args_layout(MatchArgs& a, const MatchPlan& mp, void* ws) {
    a.nbu = a.nbv = mp.nb;
    a.Vb = mp.Vb;
    a.surf = nullptr;
    a.blk = nullptr;
    if (mp.nb > 1) {
        const int V = 2 * a.r + 1;
        a.surf = (float*)ws;
        a.blk = (float4*)((char*)ws + align_up((size_t)a.n * V * V * sizeof(float), 256));
    }
}

template <int L, int DT, bool SPLIT = false>
static hipError_t launch_match_L(const MatchArgs& a, hipStream_t st) {
    using C = MatchCfg<L>;
    auto kern = match_kernel<L, DT, false, SPLIT>;
    hipError_t e = ensure_dynamic_lds((const void*)kern, (int)C::lds_bytes);
    if (e != hipSuccess) return e;
    trace_begin(st, SFOC_K_MATCH);
    hipLaunchKernelGGL(kern, dim3(a.n * a.nbu * a.nbv), dim3(C::NT), C::lds_bytes, st, a, (const MatchArgs*)nullptr,
                       (const int4*)nullptr);
    trace_end(st, SFOC_K_MATCH);
    return hipGetLastError();
}

template <int DT, int NKB, bool BATCH>
static hipError_t launch_direct_K(const MatchArgs& a, const MatchArgs* pairs, const int4* items, int nblocks,
                                  int lds, hipStream_t st) {
    auto kern = match_direct_kernel<DT, NKB, BATCH>;
    hipError_t e = ensure_dynamic_lds((const void*)kern, lds);
    if (e != hipSuccess) return e;
    trace_begin(st, SFOC_K_MATCH);
    hipLaunchKernelGGL(kern, dim3(nblocks), dim3(kDirNT), lds, st, a, pairs, items);
    trace_end(st, SFOC_K_MATCH);
    return hipGetLastError();
}

template <int DT, bool BATCH>
static hipError_t launch_direct_DT(const MatchArgs& a, const MatchArgs* pairs, const int4* items, int nblocks,
                                   DirLaunch d, hipStream_t st) {
    const int lds = dir_geom(d.m, d.nkb).bytes;
    switch (d.nkb) {
        case 1: return launch_direct_K<DT, 1, BATCH>(a, pairs, items, nblocks, lds, st);
        case 2: return launch_direct_K<DT, 2, BATCH>(a, pairs, items, nblocks, lds, st);
        case 3: return launch_direct_K<DT, 3, BATCH>(a, pairs, items, nblocks, lds, st);
        case 4: return launch_direct_K<DT, 4, BATCH>(a, pairs, items, nblocks, lds, st);
        case 5: return launch_direct_K<DT, 5, BATCH>(a, pairs, items, nblocks, lds, st);
        case 6: return launch_direct_K<DT, 6, BATCH>(a, pairs, items, nblocks, lds, st);
        default: return hipErrorInvalidValue;
    }
}

// The direct form: one workgroup per IP of one pair (items null), or per
// (pair, IP) item; d holds the largest m and chunk count of the IPs' pairs.
static hipError_t launch_direct(const MatchArgs& a, const MatchArgs* pairs, const int4* items, int nblocks,
                                DirLaunch d, int dtype, hipStream_t st) {
    if (dtype == 1)
        return items ? launch_direct_DT<1, true>(a, pairs, items, nblocks, d, st)
                     : launch_direct_DT<1, false>(a, pairs, items, nblocks, d, st);
    if (dtype == 2)
        return items ? launch_direct_DT<2, true>(a, pairs, items, nblocks, d, st)
                     : launch_direct_DT<2, false>(a, pairs, items, nblocks, d, st);
    return hipErrorInvalidValue;
}

DirLaunch direct_launch_of(int m, int r) { return DirLaunch{m, dir_nkb(m, r)}; }

template <int L, bool SPLIT = false>
static hipError_t launch_match_side(const MatchArgs& a, int dtype, hipStream_t st) {
    return dtype == 0 ? launch_match_L<L, 0, SPLIT>(a, st)
                      : dtype == 1 ? launch_match_L<L, 1, SPLIT>(a, st) : launch_match_L<L, 2, SPLIT>(a, st);
}

// ---- split form: transforms, then NCC and peaks ----------------------------
bool match_split_ok(int n, int m, int r, int dtype) {
    const MatchPlan mp = match_plan_dt(n, m, r, dtype);
    return n > 0 && mp.L != kDirectSide && mp.L != 0 && mp.nb == 1;
}

static size_t split_rst_bytes(int n, int r) {
    const size_t V = 2 * (size_t)r + 1;
    return ((size_t)n * V * V * sizeof(float) + 255) / 256 * 256;
}

size_t match_split_bytes(int n, int r) { return split_rst_bytes(n, r) + (size_t)n * 2 * sizeof(double); }

// Where the spread form is taken.  It costs a second launch and a pass of the
// products through memory (4 L^2 bytes an IP and channel), and pays while the
// fused form's workgroups, one an IP, leave CUs idle.  Times of a pair call of
// 700 x 700 pixels, z = 16 (us, fused and spread):
//   L =  64:  n = 16  191   94;  256  210  142;  512  222  188;  640  261  230
//   L = 128:  n = 16  228  130;   64  230  154;  128  243  189;  192  265  282
//   L = 160:  n = 16  367  155;   64  365  212;   96  371  258;  128  372  350
//   L = 192:  n = 16  418  181;   64  439  270;   96  451  394;  128  459  459
// (beyond the line with the NCC in a launch of its own)
// and at n = 16, L = 64: z = 4  106  86;  z = 2  84  92.  The products are held
// to 160 MB (a scene's descriptors at 2048 x 2048 are 540).
constexpr size_t kSpreadBytes = 160000000;
constexpr int kSpreadMinZ = 4;
static size_t spread_item_bytes(int L) {
    return L == 64 ? Spread<64>::item_bytes : L == 128 ? Spread<128>::item_bytes
                   : L == 160 ? Spread<160>::item_bytes : Spread<192>::item_bytes;
}
static int spread_most(int L, int z) {   // IPs
    const int cap = L == 64 ? 512 : L == 128 ? 128 : 96;
    const size_t fit = kSpreadBytes / (spread_item_bytes(L) * (size_t)z);
    return z < kSpreadMinZ ? 0 : fit < (size_t)cap ? (int)fit : cap;
}

size_t match_spread_bytes(int n, int m, int r, int z, int dtype) {
    if (!match_split_ok(n, m, r, dtype)) return 0;
    const int L = match_plan_dt(n, m, r, dtype).L;
    return n <= spread_most(L, z) ? (size_t)n * z * spread_item_bytes(L) : 0;
}

static MatchArgs split_args(const void* desc_sen, int64_t Hs, int64_t Ws, const void* desc_ref, int64_t Hr,
                            int64_t Wr, const double* i1, const double* i2, int z, int dtype, const int32_t* ips,
                            const int32_t* prior, int n, int m, int r, float* ncc, sfoc_cp* cps, void* ws,
                            void* split) {
    MatchArgs a;
    a.desc_sen = desc_sen;
    a.desc_ref = desc_ref;
    a.integ1 = i1;
    a.integ2 = i2;
    a.ips = ips;
    a.prior = prior;
    a.ncc = ncc;
    a.cps = cps;
    a.Hs = Hs;
    a.Ws = Ws;
    a.Hr = Hr;
    a.Wr = Wr;
    a.z = z;
    a.dtype = dtype;
    a.n = n;
    a.m = m;
    a.r = r;
    match_args_layout(a, match_plan_dt(n, m, r, dtype), ws);
    a.integ_win = 0;
    a.rst = (float*)split;
    a.tsum = (double*)((char*)split + split_rst_bytes(n, r));
    return a;
}

template <int L, int DT>
static hipError_t launch_spectra(const MatchArgs& a, hipStream_t st) {
    using C = MatchCfg<L>;
    auto kern = match_spectra_kernel<L, DT>;
    hipError_t e = ensure_dynamic_lds((const void*)kern, (int)C::lds_bytes);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(a.n * a.z + a.n), dim3(C::NT), C::lds_bytes, st, a);
    return hipGetLastError();
}
// The spread form's scratch (match_spread_bytes) in the arguments.
template <int L>
static void spread_args(MatchArgs& a, void* scratch) {
    const size_t items = (size_t)a.n * a.z;
    a.spec = (float2*)scratch;
    a.spec_self = a.spec + items * Spread<L>::bins;
    a.spec_sum = (double*)(a.spec_self + items * 4);
}
template <int L>
static hipError_t launch_combine(MatchArgs a, void* spread, hipStream_t st) {
    using C = MatchCfg<L>;
    spread_args<L>(a, spread);
    auto kern = match_combine_kernel<L>;
    hipError_t e = ensure_dynamic_lds((const void*)kern, (int)C::lds_bytes);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(a.n), dim3(C::NT), C::lds_bytes, st, a);
    return hipGetLastError();
}
template <int L>
static hipError_t launch_transforms(MatchArgs a, void* spread, hipStream_t st) {
    if (!spread) return launch_match_side<L, true>(a, a.dtype, st);
    spread_args<L>(a, spread);
    trace_begin(st, SFOC_K_MATCH);
    hipError_t e = a.dtype == 0   ? launch_spectra<L, 0>(a, st)
                   : a.dtype == 1 ? launch_spectra<L, 1>(a, st) : launch_spectra<L, 2>(a, st);
    if (e == hipSuccess && !spread_peak<L>()) e = launch_combine<L>(a, spread, st);
    trace_end(st, SFOC_K_MATCH);
    return e;
}

hipError_t launch_match_fft(const void* desc_sen, int64_t Hs, int64_t Ws, const void* desc_ref, int64_t Hr,
                            int64_t Wr, int z, int dtype, const int32_t* ips, const int32_t* prior, int n, int m,
                            int r, float* ncc, sfoc_cp* cps, void* ws, void* split, void* spread, hipStream_t st) {
    if (!match_split_ok(n, m, r, dtype)) return hipErrorInvalidValue;
    const MatchArgs a = split_args(desc_sen, Hs, Ws, desc_ref, Hr, Wr, nullptr, nullptr, z, dtype, ips, prior, n, m,
                                   r, ncc, cps, ws, split);
    if (!match_spread_bytes(n, m, r, z, dtype)) spread = nullptr;
    switch (match_plan_dt(n, m, r, dtype).L) {
        case 64: return launch_transforms<64>(a, spread, st);
        case 128: return launch_transforms<128>(a, spread, st);
        case 160: return launch_transforms<160>(a, spread, st);
        case 192: return launch_transforms<192>(a, spread, st);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_match_finish(const void* desc_sen, int64_t Hs, int64_t Ws, const void* desc_ref, int64_t Hr,
                               int64_t Wr, const double* i1, const double* i2, int z, int dtype, const int32_t* ips,
                               const int32_t* prior, int n, int m, int r, float* ncc, sfoc_cp* cps, void* ws,
                               void* split, void* spread, hipStream_t st, bool consistency) {
    if (!match_split_ok(n, m, r, dtype) || !i1 || !i2) return hipErrorInvalidValue;
    const MatchArgs a = split_args(desc_sen, Hs, Ws, desc_ref, Hr, Wr, i1, i2, z, dtype, ips, prior, n, m, r, ncc,
                                   cps, ws, split);
    hipError_t e;
    trace_begin(st, SFOC_K_PEAK);
    const int L = match_plan_dt(n, m, r, dtype).L;
    if (L > 64 && spread && match_spread_bytes(n, m, r, z, dtype)) {
        static_assert(!spread_peak<64>() && spread_peak<128>() && spread_peak<160>() && spread_peak<192>(), "as here");
        switch (L) {
            case 128: e = launch_combine<128>(a, spread, st); break;
            case 160: e = launch_combine<160>(a, spread, st); break;
            default: e = launch_combine<192>(a, spread, st); break;
        }
    } else {
        hipLaunchKernelGGL(ncc_finish_kernel, dim3(n), dim3(kFinishNT), 0, st, a);
        e = hipGetLastError();
    }
    trace_end(st, SFOC_K_PEAK);
    if (e != hipSuccess || !consistency) return e;
    return launch_consistency(cps, prior, n, st);
}

hipError_t launch_match(const void* desc_sen, int64_t Hs, int64_t Ws, const void* desc_ref, int64_t Hr, int64_t Wr,
                        const double* i1, const double* i2, int z, int dtype, const int32_t* ips,
                        const int32_t* prior, int n, int m, int r, float* ncc, sfoc_cp* cps, void* ws,
                        hipStream_t st, bool consistency) {
    MatchArgs a;
    a.desc_sen = desc_sen;
    a.desc_ref = desc_ref;
    a.integ1 = i1;
    a.integ2 = i2;
    a.ips = ips;
    a.prior = prior;
    a.ncc = ncc;
    a.cps = cps;
    a.Hs = Hs;
    a.Ws = Ws;
    a.Hr = Hr;
    a.Wr = Wr;
    a.z = z;
    a.dtype = dtype;
    a.n = n;
    a.m = m;
    a.r = r;
    const MatchPlan mp = match_plan_dt(n, m, r, dtype);
    const int L = mp.L;
    match_args_layout(a, mp, ws);
    a.integ_win = 0;
    hipError_t e;
    if (!i1) {   // per-window integral images, after the split-offset scratch
        double* g = (double*)((char*)ws + mp.ws_bytes);
        const size_t per = (size_t)(m + 2 * r + 1) * (m + 2 * r + 1);
        a.integ1 = g;
        a.integ2 = g + (size_t)n * per;
        a.integ_win = 1;
        trace_begin(st, SFOC_K_INTEGRAL);
        e = dtype == 0 ? launch_window_integral<0>(a, st)
                       : dtype == 1 ? launch_window_integral<1>(a, st) : launch_window_integral<2>(a, st);
        trace_end(st, SFOC_K_INTEGRAL);
        if (e != hipSuccess) return e;
    }
    switch (L) {
        case 64: e = launch_match_side<64>(a, dtype, st); break;
        case 128: e = launch_match_side<128>(a, dtype, st); break;
        case 160: e = launch_match_side<160>(a, dtype, st); break;
        case 192: e = launch_match_side<192>(a, dtype, st); break;
        case kDirectSide: e = launch_direct(a, nullptr, nullptr, n, direct_launch_of(m, r), dtype, st); break;
        default: return hipErrorInvalidValue;
    }
    if (e != hipSuccess) return e;
    if (mp.nb > 1) {
        trace_begin(st, SFOC_K_PEAK);
        hipLaunchKernelGGL(peak_kernel<false>, dim3((n + 255) / 256), dim3(256), 0, st, a, (const MatchArgs*)nullptr,
                           (const int4*)nullptr);
        trace_end(st, SFOC_K_PEAK);
    }
    if (!consistency) return hipGetLastError();
    return launch_consistency(cps, prior, n, st);
}

hipError_t launch_consistency(sfoc_cp* cps, const int32_t* prior, int n, hipStream_t st) {
    if (n == 0) return hipSuccess;
    trace_begin(st, SFOC_K_CONSISTENCY);
    hipLaunchKernelGGL(consistency_kernel, dim3(1), dim3(kConsNT), 0, st, cps, prior, n, (const MatchArgs*)nullptr);
    trace_end(st, SFOC_K_CONSISTENCY);
    return hipGetLastError();
}

// Adds dy to the sensed row of n CP records (records of IPs matched in a
// band of rows, whose coordinates were taken relative to the band).
__global__ __launch_bounds__(256) void cp_row_shift_kernel(sfoc_cp* cps, int n, int dy) {
    const int i = (int)(blockIdx.x * 256 + threadIdx.x);
    if (i < n) cps[i].sen_row += dy;
}

hipError_t launch_cp_row_shift(sfoc_cp* cps, int n, int dy, hipStream_t st) {
    if (n == 0 || dy == 0) return hipSuccess;
    hipLaunchKernelGGL(cp_row_shift_kernel, dim3((n + 255) / 256), dim3(256), 0, st, cps, n, dy);
    return hipGetLastError();
}

// ---- batched launches ---------------------------------------------------
template <int L, int DT>
static hipError_t launch_match_items_L(const MatchArgs* pairs, const int4* items, int nitems, int* counter, int grid,
                                       hipStream_t st) {
    using C = MatchCfg<L>;
    MatchArgs none{};
    hipError_t e;
    if (counter) {
        auto kern = match_persistent_kernel<L, DT>;
        if ((e = ensure_dynamic_lds((const void*)kern, (int)C::lds_bytes)) != hipSuccess) return e;
        trace_begin(st, SFOC_K_MATCH);
        hipLaunchKernelGGL(zero_counter_kernel, dim3(1), dim3(1), 0, st, counter);
        const int g = grid * C::MINB;   // `grid` counts CUs
        hipLaunchKernelGGL(kern, dim3(g < nitems ? g : nitems), dim3(C::NT), C::lds_bytes, st, pairs, items,
                           nitems, counter);
        trace_end(st, SFOC_K_MATCH);
    } else {
        auto kern = match_kernel<L, DT, true>;
        if ((e = ensure_dynamic_lds((const void*)kern, (int)C::lds_bytes)) != hipSuccess) return e;
        trace_begin(st, SFOC_K_MATCH);
        hipLaunchKernelGGL(kern, dim3(nitems), dim3(C::NT), C::lds_bytes, st, none, pairs, items);
        trace_end(st, SFOC_K_MATCH);
    }
    return hipGetLastError();
}

template <int L>
static hipError_t launch_match_items_side(int dtype, const MatchArgs* pairs, const int4* items, int nitems,
                                          int* counter, int grid, hipStream_t st) {
    return dtype == 0 ? launch_match_items_L<L, 0>(pairs, items, nitems, counter, grid, st)
         : dtype == 1 ? launch_match_items_L<L, 1>(pairs, items, nitems, counter, grid, st)
                      : launch_match_items_L<L, 2>(pairs, items, nitems, counter, grid, st);
}

// One launch over (pair, IP, block) items that share the transform side L:
// one workgroup per item, or (counter != null) a persistent grid of `grid`
// workgroups taking items from *counter.  The direct form (L = kDirectSide)
// takes one workgroup per item, sized by `dir`.
hipError_t launch_match_items(int L, int dtype, const MatchArgs* pairs, const int4* items, int nitems, int* counter,
                              int grid, DirLaunch dir, hipStream_t st) {
    if (nitems == 0) return hipSuccess;
    if (L == kDirectSide) {
        if (counter) return hipErrorInvalidValue;
        MatchArgs none{};
        return launch_direct(none, pairs, items, nitems, dir, dtype, st);
    }
    switch (L) {
        case 64: return launch_match_items_side<64>(dtype, pairs, items, nitems, counter, grid, st);
        case 128: return launch_match_items_side<128>(dtype, pairs, items, nitems, counter, grid, st);
        case 160: return launch_match_items_side<160>(dtype, pairs, items, nitems, counter, grid, st);
        case 192: return launch_match_items_side<192>(dtype, pairs, items, nitems, counter, grid, st);
        default: return hipErrorInvalidValue;
    }
}

// Peak of split pairs: items {pair, first IP of a run of 256}.
hipError_t launch_peak_batched(const MatchArgs* pairs, const int4* items, int nitems, hipStream_t st) {
    if (nitems == 0) return hipSuccess;
    MatchArgs none{};
    trace_begin(st, SFOC_K_PEAK);
    hipLaunchKernelGGL(peak_kernel<true>, dim3(nitems), dim3(256), 0, st, none, pairs, items);
    trace_end(st, SFOC_K_PEAK);
    return hipGetLastError();
}

// Consistency of every pair of a plan: one workgroup per pair.
hipError_t launch_consistency_batched(const MatchArgs* pairs, int npairs, hipStream_t st) {
    if (npairs == 0) return hipSuccess;
    trace_begin(st, SFOC_K_CONSISTENCY);
    hipLaunchKernelGGL(consistency_kernel, dim3(npairs), dim3(kConsNT), 0, st, (sfoc_cp*)nullptr,
                       (const int32_t*)nullptr, 0, pairs);
    trace_end(st, SFOC_K_CONSISTENCY);
    return hipGetLastError();
}

}  // namespace sfoc
