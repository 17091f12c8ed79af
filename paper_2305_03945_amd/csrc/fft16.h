// Workgroup FFT, V = 4, 8 or 16 values per thread.
//
// A length-N transform (N = 2^LOGN, 16 <= N <= 4096) is done by N/V threads, in an
// LDS region of N complex values with padding (lds_pad), which keeps the stride-R
// writes of a Stockham pass off a single bank group.  Threads of one wave synchronise
// within it, a transform over several waves by the workgroup's barrier.  Passes are
// Stockham autosort passes of radix V, then one pass of a smaller radix for the
// remaining bits; each thread runs V/R butterflies of a radix-R pass.  A butterfly gathers
// the powers W^{k}, W^{2k}, W^{4k}, W^{8k} of its twiddle and applies them in its radix-2
// steps (twiddled_dft).
#pragma once
#include "fft.h"

namespace rdk {

// ---- twiddled DFT of one butterfly
//
// V_q = sum_r v_r w^r W_R^{qr}, W_R = exp(DIR 2 pi i / R), by decimation in time: radix-2
// steps on the DFTs E, O (of R/2 points, for w^2) of the even and odd inputs,
//     V_q = E_q + t O_q,   V_{q+R/2} = E_q - t O_q,   t = w W_R^q,
// in eight multiply-adds, so that only w, w^2, w^4, ... are needed; t for q >= R/4 is t
// for q - R/4 turned by 90 degrees.  A radix-16 butterfly takes 256 operations, against 272
// when its 15 twiddles are formed and applied first.
//
// The rounding error is to be no larger than with twiddles formed and applied first.  G^-1
// at 512^2 against 80-bit transforms: 4.3e-16 (FP64) and 2.4e-7 (FP32), 4.5e-16 and 2.7e-7
// that way, 5.2e-16 and 2.8e-7 with the cheaper butterfly of the next lines, against which
// this one costs 2 % of a step (2048^2 1246 -> 1276 us mixed, 2608 -> 2673 FP64).  Of a
// 512-point FP64 transform and its inverse, in units of the rounding (FP32): 2.57 (2.80)
// that way; 2.51 (2.59) this with 8 values per thread, 2.45 (2.65) with 16.  What was
// found to cost accuracy:
//  - V_{q+R/2} as 2 E_q - V_q, which saves two operations but takes over V_q's rounding
//    (one transform: 2.01 against 1.80 formed first);
//  - w W_8 by the rounded sqrt(1/2), whose error goes into every value with the same sign
//    (2.60, 16 values; turn8 adds its lower part);
//  - radix-2 steps down to two points on short transforms, whose error is small (32
//    points, 8 values: 1.69, formed first 1.65).  Up to 64 points the DFTs of four multiply
//    their twiddles in first and w W_8 is gathered (1.61); above, the two twiddles more
//    would cost registers.
template <typename T> __device__ __forceinline__ T fma_(T a, T b, T c) { return __builtin_elementwise_fma(a, b, c); }

// exp(DIR 2 pi i m / 16), m = 1, 2, 3
template <typename T, int DIR, int M> __device__ __forceinline__ cplx<T> root16() {
    static_assert(M >= 1 && M <= 3, "first-quadrant roots");
    constexpr T c[4] = {(T)1, (T)0.923879532511286756128183189396788934, (T)0.707106781186547524400844362104849039,
                        (T)0.382683432365089771728459984030398867};
    return {c[M], (T)DIR * c[4 - M]};
}

// w exp(DIR 2 pi i / 8), with sqrt(1/2) in two parts.
template <typename T, int DIR> __device__ __forceinline__ cplx<T> turn8(cplx<T> w) {
    constexpr T hi = (T)0.707106781186547524400844362104849039;
    constexpr T lo = (T)(sizeof(T) == 8 ? -4.83364665672645651859e-17 : 1.21016171044788e-08);
    const cplx<T> c = cadd(w, rot90<T, DIR>(w));
    return {fma_(hi, c.re, lo * c.re), fma_(hi, c.im, lo * c.im)};
}

// a + t b and a - t b.  QUARTER: t is to be turned by DIR 90 degrees.
template <typename T, int DIR, bool QUARTER>
__device__ __forceinline__ void bfly(cplx<T> a, cplx<T> b, cplx<T> t, cplx<T> &lo, cplx<T> &hi) {
    if constexpr (QUARTER) b = rot90<T, DIR>(b);
    lo.re = fma_(-t.im, b.im, fma_(t.re, b.re, a.re));
    lo.im = fma_(t.im, b.re, fma_(t.re, b.im, a.im));
    hi.re = fma_(t.im, b.im, fma_(-t.re, b.re, a.re));
    hi.im = fma_(-t.im, b.re, fma_(-t.re, b.im, a.im));
}

// The radix-2 step of R points; t: the R / 4 twiddles.
template <typename T, int R, int DIR>
__device__ __forceinline__ void radix2_step(const cplx<T> *e, const cplx<T> *o, const cplx<T> *t, cplx<T> *out) {
    constexpr int QT = R / 4;
#pragma unroll
    for (int q = 0; q < QT; ++q) {
        bfly<T, DIR, false>(e[q], o[q], t[q], out[q], out[q + R / 2]);
        bfly<T, DIR, true>(e[q + QT], o[q + QT], t[q], out[q + QT], out[q + QT + R / 2]);
    }
}

template <typename T> __device__ __forceinline__ void dft2(cplx<T> *v) {
    const cplx<T> a = v[0], b = v[1];
    v[0] = cadd(a, b);
    v[1] = csub(a, b);
}

template <typename T, int DIR> __device__ __forceinline__ void dft4(cplx<T> *v) {
    const cplx<T> e0 = cadd(v[0], v[2]), e1 = csub(v[0], v[2]);
    const cplx<T> o0 = cadd(v[1], v[3]), o1 = rot90<T, DIR>(csub(v[1], v[3]));
    v[0] = cadd(e0, o0);
    v[1] = cadd(e1, o1);
    v[2] = csub(e0, o0);
    v[3] = csub(e1, o1);
}

// Two DFTs of four, and the radix-2 step with W_8 = sqrt(1/2) (1 + DIR i).
template <typename T, int DIR> __device__ __forceinline__ void dft8(cplx<T> *v) {
    cplx<T> e[4] = {v[0], v[2], v[4], v[6]}, o[4] = {v[1], v[3], v[5], v[7]};
    dft4<T, DIR>(e);
    dft4<T, DIR>(o);
    o[2] = rot90<T, DIR>(o[2]);
    o[3] = rot90<T, DIR>(o[3]);
    const T s = root16<T, DIR, 2>().re;
#pragma unroll
    for (int q = 0; q < 4; q += 2) {
        v[q] = cadd(e[q], o[q]);
        v[q + 4] = csub(e[q], o[q]);
    }
#pragma unroll
    for (int q = 1; q < 4; q += 2) {
        const cplx<T> r = rot90<T, DIR>(o[q]), c = cadd(o[q], r);
        v[q] = {fma_(s, c.re, e[q].re), fma_(s, c.im, e[q].im)};
        v[q + 4] = {fma_(-s, c.re, e[q].re), fma_(-s, c.im, e[q].im)};
    }
}

// DFTs of four over inputs four apart, W_16^{s q}, DFTs of four over s.
template <typename T, int DIR> __device__ __forceinline__ void dft16(cplx<T> *v) {
    cplx<T> a[4][4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
#pragma unroll
        for (int r = 0; r < 4; ++r) a[s][r] = v[s + 4 * r];
        dft4<T, DIR>(a[s]);
    }
    a[1][1] = cmul(a[1][1], root16<T, DIR, 1>());
    a[1][2] = cmul(a[1][2], root16<T, DIR, 2>());
    a[1][3] = cmul(a[1][3], root16<T, DIR, 3>());
    a[2][1] = cmul(a[2][1], root16<T, DIR, 2>());
    a[2][2] = rot90<T, DIR>(a[2][2]);
    a[2][3] = rot90<T, DIR>(cmul(a[2][3], root16<T, DIR, 2>()));
    a[3][1] = cmul(a[3][1], root16<T, DIR, 3>());
    a[3][2] = rot90<T, DIR>(cmul(a[3][2], root16<T, DIR, 2>()));
    a[3][3] = cmul(a[3][3], root16<T, DIR, 1>());   // W_16^9 = -W_16
    a[3][3] = {-a[3][3].re, -a[3][3].im};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        cplx<T> b[4] = {a[0][q], a[1][q], a[2][q], a[3][q]};
        dft4<T, DIR>(b);
#pragma unroll
        for (int r = 0; r < 4; ++r) v[q + 4 * r] = b[r];
    }
}

// DFT_R of v in place.
template <typename T, int R, int DIR> __device__ __forceinline__ void dftR(cplx<T> *v) {
    if constexpr (R == 16) dft16<T, DIR>(v);
    else if constexpr (R == 8) dft8<T, DIR>(v);
    else if constexpr (R == 4) dft4<T, DIR>(v);
    else dft2<T>(v);
}

// Twiddles kept per butterfly of an N-point transform by V values per thread: the powers
// w, w^2, w^4, ..., then (tw_has_w3) w^{3R/4}, the last input's in a DFT of four, then
// (tw_has_w8) the 8-point step's power times W_8.
template <int V> constexpr int logv() { return V == 16 ? 4 : V == 8 ? 3 : 2; }
template <int LOGN> constexpr bool twiddles_first() { return LOGN <= 6; }
template <int LOGN, int V> constexpr bool tw_has_w3() { return twiddles_first<LOGN>() && V <= 8; }
template <int LOGN, int V> constexpr bool tw_has_w8() { return twiddles_first<LOGN>() && V == 8; }
template <int LOGN, int V> constexpr int tw_count() {
    return logv<V>() + (tw_has_w3<LOGN, V>() ? 1 : 0) + (tw_has_w8<LOGN, V>() ? 1 : 0);
}

// Gather a radix-R butterfly's twiddles: w = W_N^i, table tw of W_N (forward sign).
template <typename T, int LOGN, int V, int R, class TAB>
__device__ __forceinline__ void gather_twiddles(cplx<T> *p, TAB tw, int i) {
    constexpr int N = 1 << LOGN;
    auto at = [&](int m) { return cplx<T>{tw[m & (N - 1)].re, tw[m & (N - 1)].im}; };
#pragma unroll
    for (int e = 0; e < logv<V>(); ++e)
        if ((1 << e) < R) p[e] = at(i << e);
    if constexpr (tw_has_w3<LOGN, V>() && R >= 4) p[logv<V>()] = at(i * (3 * R / 4));
    if constexpr (tw_has_w8<LOGN, V>() && R >= 8) p[tw_count<LOGN, V>() - 1] = at(i * (R / 8) + N / 8);
}

// DFT_R of v in place, input r multiplied by w^r first; p: gather_twiddles (forward sign,
// conjugated here for the inverse).
template <typename T, int LOGN, int V, int R, int DIR>
__device__ __forceinline__ void twiddled_dft(cplx<T> *v, const cplx<T> *p) {
    auto tw = [&](int e) { return DIR > 0 ? cconj(p[e]) : p[e]; };
    if constexpr (R == 2) {
        bfly<T, DIR, false>(v[0], v[1], tw(0), v[0], v[1]);
    } else {
        constexpr int NL = R / 4;                                // DFTs of four
        constexpr int E = R == 16 ? 2 : R == 8 ? 1 : 0;          // their twiddle is w^{R/4}
        const cplx<T> l1 = tw(E), l2 = tw(E + 1);
        cplx<T> a[NL][4];
        if constexpr (twiddles_first<LOGN>()) {
            cplx<T> l3;
            if constexpr (tw_has_w3<LOGN, V>()) l3 = tw(logv<V>());
            else l3 = cmul(l1, l2);
#pragma unroll
            for (int s = 0; s < NL; ++s) {
                a[s][0] = v[s];
                a[s][1] = cmul(v[s + NL], l1);
                a[s][2] = cmul(v[s + 2 * NL], l2);
                a[s][3] = cmul(v[s + 3 * NL], l3);
                dft4<T, DIR>(a[s]);
            }
        } else {
#pragma unroll
            for (int s = 0; s < NL; ++s) {
                cplx<T> e[2], o[2];
                bfly<T, DIR, false>(v[s], v[s + 2 * NL], l2, e[0], e[1]);
                bfly<T, DIR, false>(v[s + NL], v[s + 3 * NL], l2, o[0], o[1]);
                radix2_step<T, 4, DIR>(e, o, &l1, a[s]);
            }
        }
        if constexpr (R == 4) {
#pragma unroll
            for (int q = 0; q < 4; ++q) v[q] = a[0][q];
        } else {
            cplx<T> t8[2] = {tw(E - 1)};
            if constexpr (tw_has_w8<LOGN, V>()) t8[1] = tw(tw_count<LOGN, V>() - 1);
            else t8[1] = turn8<T, DIR>(t8[0]);
            if constexpr (R == 8) {
                radix2_step<T, 8, DIR>(a[0], a[1], t8, v);
            } else {
                cplx<T> e[8], o[8];
                radix2_step<T, 8, DIR>(a[0], a[2], t8, e);
                radix2_step<T, 8, DIR>(a[1], a[3], t8, o);
                const cplx<T> w = tw(0);
                const cplx<T> t16[4] = {w, cmul(w, root16<T, DIR, 1>()), turn8<T, DIR>(w),
                                        cmul(w, root16<T, DIR, 3>())};
                radix2_step<T, 16, DIR>(e, o, t16, v);
            }
        }
    }
}

// Values per thread of a transform, V: 16 where the chip is full of transforms, 8 or 4
// where it is not (short serial chains; see RowsPlan and col_values).  Radix of pass q of a
// length-2^LOGN transform: radix V while that many bits remain, then one pass of
// what is left.
template <int LOGN, int V = 16> constexpr int npasses16() { return (LOGN + logv<V>() - 1) / logv<V>(); }
template <int LOGN, int V = 16> constexpr int pass_radix(int q) {
    return LOGN - logv<V>() * q >= logv<V>() ? V : (1 << (LOGN - logv<V>() * q));
}

// The twiddles of one thread for every pass after the first: those of butterfly b of
// pass q for w = exp(-2 pi i k / (NS R)), k = j mod NS.  They depend only on the thread's
// index in its transform team, so a kernel loads them once, at its start, and
// every transform (forward and inverse) of the kernel reuses them.
template <typename T, int LOGN, int V = 16> struct Tw16 {
    cplx<T> p[npasses16<LOGN, V>() > 1 ? npasses16<LOGN, V>() - 1 : 1][V / 2][tw_count<LOGN, V>()];
};

template <typename T, int LOGN, int V, int Q = 1>
__device__ __forceinline__ void load_tw16(Tw16<T, LOGN, V> &w, const cplx<T> *__restrict__ tw, int t) {
    if constexpr (Q < npasses16<LOGN, V>()) {
        constexpr int R = pass_radix<LOGN, V>(Q), NS = 1 << (logv<V>() * Q), N = 1 << LOGN;
#pragma unroll
        for (int b = 0; b < V / R; ++b)
            gather_twiddles<T, LOGN, V, R>(w.p[Q - 1][b], gp(tw), ((t + b * (N / V)) & (NS - 1)) * (N / (NS * R)));
        load_tw16<T, LOGN, V, Q + 1>(w, tw, t);
    }
}

template <typename T, int LOGN, int V>
__device__ __forceinline__ void load_tw16(Tw16<T, LOGN, V> &w, const cplx<T> *__restrict__ tw) {
    load_tw16<T, LOGN, V>(w, tw, (int)(threadIdx.x % ((1 << LOGN) / V)));
}

// One Stockham pass of radix R (NS = product of earlier radices).  Butterfly j
// reads x[j + r N/R], twiddles input r by W_{NS R}^{r k} (k = j mod NS), applies
// DFT_R, and writes output q to ((j - k) R + k) + q NS.  pw: the thread's
// gathered powers for this pass (unused when NS = 1).  Thread t of a transform
// runs butterflies j = t + b N/V, b < V/R.
//
// x: accessor of the transform's elements (x(i): element i in LDS); a region is
// Region<T, LOGN>{pointer}.
template <typename T, int LOGN> struct Region {
    cplx<T> *p;
    __device__ __forceinline__ cplx<T> &operator()(int i) const { return p[lds_pad<LOGN>(i)]; }
};

// pass_in: the reads, twiddles and butterflies of the thread (outputs in v).
template <typename T, int LOGN, int R, int NS, int DIR, int V = 16, class X>
__device__ __forceinline__ void pass_in(X x, int t, const cplx<T> (*pw)[tw_count<LOGN, V>()], cplx<T> (*v)[R]) {
    constexpr int N = 1 << LOGN;
    constexpr int TPF = N / V;       // threads per transform
    constexpr int NB = N / R;        // butterflies
    constexpr int BPT = V / R;       // butterflies per thread
#pragma unroll
    for (int b = 0; b < BPT; ++b) {
        const int j = t + b * TPF;
#pragma unroll
        for (int r = 0; r < R; ++r) v[b][r] = x(j + r * NB);
        if constexpr (NS > 1) twiddled_dft<T, LOGN, V, R, DIR>(v[b], pw[b]);
        else dftR<T, R, DIR>(v[b]);
    }
}

// pass_out: the Stockham writes of the thread's butterfly outputs.
template <typename T, int LOGN, int R, int NS, int V = 16, class X>
__device__ __forceinline__ void pass_out(X x, int t, const cplx<T> (*v)[R]) {
    constexpr int TPF = (1 << LOGN) / V;
#pragma unroll
    for (int b = 0; b < V / R; ++b) {
        const int j = t + b * TPF;
        const int k = j & (NS - 1);
        const int base = (j - k) * R + k;
#pragma unroll
        for (int q = 0; q < R; ++q) x(base + q * NS) = v[b][q];
    }
}

// Barrier between the passes of a transform.  WAVE: the transform's threads are
// lanes of one wave, whose LDS accesses execute in order, so only the compiler
// has to keep them in order and the workgroup's other waves need not be waited for.
template <bool WAVE> __device__ __forceinline__ void pass_sync() {
    if constexpr (WAVE) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    } else {
        __syncthreads();
    }
}

template <typename T, int LOGN, int R, int NS, int DIR, int V = 16, bool WAVE = false, class X>
__device__ __forceinline__ void pass16(X x, int t, bool active, const cplx<T> (*pw)[tw_count<LOGN, V>()]) {
    cplx<T> v[V / R][R];
    if (active) pass_in<T, LOGN, R, NS, DIR, V>(x, t, pw, v);
    pass_sync<WAVE>();
    if (active) pass_out<T, LOGN, R, NS, V>(x, t, v);
    pass_sync<WAVE>();
}

template <typename T, int LOGN, int DIR, int DONE, int V, bool WAVE, class X>
__device__ __forceinline__ void passes16(X x, int t, bool active, const Tw16<T, LOGN, V> &w) {
    if constexpr (DONE < LOGN) {
        constexpr int q = DONE / logv<V>();
        constexpr int R = pass_radix<LOGN, V>(q);
        constexpr int LOGR = LOGN - DONE >= logv<V>() ? logv<V>() : LOGN - DONE;
        pass16<T, LOGN, R, (1 << DONE), DIR, V, WAVE>(x, t, active, w.p[q > 0 ? q - 1 : 0]);
        passes16<T, LOGN, DIR, DONE + LOGR, V, WAVE>(x, t, active, w);
    }
}

// ---- transforms whose first input and last output stay in registers
//
// Thread t of a transform holds its V values in "stride order": value r is
// element t + r N/V.  That is what the first radix-V pass reads (NS = 1,
// butterfly j = t) and, for the last pass of radix RL (NS = N/RL, butterflies
// j = t + b N/V with k = j), output q of butterfly b lands at
// t + (b + q V/RL) N/V, again element t + r N/V with r = b + q V/RL.  So a
// transform can start from values loaded straight from global memory and end
// with values ready to be stored, with LDS used only between passes.

// Radix of the last pass and the register index of its output (b, q).
template <int LOGN, int V = 16> constexpr int last_radix() {
    return pass_radix<LOGN, V>(npasses16<LOGN, V>() - 1);
}
template <int LOGN, int V = 16> __host__ __device__ constexpr int last_slot(int b, int q) {
    return b + q * (V / last_radix<LOGN, V>());
}

// Middle passes q = 1 .. npasses - 2 (all radix V), each ending with a barrier.
template <typename T, int LOGN, int DIR, int Q, int V, class X>
__device__ __forceinline__ void middle_passes(X x, int t, const Tw16<T, LOGN, V> &w) {
    if constexpr (Q < npasses16<LOGN, V>() - 1) {
        pass16<T, LOGN, V, (1 << (logv<V>() * Q)), DIR, V>(x, t, true, w.p[Q - 1]);
        middle_passes<T, LOGN, DIR, Q + 1, V>(x, t, w);
    }
}

// Transform of one region whose input v (stride order) is in registers; the
// output is left in v (stride order).  Needs at least two passes.  Starts by
// writing the region (the caller makes sure no thread still reads it) and ends with the
// last pass's reads of it (the caller places a barrier before it is rewritten).
template <typename T, int LOGN, int DIR, int V>
__device__ __forceinline__ void fft16_regs(cplx<T> *region, int t, const Tw16<T, LOGN, V> &w, cplx<T> *v) {
    const Region<T, LOGN> x{region};
    static_assert(npasses16<LOGN, V>() >= 2, "register-ended transforms need two passes");
    constexpr int NP = npasses16<LOGN, V>();
    constexpr int RL = last_radix<LOGN, V>();
    dftR<T, V, DIR>(v);
#pragma unroll
    for (int q = 0; q < V; ++q) x(V * t + q) = v[q];
    __syncthreads();
    middle_passes<T, LOGN, DIR, 1, V>(x, t, w);
    cplx<T> o[V / RL][RL];
    pass_in<T, LOGN, RL, (1 << (logv<V>() * (NP - 1))), DIR, V>(x, t, w.p[NP - 2], o);
#pragma unroll
    for (int b = 0; b < V / RL; ++b)
#pragma unroll
        for (int q = 0; q < RL; ++q) v[last_slot<LOGN, V>(b, q)] = o[b][q];
}

// In-place transforms of NREG regions (region i at buf + i * lds_region<LOGN>(),
// padded indexing) by a workgroup of NTH threads; teams of N/V consecutive
// threads take regions round-robin.  Ends with a barrier.  DIR -1 forward, +1
// inverse.  w: the thread's twiddles (load_tw16).
template <typename T, int LOGN, int DIR, int NREG, int NTH, int V = 16>
__device__ __forceinline__ void wg_fft16(cplx<T> *buf, const Tw16<T, LOGN, V> &w) {
    constexpr int TPF = (1 << LOGN) / V;
    static_assert(NTH % TPF == 0 || TPF > NTH, "team must divide the workgroup");
    constexpr int NTEAMS = NTH / TPF;
    constexpr bool WAVE = TPF <= 64;
    const int team = threadIdx.x / TPF, t = threadIdx.x % TPF;
#pragma unroll 1
    for (int g = 0; g < NREG; g += NTEAMS) {
        const int reg = g + team;
        const bool active = reg < NREG;
        const Region<T, LOGN> x{buf + (active ? reg : 0) * lds_region<LOGN>()};
        passes16<T, LOGN, DIR, 0, V, WAVE>(x, t, active, w);
    }
    if constexpr (WAVE) __syncthreads();
}

}  // namespace rdk
