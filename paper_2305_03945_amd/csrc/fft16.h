// Workgroup FFT, V = 4, 8 or 16 values per thread.
//
// A length-N transform (N = 2^LOGN, 16 <= N <= 4096) is done by N/V threads, in an
// LDS region of N complex values with padding (lds_pad), which keeps the stride-R
// writes of a Stockham pass off a single bank group.  Threads of one wave synchronise
// within it, a transform over several waves by the workgroup's barrier.  Passes are
// Stockham autosort passes of radix V, then one pass of a smaller radix for the
// remaining bits; each thread runs V/R butterflies of a radix-R pass.  A butterfly gathers the powers W^{k}, W^{2k}, W^{4k}, W^{8k}
// of its twiddle and applies them in its radix-2 steps (twiddled_dft).
#pragma once
#include "fft.h"

namespace rdk {

// ---- twiddled DFT of one butterfly, in multiply-adds
//
// V_q = sum_r v_r w^r W_R^{qr}, W_R = exp(DIR 2 pi i / R), by radix-2 steps on the
// even and odd inputs: with E, O the DFTs (of R/2 points, for w^2) of the two halves
// and t = w W_R^q,
//     V_q = E_q + t O_q,   V_{q+R/2} = 2 E_q - V_q:
// six multiply-adds for a complex butterfly and its twiddle together.  Only w, w^2,
// w^4, ... are needed (one per step); t for q >= R/4 is t for q - R/4 turned by 90
// degrees.  A radix-16 butterfly takes 208 operations, against 272 when its 15
// twiddles are formed and applied first.
template <typename T> __device__ __forceinline__ T fma_(T a, T b, T c) { return __builtin_elementwise_fma(a, b, c); }

// cos and sin of 2 pi m / R for R = 16 (m = 1..3) and R = 8 (m = 1)
template <typename T, int R, int M> __device__ __forceinline__ cplx<T> root_of_one() {
    static_assert((R == 16 && M >= 1 && M <= 3) || (R == 8 && M == 1), "first-octant roots");
    constexpr int m = M * 16 / R;
    if constexpr (m == 1) return {(T)0.923879532511286756128183189396788934, (T)0.382683432365089771728459984030398867};
    else if constexpr (m == 2) return {(T)0.707106781186547524400844362104849039, (T)0.707106781186547524400844362104849039};
    else return {(T)0.382683432365089771728459984030398867, (T)0.923879532511286756128183189396788934};
}

// the butterfly: lo = a + t b, hi = a - t b.  QUARTER: t is to be turned by DIR 90
// degrees.  ONE: t = 1.
template <typename T, int DIR, bool ONE, bool QUARTER>
__device__ __forceinline__ void bfly(cplx<T> a, cplx<T> b, cplx<T> t, cplx<T> &lo, cplx<T> &hi) {
    if constexpr (ONE) {
        const cplx<T> c = QUARTER ? rot90<T, DIR>(b) : b;
        lo = cadd(a, c);
        hi = csub(a, c);
    } else {
        if constexpr (QUARTER) b = rot90<T, DIR>(b);
        lo.re = fma_(-t.im, b.im, fma_(t.re, b.re, a.re));
        lo.im = fma_(t.im, b.re, fma_(t.re, b.im, a.im));
        hi.re = fma_((T)2, a.re, -lo.re);
        hi.im = fma_((T)2, a.im, -lo.im);
    }
}

// t_q = w W_R^q for 0 <= q < max(1, R/4)
template <typename T, int R, int DIR, bool TW, int Q = 0> __device__ __forceinline__ void step_twiddles(cplx<T> w, cplx<T> *t) {
    if constexpr (Q < (R >= 8 ? R / 4 : 1)) {
        if constexpr (Q == 0) {
            t[0] = w;
        } else {
            cplx<T> c = root_of_one<T, R, Q>();
            c.im *= (T)DIR;
            t[Q] = TW ? cmul(w, c) : c;
        }
        step_twiddles<T, R, DIR, TW, Q + 1>(w, t);
    }
}

// The twiddles of every step of a radix-R butterfly: steps of 16, 8, 4, 2 points.
template <typename T, int R, int DIR, bool TW> struct StepTw {
    cplx<T> t[R >= 8 ? R / 4 : 1];
    StepTw<T, R / 2, DIR, TW> next;
    __device__ __forceinline__ void set(const cplx<T> *p) {
        step_twiddles<T, R, DIR, TW>(TW ? p[0] : cplx<T>{(T)1, (T)0}, t);
        next.set(p + 1);
    }
};
template <typename T, int DIR, bool TW> struct StepTw<T, 1, DIR, TW> {
    __device__ __forceinline__ void set(const cplx<T> *) {}
};

// in: R inputs at stride S; out: R outputs in natural order.
template <typename T, int R, int DIR, bool TW, int S>
__device__ __forceinline__ void dit(const cplx<T> *in, cplx<T> *out, const StepTw<T, R, DIR, TW> &w) {
    if constexpr (R == 1) {
        out[0] = in[0];
    } else {
        cplx<T> e[R / 2], o[R / 2];
        dit<T, R / 2, DIR, TW, 2 * S>(in, e, w.next);
        dit<T, R / 2, DIR, TW, 2 * S>(in + S, o, w.next);
        constexpr int QT = R >= 4 ? R / 4 : 1;   // q >= QT: turned by 90 degrees
#pragma unroll
        for (int q = 0; q < QT; ++q) {
            if constexpr (!TW) {
                if (q == 0) bfly<T, DIR, true, false>(e[0], o[0], w.t[0], out[0], out[R / 2]);
                else bfly<T, DIR, false, false>(e[q], o[q], w.t[q], out[q], out[q + R / 2]);
            } else {
                bfly<T, DIR, false, false>(e[q], o[q], w.t[q], out[q], out[q + R / 2]);
            }
        }
        if constexpr (R >= 4) {
#pragma unroll
            for (int q = 0; q < QT; ++q) {
                if constexpr (!TW) {
                    if (q == 0) bfly<T, DIR, true, true>(e[QT], o[QT], w.t[0], out[QT], out[QT + R / 2]);
                    else bfly<T, DIR, false, true>(e[q + QT], o[q + QT], w.t[q], out[q + QT], out[q + QT + R / 2]);
                } else {
                    bfly<T, DIR, false, true>(e[q + QT], o[q + QT], w.t[q], out[q + QT], out[q + QT + R / 2]);
                }
            }
        }
    }
}

// DFT_R of v in place, input r multiplied by w^r first; p: w, w^2, w^4, ... (forward
// sign, conjugated here for the inverse).
template <typename T, int R, int DIR> __device__ __forceinline__ void twiddled_dft(cplx<T> *v, const cplx<T> *p) {
    cplx<T> pd[4];
#pragma unroll
    for (int e = 0; e < 4; ++e)
        if ((1 << e) < R) pd[e] = DIR > 0 ? cconj(p[e]) : p[e];
    // step sizes R, R/2, ..., 2 take w, w^2, ...
    StepTw<T, R, DIR, true> w;
    w.set(pd);
    cplx<T> out[R];
    dit<T, R, DIR, true, 1>(v, out, w);
#pragma unroll
    for (int q = 0; q < R; ++q) v[q] = out[q];
}

// DFT_R of v in place.
template <typename T, int R, int DIR> __device__ __forceinline__ void dftR(cplx<T> *v) {
    StepTw<T, R, DIR, false> w;
    w.set(nullptr);
    cplx<T> out[R];
    dit<T, R, DIR, false, 1>(v, out, w);
#pragma unroll
    for (int q = 0; q < R; ++q) v[q] = out[q];
}

// Values per thread of a transform, V: 16 where the chip is full of transforms, 8 or 4
// where it is not (short serial chains; see RowsPlan and col_values).  Radix of pass q of a
// length-2^LOGN transform: radix V while that many bits remain, then one pass of
// what is left.
template <int V> constexpr int logv() { return V == 16 ? 4 : V == 8 ? 3 : 2; }
template <int LOGN, int V = 16> constexpr int npasses16() { return (LOGN + logv<V>() - 1) / logv<V>(); }
template <int LOGN, int V = 16> constexpr int pass_radix(int q) {
    return LOGN - logv<V>() * q >= logv<V>() ? V : (1 << (LOGN - logv<V>() * q));
}

// The twiddles of one thread for every pass after the first: for butterfly b of
// pass q, the gathered powers W^{k}, W^{2k}, W^{4k}, W^{8k} (forward sign) of
// W = exp(-2 pi i / (NS R)), k = j mod NS.  They depend only on the thread's
// index in its transform team, so a kernel loads them once, at its start, and
// every transform (forward and inverse) of the kernel reuses them.
template <typename T, int LOGN, int V = 16> struct Tw16 {
    cplx<T> p[npasses16<LOGN, V>() > 1 ? npasses16<LOGN, V>() - 1 : 1][V / 2][logv<V>()];
};

template <typename T, int LOGN, int V>
__device__ __forceinline__ void load_tw16(Tw16<T, LOGN, V> &w, const cplx<T> *__restrict__ tw, int t) {
    constexpr int N = 1 << LOGN;
    constexpr int TPF = N / V;
    const auto tg = gp(tw);
#pragma unroll
    for (int q = 1; q < npasses16<LOGN, V>(); ++q) {
        const int R = pass_radix<LOGN, V>(q), NS = 1 << (logv<V>() * q);
        const int TWSTEP = N / (NS * R);
#pragma unroll
        for (int b = 0; b < V / R; ++b) {
            const int k = (t + b * TPF) & (NS - 1);
#pragma unroll
            for (int e = 0; e < logv<V>(); ++e)
                if ((1 << e) < R) {
                    const int i = ((k * TWSTEP) << e) & (N - 1);
                    w.p[q - 1][b][e] = {tg[i].re, tg[i].im};
                }
        }
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
__device__ __forceinline__ void pass_in(X x, int t, const cplx<T> (*pw)[logv<V>()], cplx<T> (*v)[R]) {
    constexpr int N = 1 << LOGN;
    constexpr int TPF = N / V;       // threads per transform
    constexpr int NB = N / R;        // butterflies
    constexpr int BPT = V / R;       // butterflies per thread
#pragma unroll
    for (int b = 0; b < BPT; ++b) {
        const int j = t + b * TPF;
#pragma unroll
        for (int r = 0; r < R; ++r) v[b][r] = x(j + r * NB);
        if constexpr (NS > 1) twiddled_dft<T, R, DIR>(v[b], pw[b]);
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
__device__ __forceinline__ void pass16(X x, int t, bool active, const cplx<T> (*pw)[logv<V>()]) {
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
