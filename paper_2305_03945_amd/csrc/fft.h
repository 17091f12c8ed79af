// Workgroup FFTs in LDS and the real-data / cosine-transform wrappers around them.
//
// The preconditioner G is diagonal in the 2-D DFT basis (periodic grids) and in
// the 2-D DCT-II basis (Neumann grids) (Sec. 2.1, "Application of FFT"; Remark 1).
// Both are computed here from complex FFTs of length N:
//
//  * Two real rows a, b are packed as one complex row z = a + i b.  From
//    Z = FFT(z) the two half spectra are A_k = (Z_k + conj Z_{N-k}) / 2 and
//    B_k = (Z_k - conj Z_{N-k}) / (2i).  A row's N/2 + 1 bins are stored as N/2
//    complex slots, slot 0 holding the two real bins (A_0, A_{N/2}).
//  * DCT-II (unnormalised, X_k = sum_n x_n cos(pi k (2n+1) / (2N))) by Makhoul's
//    method: reorder v_n = x_{2n}, v_{N-1-n} = x_{2n+1}, V = FFT(v), then
//    X_k = Re(w_k V_k) and X_{N-k} = -Im(w_k V_k) with w_k = exp(-i pi k / (2N)).
//    The inverse rebuilds V_k = conj(w_k) (X_k - i X_{N-k}) (X_N = 0) and applies
//    an inverse FFT.  Two real sequences are again packed into one complex FFT.
//
// The complex FFTs themselves are in fft16.h (Stockham passes in LDS);
// forward sign -1, both directions unnormalised; the 1/N^2 of the 2-D inverse is
// folded into the symbol multiplier.  This file holds the pair / cosine pre- and
// post-processing over padded LDS regions and the symbol.
#pragma once
#include "rd_dev.h"

namespace rdk {

// LDS regions hold N complex values with a padding slot after every 8 (N <= 64) or 16
// values, which sets a pass's stride-8 or stride-16 writes by neighbouring threads on
// different banks.  The single-workgroup step (N <= 64), which LDS bounds, needs 8: in
// FP64 (16-byte values) 16 leaves two lanes of eight on each bank, a third of its LDS
// cycles.  Above, the step's other LDS accesses make up for it (8: 1-2 % slower).
template <int LOGN> constexpr int pad_shift() { return LOGN <= 6 ? 3 : 4; }
template <int LOGN> __host__ __device__ constexpr int lds_pad(int i) { return i + (i >> pad_shift<LOGN>()); }
// Values from one transform's region to the next.  128 and 256: one more than the
// padded transform (136, 272 values), so that lanes over equal offsets of adjacent
// regions, as the 3-D line passes load and store, spread over the banks (128^3 Neumann
// FP64 step 2.28 -> 2.17 ms; the 2-D steps are within 1 % either way).
template <int LOGN> __host__ __device__ constexpr int lds_region() {
    return lds_pad<LOGN>(1 << LOGN) + (LOGN == 7 || LOGN == 8 ? 1 : 0);
}

template <typename T, int DIR> __device__ __forceinline__ cplx<T> rot90(cplx<T> a) {
    // multiply by exp(DIR i pi / 2): -i for the forward transform, +i for the inverse
    return DIR < 0 ? cplx<T>{a.im, -a.re} : cplx<T>{-a.im, a.re};
}

// Complex element i of region r.
template <int LOGN> __device__ __forceinline__ int rix(int reg, int i) { return reg * lds_region<LOGN>() + lds_pad<LOGN>(i); }

// Real element m (< 2N) of a region viewed as 2N reals (re, im interleaved).
template <typename T, int LOGN> __device__ __forceinline__ T &rreal(cplx<T> *buf, int reg, int m) {
    return reinterpret_cast<T *>(&buf[rix<LOGN>(reg, m >> 1)])[m & 1];
}

// Work items for the pair steps: item (region, l), l < N/2, owns bins l and N-l
// (item 0 owns bins 0 and N/2).
template <int LOGN, int NREG, int NTH> constexpr int pair_items_per_thread() {
    constexpr int total = NREG * ((1 << LOGN) / 2);
    return (total + NTH - 1) / NTH;
}

// ---- row pass, forward: packed pair spectrum Z -> two rows of slots (in place).
// Periodic: slots of row a hold (A_0, A_{N/2}) then A_1..A_{N/2-1}; row b likewise.
// Neumann: the region, viewed as 2N reals, holds X_a[0..N) then X_b[0..N).
template <typename T, int LOGN, int BC, int NREG, int NTH>
__device__ __forceinline__ void rows_post_forward(cplx<T> *buf, const cplx<T> *__restrict__ twd) {
    constexpr int N = 1 << LOGN, H = N / 2;
    constexpr int IPT = pair_items_per_thread<LOGN, NREG, NTH>();
    cplx<T> oa[IPT], ob[IPT];
#pragma unroll
    for (int i = 0; i < IPT; ++i) {
        const int it = threadIdx.x + i * NTH;
        if (it >= NREG * H) break;
        const int reg = it / H, l = it % H;
        if (l == 0) {
            const cplx<T> z0 = buf[rix<LOGN>(reg, 0)], zh = buf[rix<LOGN>(reg, H)];
            if constexpr (BC == BC_P) {
                oa[i] = {z0.re, zh.re};
                ob[i] = {z0.im, zh.im};
            } else {
                const T s = (T)0.707106781186547524400844362104849039;
                oa[i] = {z0.re, s * zh.re};   // X_a[0], X_a[N/2]
                ob[i] = {z0.im, s * zh.im};
            }
        } else {
            const cplx<T> zl = buf[rix<LOGN>(reg, l)], zn = buf[rix<LOGN>(reg, N - l)];
            const cplx<T> A = {(zl.re + zn.re) * (T)0.5, (zl.im - zn.im) * (T)0.5};
            const cplx<T> B = {(zl.im + zn.im) * (T)0.5, (zn.re - zl.re) * (T)0.5};
            if constexpr (BC == BC_P) {
                oa[i] = A;
                ob[i] = B;
            } else {
                const cplx<T> w = twd[l];
                const cplx<T> qa = cmul(A, w), qb = cmul(B, w);
                oa[i] = {qa.re, -qa.im};      // X_a[l], X_a[N-l]
                ob[i] = {qb.re, -qb.im};
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < IPT; ++i) {
        const int it = threadIdx.x + i * NTH;
        if (it >= NREG * H) break;
        const int reg = it / H, l = it % H;
        if constexpr (BC == BC_P) {
            buf[rix<LOGN>(reg, l)] = oa[i];
            buf[rix<LOGN>(reg, H + l)] = ob[i];
        } else {
            if (l == 0) {
                rreal<T, LOGN>(buf, reg, 0) = oa[i].re;
                rreal<T, LOGN>(buf, reg, H) = oa[i].im;
                rreal<T, LOGN>(buf, reg, N) = ob[i].re;
                rreal<T, LOGN>(buf, reg, N + H) = ob[i].im;
            } else {
                rreal<T, LOGN>(buf, reg, l) = oa[i].re;
                rreal<T, LOGN>(buf, reg, N - l) = oa[i].im;
                rreal<T, LOGN>(buf, reg, N + l) = ob[i].re;
                rreal<T, LOGN>(buf, reg, 2 * N - l) = ob[i].im;
            }
        }
    }
    __syncthreads();
}

// ---- row pass, inverse: two rows of slots -> packed pair spectrum Z (in place).
template <typename T, int LOGN, int BC, int NREG, int NTH>
__device__ __forceinline__ void rows_pre_inverse(cplx<T> *buf, const cplx<T> *__restrict__ twd) {
    constexpr int N = 1 << LOGN, H = N / 2;
    constexpr int IPT = pair_items_per_thread<LOGN, NREG, NTH>();
    cplx<T> zl_out[IPT], zn_out[IPT];
#pragma unroll
    for (int i = 0; i < IPT; ++i) {
        const int it = threadIdx.x + i * NTH;
        if (it >= NREG * H) break;
        const int reg = it / H, l = it % H;
        if constexpr (BC == BC_P) {
            const cplx<T> a = buf[rix<LOGN>(reg, l)], b = buf[rix<LOGN>(reg, H + l)];
            if (l == 0) {
                zl_out[i] = {a.re, b.re};   // Z_0 = A_0 + i B_0
                zn_out[i] = {a.im, b.im};   // Z_{N/2}
            } else {
                zl_out[i] = {a.re - b.im, a.im + b.re};
                zn_out[i] = {a.re + b.im, b.re - a.im};
            }
        } else {
            if (l == 0) {
                const T r2 = (T)1.41421356237309504880168872420969808;
                zl_out[i] = {rreal<T, LOGN>(buf, reg, 0), rreal<T, LOGN>(buf, reg, N)};
                zn_out[i] = {r2 * rreal<T, LOGN>(buf, reg, H), r2 * rreal<T, LOGN>(buf, reg, N + H)};
            } else {
                const cplx<T> wc = cconj(twd[l]);
                const cplx<T> va = cmul(wc, cplx<T>{rreal<T, LOGN>(buf, reg, l), -rreal<T, LOGN>(buf, reg, N - l)});
                const cplx<T> vb =
                    cmul(wc, cplx<T>{rreal<T, LOGN>(buf, reg, N + l), -rreal<T, LOGN>(buf, reg, 2 * N - l)});
                zl_out[i] = {va.re - vb.im, va.im + vb.re};
                zn_out[i] = {va.re + vb.im, vb.re - va.im};
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < IPT; ++i) {
        const int it = threadIdx.x + i * NTH;
        if (it >= NREG * H) break;
        const int reg = it / H, l = it % H;
        buf[rix<LOGN>(reg, l)] = zl_out[i];
        buf[rix<LOGN>(reg, l == 0 ? H : N - l)] = zn_out[i];
    }
    __syncthreads();
}

// Symbol multiplier invNd / g, g = (1 + alpha mu + beta mu^2 + gamma mu^3)^2, invNd a power
// of two.  The reciprocal is the hardware's estimate (within 2^-22) and two Newton steps,
// which leave its last rounding: the division's bits, without its scaling.  The fix-up
// is the division's: an overflowing g gives 0, a vanishing one infinity.
__device__ __forceinline__ double symbol_of(double mu, double alpha, double beta, double gamma, double invNd) {
    const double a = 1.0 + mu * (alpha + mu * (beta + gamma * mu));
    const double g = a * a;
    double r = __builtin_amdgcn_rcp(g);
    r = __builtin_fma(__builtin_fma(-g, r, 1.0), r, r);
    r = __builtin_fma(__builtin_fma(-g, r, 1.0), r, r);
    return __builtin_amdgcn_div_fixup(invNd * r, g, invNd);
}

// What a pair item of the symbol pass reads besides its two bins: the eigenvalues
// at its bins l and nl = N - l (l = 0: bins 0 and N/2) and the DCT twiddle w_l.
template <typename T> struct SymPair {
    double el, en;
    cplx<T> w;
};
template <typename T, int LOGN, int BC>
__device__ __forceinline__ SymPair<T> load_sym_pair(const double *__restrict__ eig, const cplx<T> *__restrict__ twd,
                                                    int l) {
    constexpr int N = 1 << LOGN;
    SymPair<T> p;
    p.el = eig[l];
    p.en = eig[l == 0 ? N / 2 : N - l];
    if constexpr (BC == BC_N) p.w = twd[l];
    return p;
}

// The symbol multipliers of a pair item (bins l and nl of a line that holds one complex
// sequence -- plain; eigenvalue ea of the other directions -- or two real ones packed
// as real and imaginary part, ea and eb; Neumann: two cosine sequences).
template <typename T> struct PairMult {
    T al, an, bl, bn;
};
template <typename T, int BC>
__device__ __forceinline__ PairMult<T> pair_mults(int l, bool plain, double ea, double eb, const SymPair<T> &p,
                                                  double al, double be, double ga, double invNd) {
    auto m = [&](double ex, double ey) { return (T)symbol_of(ex + ey, al, be, ga, invNd); };
    PairMult<T> r{};
    r.al = m(ea, p.el);
    if (BC == BC_N || plain || l == 0) r.an = m(ea, p.en);
    if (BC == BC_N || !plain) {
        r.bl = m(eb, p.el);
        if (BC == BC_N || l == 0) r.bn = m(eb, p.en);
    }
    return r;
}

// Multiply the item's bins.  w: the DCT twiddle w_l (Neumann).
template <typename T, int BC>
__device__ __forceinline__ void apply_pair(cplx<T> &zlr, cplx<T> &znr, int l, bool plain, const PairMult<T> &m,
                                           cplx<T> w) {
    const cplx<T> zl = zlr, zn = znr;
    if (BC == BC_P && plain) {
        zlr = {zl.re * m.al, zl.im * m.al};
        znr = {zn.re * m.an, zn.im * m.an};
    } else if (l == 0) {
        // bins 0 and N/2 of two real sequences: real pairs
        zlr = {zl.re * m.al, zl.im * m.bl};
        znr = {zn.re * m.an, zn.im * m.bn};
    } else {
        cplx<T> A = {(zl.re + zn.re) * (T)0.5, (zl.im - zn.im) * (T)0.5};
        cplx<T> B = {(zl.im + zn.im) * (T)0.5, (zn.re - zl.re) * (T)0.5};
        if constexpr (BC == BC_P) {
            A = {A.re * m.al, A.im * m.al};
            B = {B.re * m.bl, B.im * m.bl};
            zlr = {A.re - B.im, A.im + B.re};
            znr = {A.re + B.im, B.re - A.im};
        } else {
            const cplx<T> qa = cmul(A, w), qb = cmul(B, w);
            // cosine coefficients at l and N-l, scaled by their symbols
            const T xal = qa.re * m.al, xan = -qa.im * m.an;
            const T xbl = qb.re * m.bl, xbn = -qb.im * m.bn;
            const cplx<T> wc = cconj(w);
            const cplx<T> va = cmul(wc, cplx<T>{xal, -xan});
            const cplx<T> vb = cmul(wc, cplx<T>{xbl, -xbn});
            zlr = {va.re - vb.im, va.im + vb.re};
            znr = {va.re + vb.im, vb.re - va.im};
        }
    }
}

template <typename T, int BC>
__device__ __forceinline__ void apply_symbol_pair(cplx<T> &zl, cplx<T> &zn, int l, bool plain, double ea, double eb,
                                                  const SymPair<T> &p, double al, double be, double ga, double invNd) {
    apply_pair<T, BC>(zl, zn, l, plain, pair_mults<T, BC>(l, plain, ea, eb, p, al, be, ga, invNd), p.w);
}

// ---- column pass, between the forward and inverse column FFTs: multiply by the
// symbol.  Region `reg` holds column job (component c, column j) with
// c = job / H, j = job % H.  Periodic: column j is the row spectrum at kx = j;
// column 0 packs kx = 0 (real part) and kx = N/2 (imaginary part).  Neumann:
// column j packs kx = 2j (real) and kx = 2j + 1 (imaginary), both cosine
// coefficients.  Each item rewrites its own two bins, so no barrier is needed
// between reading and writing.  pre: the items' SymPairs, loaded ahead (nullptr:
// loaded here).
template <typename T, int LOGN, int BC, int NREG, int NTH>
__device__ __forceinline__ void cols_apply_symbol(cplx<T> *buf, int job0, int njobs, SlotRef s,
                                                  const cplx<T> *__restrict__ twd, const SymPair<T> *pre) {
    constexpr int N = 1 << LOGN, H = N / 2;
    constexpr int IPT = pair_items_per_thread<LOGN, NREG, NTH>();
    const double invN2 = 1.0 / ((double)N * (double)N);
    // FP32: not unrolled, which keeps the FP32 column pass within 128 registers
    // (no spills) so that two of its workgroups fit on a compute unit
    constexpr int UNR = sizeof(T) == 4 && IPT > 4 ? 1 : IPT;
#pragma unroll UNR
    for (int i = 0; i < IPT; ++i) {
        const int it = threadIdx.x + i * NTH;
        if (it >= NREG * H) break;
        const int reg = it / H, l = it % H;
        if (reg >= njobs) continue;
        const int job = job0 + reg;
        const int c = job / H, j = job % H;
        const double al = s.alpha[c], be = s.beta[c], ga = s.gamma[c];
        const int nl = (l == 0) ? H : N - l;
        const SymPair<T> p = pre ? pre[i] : load_sym_pair<T, LOGN, BC>(s.eig, twd, l);
        const int ka = BC == BC_P ? j : 2 * j, kb = BC == BC_P ? H : 2 * j + 1;
        apply_symbol_pair<T, BC>(buf[rix<LOGN>(reg, l)], buf[rix<LOGN>(reg, nl)], l, j > 0, s.eig[ka], s.eig[kb], p,
                                 al, be, ga, invN2);
    }
    __syncthreads();
}

}  // namespace rdk
