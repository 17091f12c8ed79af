// Small grids: one workgroup runs a whole implicit step.
//
// On N <= 64 grids an iteration moves a few hundred KB, and the launches of the
// batched iteration (column pass, row pass) cost their latency, not their bytes.  Here one workgroup per slot takes
// the whole step, Algorithm 1 with its stop test, in one launch:
//
//   W = F(U_n) (stencil);  Z = Q + (1 + omega) W -> spectrum S in LDS (row pairs
//   packed as complex rows);  Q += W (registers; the sums of kernels_rows.h)
//   ||W / h_t|| (fixed-order workgroup sum), stop decision (decide<>, thread 0)
//   row FFTs, column FFTs (on the row layout), 1 / (N^2 g), inverse column
//   FFTs, inverse row FFTs                          -> P~ = tau_p G^-1 Z in LDS
//   U_{n+1} = U_n - tau_u grad F(U_n)^T P~
//
// and, in the mixed precision, the same FP32 inner loop on the correction e with
// the FP64 outer passes (U += e, r = F(U), stop test) between inner loops.  The
// spectrum always lives in LDS; the iterate and (mixed) the FP32 copy of U take
// LDS in that order while the 160 KB of a gfx950 workgroup allow, and otherwise stay
// in the slot's HBM buffers (then L2-resident).  What a thread alone reads, Q, U^k (FP64)
// or r (mixed) at its own points and its symbol multipliers, stays in registers for
// the whole step: LDS, not arithmetic, bounds this kernel.  The arithmetic
// per point is that of the batched kernels (the same eval_F / eval_Ftilde /
// eval_adjoint code, the pair / cosine processing and symbol of fft.h); the
// transforms are radix-8 passes and the norm's sums run in another order.
#pragma once
#include "kernels.h"

namespace rdk {

constexpr int NT7 = 512;                // threads of a step workgroup
constexpr size_t WG_LDS_BYTES = 163840; // LDS of one gfx950 workgroup

// Which fields of a step fit in LDS beside the spectrum.
template <typename T, int LOGN, int C> struct WgPlan {
    static constexpr int N = 1 << LOGN;
    static constexpr size_t NN = (size_t)N * N;
    static constexpr size_t spec = (size_t)C * (N / 2) * lds_region<LOGN>() * sizeof(cplx<T>);
    static constexpr size_t fixed = 4096;                      // sums, State, tables
    static constexpr size_t fieldT = (size_t)C * NN * sizeof(T);
    static constexpr size_t field32 = (size_t)C * NN * sizeof(float);
    static constexpr size_t room = WG_LDS_BYTES - fixed;
    static constexpr bool ok = spec <= room;
    static constexpr bool u_lds = ok && spec + fieldT <= room;
    static constexpr bool ub_lds = sizeof(T) == 4 && u_lds && spec + fieldT + field32 <= room;
    static constexpr size_t bytes = spec + (u_lds ? fieldT : 0) + (ub_lds ? field32 : 0);
};

// Whether the single-workgroup step serves (T, N, equation): N <= 64, the
// spectrum fits, and an adjoint that reads U only at its own point (the
// update is made in place), which excludes the sixth-order equation.  (At 128^2
// the fields leave LDS for L2 and the kernel runs out of registers; there the
// batched kernels are faster.)
constexpr int WG_MAX_LOGN = 6;
template <typename T, int LOGN, int EQ> constexpr bool wg_step_available() {
    return LOGN <= WG_MAX_LOGN && EQ != EQ_FCH && WgPlan<T, LOGN, EQ == EQ_SCHNAK ? 2 : 1>::ok;
}

// ---------------------------------------------------------------- column transforms in place
// The column transforms run on the spectrum where the row pass left it (row pairs
// packed per LDS region): element i of column job reg (component c = reg / H,
// column kx = reg % H) is row y of that column, y = i on periodic grids and the
// row whose Makhoul position is i on Neumann grids, at slot (y & 1) H + kx of
// region c H + y / 2.  The transforms below take an address map, so no transpose
// is needed between the row and the column transforms.
template <int LOGN, int BC> struct ColMap {
    static constexpr int N = 1 << LOGN, H = N / 2;
    static constexpr bool COLUMNS = true;
    __device__ __forceinline__ static int row_of(int i) {
        if (BC == BC_P) return i;
        return i < H ? 2 * i : 2 * (N - 1 - i) + 1;   // inverse of dct_pos
    }
    __device__ __forceinline__ static int at(int reg, int i) {
        const int c = reg / H, kx = reg % H, y = row_of(i);
        return rix<LOGN>(c * H + (y >> 1), (y & 1) * H + kx);
    }
};

// ---------------------------------------------------------------- radix-8 transforms
// The single-workgroup step's transforms (N <= 64): Stockham passes of radix 8 while
// three bits remain, then one of radix 4 or 2, with 8 values per thread (N/8 threads
// per transform: twice the threads of the radix-16 passes on these short
// transforms, whose passes are bound by arithmetic latency, not LDS).  Pass q reads
// element j + r N/R of butterfly j, multiplies input r by W_{NS R}^{r k} (k = j mod
// NS), applies DFT_R and writes output q to (j - k) R + k + q NS.  The twiddles of a
// thread depend only on its index in its team, so they are read from the table
// exp(-2 pi i m / N) once per step and kept in registers; the inverse conjugates.  FP64
// butterflies are those of fft16.h; FP32 ones multiply all R - 1 twiddles in first, whose
// rounding error is the smaller there (64 points, in units of the rounding: 1.33; 1.41 by
// radix-2 steps) and for whose registers the FP32 step has room.
template <int LOGN> constexpr int r8_radix(int q) { return LOGN - 3 * q >= 3 ? 8 : (1 << (LOGN - 3 * q)); }
template <int LOGN> constexpr int r8_passes() { return (LOGN + 2) / 3; }

template <typename T, int LOGN> struct TwR8 {
    // pass 1 (the only pass with NS > 1 for N <= 64): butterflies b < 8 / R, powers
    // FP64: gather_twiddles; FP32: the twiddles of inputs 1 .. R - 1
    cplx<T> w[4][sizeof(T) == 8 ? tw_count<LOGN, 8>() : 7];
};

template <typename T, int LOGN>
__device__ __forceinline__ void load_twr8(TwR8<T, LOGN> &tw, const cplx<T> *table, int t) {
    static_assert(r8_passes<LOGN>() <= 2, "radix-8 step transforms: N <= 64");
    constexpr int N = 1 << LOGN, TPT = N / 8;
    if constexpr (r8_passes<LOGN>() == 2) {
        constexpr int R = r8_radix<LOGN>(1), NS = 8, NB = N / R, BPT = 8 / R;
        constexpr int STEP = N / (NS * R);
#pragma unroll
        for (int b = 0; b < BPT; ++b) {
            const int j = t + b * TPT;
            const int k = j & (NS - 1);
            (void)NB;
            if constexpr (sizeof(T) == 8) {
                gather_twiddles<T, LOGN, 8, R>(tw.w[b], table, k * STEP);
            } else {
#pragma unroll
                for (int r = 1; r < R; ++r) tw.w[b][r - 1] = table[(r * k * STEP) & (N - 1)];
            }
        }
    }
}

template <typename T, int LOGN, int Q, int DIR, class M>
__device__ __forceinline__ void r8_pass(cplx<T> *buf, int reg, int t, bool active, const TwR8<T, LOGN> &tw) {
    constexpr int N = 1 << LOGN, TPT = N / 8;
    constexpr int R = r8_radix<LOGN>(Q), NS = Q == 0 ? 1 : 8, NB = N / R, BPT = 8 / R;
    cplx<T> v[BPT][R];
    if (active) {
#pragma unroll
        for (int b = 0; b < BPT; ++b) {
            const int j = t + b * TPT;
#pragma unroll
            for (int r = 0; r < R; ++r) v[b][r] = buf[M::at(reg, j + r * NB)];
            if constexpr (NS > 1 && sizeof(T) == 8) {
                twiddled_dft<T, LOGN, 8, R, DIR>(v[b], tw.w[b]);
            } else {
                if constexpr (NS > 1) {
#pragma unroll
                    for (int r = 1; r < R; ++r)
                        v[b][r] = cmul(v[b][r], DIR < 0 ? tw.w[b][r - 1] : cconj(tw.w[b][r - 1]));
                }
                dftR<T, R, DIR>(v[b]);
            }
        }
    }
    pass_sync<true>();
    if (active) {
#pragma unroll
        for (int b = 0; b < BPT; ++b) {
            const int j = t + b * TPT;
            const int k = j & (NS - 1);
            const int base = (j - k) * R + k;
#pragma unroll
            for (int q = 0; q < R; ++q) buf[M::at(reg, base + q * NS)] = v[b][q];
        }
    }
    pass_sync<true>();
}

// In-place transforms of NREG regions (address map M) by NTH threads; teams of N/8
// threads, each within one wave, take regions round-robin.  Rows: a team is N/8
// consecutive lanes, whose reads are contiguous.  Columns: consecutive lanes take
// consecutive columns, which are contiguous in LDS at every row (a team's own rows are
// region strides apart).  Ends with a barrier.
template <typename T, int LOGN, int DIR, int NREG, int NTH, class M>
__device__ __forceinline__ void wg_fft_r8(cplx<T> *buf, const TwR8<T, LOGN> &tw) {
    constexpr int TPT = (1 << LOGN) / 8, TPW = 64 / TPT;
    constexpr int NTEAMS = NTH / TPT;
    const int lane = threadIdx.x & 63;
    const int t = M::COLUMNS ? lane / TPW : lane % TPT;
    const int team = (threadIdx.x >> 6) * TPW + (M::COLUMNS ? lane % TPW : lane / TPT);
#pragma unroll 1
    for (int g = 0; g < NREG; g += NTEAMS) {
        const int reg = g + team;
        const bool active = reg < NREG;
        r8_pass<T, LOGN, 0, DIR, M>(buf, active ? reg : 0, t, active, tw);
        if constexpr (r8_passes<LOGN>() == 2) r8_pass<T, LOGN, 1, DIR, M>(buf, active ? reg : 0, t, active, tw);
    }
    __syncthreads();
}

template <int LOGN> struct RowMap {
    static constexpr bool COLUMNS = false;
    __device__ __forceinline__ static int at(int reg, int i) { return rix<LOGN>(reg, i); }
};

// 1 / (N^2 g) on the transformed columns (cols_apply_symbol of fft.h on the
// mapped layout): column job reg of component c = reg / H is kx = reg % H
// (periodic; column 0 packs kx = 0 and kx = N/2) or the cosine pair kx = 2j, 2j + 1
// (Neumann).  Item i of a thread is the pair (reg, l); eight neighbouring lanes take
// eight neighbouring columns, which are contiguous in LDS.  The multipliers depend on
// the step only, so a thread forms them once (load_wg_symbol).
template <int LOGN> __device__ __forceinline__ void wg_symbol_item(int it, int &reg, int &l) {
    constexpr int H = (1 << LOGN) / 2;
    reg = (it & 7) + 8 * (it / (8 * H));
    l = (it >> 3) % H;
}
template <int NREG, int LOGN> constexpr int wg_symbol_items() { return (NREG * (1 << LOGN) / 2 + NT7 - 1) / NT7; }

template <typename T, int LOGN, int BC, int NREG>
__device__ __forceinline__ void load_wg_symbol(PairMult<T> *m, SlotRef s) {
    constexpr int N = 1 << LOGN, H = N / 2;
    const double invN2 = 1.0 / ((double)N * (double)N);
#pragma unroll
    for (int i = 0; i < wg_symbol_items<NREG, LOGN>(); ++i) {
        int reg, l;
        wg_symbol_item<LOGN>(threadIdx.x + i * NT7, reg, l);
        if (reg >= NREG) break;
        const int c = reg / H, j = reg % H;
        const int ka = BC == BC_P ? j : 2 * j, kb = BC == BC_P ? H : 2 * j + 1;
        const SymPair<T> p{s.eig[l], s.eig[l == 0 ? H : N - l], {}};
        m[i] = pair_mults<T, BC>(l, j > 0, s.eig[ka], s.eig[kb], p, s.alpha[c], s.beta[c], s.gamma[c], invN2);
    }
}

template <typename T, int LOGN, int BC, int NREG, class M>
__device__ __forceinline__ void cols_symbol_mapped(cplx<T> *buf, const PairMult<T> *m, const cplx<T> *twd) {
    constexpr int N = 1 << LOGN, H = N / 2;
#pragma unroll
    for (int i = 0; i < wg_symbol_items<NREG, LOGN>(); ++i) {
        int reg, l;
        wg_symbol_item<LOGN>(threadIdx.x + i * NT7, reg, l);
        if (reg >= NREG) break;
        apply_pair<T, BC>(buf[M::at(reg, l)], buf[M::at(reg, l == 0 ? H : N - l)], l, reg % H > 0, m[i],
                          BC == BC_N ? twd[l] : cplx<T>{});
    }
    __syncthreads();
}

// Strips: in the point phases thread t takes rows y0 .. y0 + L - 1 of column
// x = t mod N (L = N^2 / NT7, at least 1), in sub-strips of LS rows whose stencil
// neighbourhood (reach HY, the diamond |dy| + |dx| <= HY: 5 or 13 points) it loads
// into registers once.  The rows of a sub-strip pair up (2q, 2q + 1), the two rows
// a complex slot of the spectrum packs, so W and Y move as one complex value.
template <int LOGN> constexpr int wg_strip() { return (1 << (2 * LOGN)) >= NT7 ? (1 << (2 * LOGN)) / NT7 : 1; }
template <int LOGN, int HY, int C> constexpr int wg_substrip() {
    constexpr int L = wg_strip<LOGN>();
    constexpr int cap = (HY >= 2 || C == 2) ? 2 : 8;   // windows within the register budget
    return L < cap ? L : cap;
}
// Whether window row r (-HY .. LS - 1 + HY) at column offset dx is in the
// neighbourhood of some row of a sub-strip of LS rows.
template <int HY, int LS> __host__ __device__ constexpr bool wg_needed(int r, int dx) {
    const int dist = r < 0 ? -r : (r >= LS ? r - LS + 1 : 0);
    return dist + (dx < 0 ? -dx : dx) <= HY;
}

template <typename T, int LOGN, int BC, int EQ, int MODE>
__global__ __launch_bounds__(NT7) void k_step_wg(Slot *const *slots) {
    constexpr int C = EQ == EQ_SCHNAK ? 2 : 1;
    constexpr int N = 1 << LOGN, H = N / 2;
    constexpr int NN = N * N;
    constexpr int NREG = C * H;   // row-pair regions = column regions
    constexpr int HY = stencil_hy<EQ>();
    constexpr int HU = EQ == EQ_BIH ? 1 : 0;   // reach of U in the mixed inner residual
    using Plan = WgPlan<T, LOGN, C>;
    static_assert(Plan::ok, "the spectrum must fit in LDS");
    static_assert(MODE == MODE_F64 ? sizeof(T) == 8 : sizeof(T) == 4, "FP64 step or FP32 inner loop");
    __shared__ __align__(16) unsigned char lds[Plan::bytes];
    __shared__ double red[2 * C * (NT7 / 64)];
    __shared__ State stl;
    __shared__ cplx<T> twd_l[N];       // the DCT twiddles, staged once rather than fetched from L2

    SlotRef s = slot_of(slots);
    const int tid = threadIdx.x;
    cplx<T> *S = (cplx<T> *)lds;
    unsigned char *nxt = lds + Plan::spec;
    // iterate: FP64 U, or the mixed path's correction e
    T *U = Plan::u_lds ? (T *)nxt : (T *)s.U[0];
    nxt += Plan::u_lds ? Plan::fieldT : 0;
    float *Ub = Plan::ub_lds ? (float *)nxt : s.Ub32;
    const double *src = s.src;     // U^k: the caller's input, read-only for the whole step
    double *U64 = s.U64[0];        // mixed: FP64 U (never bound to the caller's input)
    TwR8<T, LOGN> twr, twc;   // of this thread's place in a row team, and in a column team
    load_twr8<T, LOGN>(twr, (const cplx<T> *)s.tw, (threadIdx.x & 63) % (N / 8));
    load_twr8<T, LOGN>(twc, (const cplx<T> *)s.tw, (threadIdx.x & 63) / (64 / (N / 8)));
    const StopRule rule{s.tol, s.inner_rtol, s.max_iter, s.max_outer};
    auto pos = [](int x) { return BC == BC_P ? x : dct_pos(x, N); };
    auto at = [](int c, int y, int x) { return c * NN + wrap<BC>(y, N) * N + wrap<BC>(x, N); };
    constexpr int L = wg_strip<LOGN>();
    constexpr int LS = wg_substrip<LOGN, HY, C>();
    constexpr int STRIP_THREADS = N * (N / L);
    static_assert(L % LS == 0 && (LS == 1 || LS % 2 == 0), "sub-strips of whole row pairs");
    // W of rows ys .. ys + LS - 1 at column x into the spectrum's row-pair layout
    auto store_w = [&](int c, int ys, int x, const double *W) {
        if constexpr (LS >= 2) {
#pragma unroll
            for (int q = 0; q < LS / 2; ++q)
                S[rix<LOGN>(c * H + (ys >> 1) + q, pos(x))] = cplx<T>{(T)W[2 * q], (T)W[2 * q + 1]};
        } else {
            rreal<T, LOGN>(S, c * H + ys / 2, 2 * pos(x) + (ys & 1)) = (T)W[0];
        }
    };
    if (tid == 0) stl = State{};
    for (int i = tid; i < N; i += NT7) twd_l[i] = ((const cplx<T> *)s.twd)[i];
    const cplx<T> *twd = twd_l;
    PairMult<T> sym[wg_symbol_items<NREG, LOGN>()];
    load_wg_symbol<T, LOGN, BC, NREG>(sym, s);
    // at this thread's strip: Q, and U^k (FP64) or the outer residual r (mixed)
    T q[C][L], own[C][L];
    const T om1 = (T)1 + (T)s.omega;
    if constexpr (MODE == MODE_F64) {
        if (tid < STRIP_THREADS) {
#pragma unroll
            for (int c = 0; c < C; ++c)
#pragma unroll
                for (int i = 0; i < L; ++i) own[c][i] = src[c * NN + ((tid / N) * L + i) * N + tid % N];
        }
    }

    // ---- the residual of an FP64 state (U_0, or the mixed outer U) into S; its
    // norm and sum(U - U^k) decided by thread 0
    // (start: an initial or outer pass, which begins an iteration loop: S = W, Q = W)
    auto residual64 = [&](const double *Uf, bool start, auto decide_fn) {
        double acc[2 * C];
#pragma unroll
        for (int k = 0; k < 2 * C; ++k) acc[k] = 0.0;
        if (tid < STRIP_THREADS) {
            const int x = tid % N, y0 = (tid / N) * L;
#pragma unroll
            for (int s0 = 0; s0 < L; s0 += LS) {
                const int ys = y0 + s0;
                double v[C][LS + 2 * HY][2 * HY + 1], uk[C][LS];
#pragma unroll
                for (int c = 0; c < C; ++c) {
#pragma unroll
                    for (int r = -HY; r < LS + HY; ++r)
#pragma unroll
                        for (int dx = -HY; dx <= HY; ++dx)
                            if (wg_needed<HY, LS>(r, dx)) v[c][r + HY][dx + HY] = Uf[at(c, ys + r, x + dx)];
#pragma unroll
                    for (int i = 0; i < LS; ++i)
                        uk[c][i] = MODE == MODE_F64 ? (double)own[c][s0 + i] : src[c * NN + (ys + i) * N + x];
                }
                double W[C][LS];
#pragma unroll
                for (int i = 0; i < LS; ++i) {
                    double Wi[C], Uc[C], ukc[C];
#pragma unroll
                    for (int c = 0; c < C; ++c) ukc[c] = uk[c][i];
                    eval_F<EQ, double>(s, [&](int c, int dy, int dx) { return v[c][i + dy + HY][dx + HY]; }, ukc, Wi,
                                       Uc);
#pragma unroll
                    for (int c = 0; c < C; ++c) {
                        acc[c] += Wi[c] * Wi[c];
                        acc[C + c] += Uc[c] - ukc[c];
                        if (start) {
                            q[c][s0 + i] = (T)Wi[c];
                            W[c][i] = Wi[c];
                        } else {
                            W[c][i] = q[c][s0 + i] + om1 * (T)Wi[c];
                            q[c][s0 + i] += (T)Wi[c];
                        }
                        if constexpr (MODE == MODE_MIXED) {
                            own[c][s0 + i] = (T)Wi[c];
                            Ub[c * NN + (ys + i) * N + x] = (float)Uc[c];
                        }
                    }
                }
#pragma unroll
                for (int c = 0; c < C; ++c) store_w(c, ys, x, W[c]);
            }
        }
        block_sum<2 * C, NT7>(acc, red);
        if (tid == 0) {
            double res = 0.0, m = 0.0;
#pragma unroll
            for (int c = 0; c < C; ++c) {
                res += sqrt(acc[c]);
                m += acc[C + c];
            }
            decide_fn(res / s.ht, m);
        }
        __syncthreads();
    };

    // ---- the mixed inner residual F~(e) into S; its norm decided by thread 0
    auto residual32 = [&]() {
        double acc[C];
#pragma unroll
        for (int c = 0; c < C; ++c) acc[c] = 0.0;
        if (tid < STRIP_THREADS) {
            const int x = tid % N, y0 = (tid / N) * L;
#pragma unroll
            for (int s0 = 0; s0 < L; s0 += LS) {
                const int ys = y0 + s0;
                float ve[C][LS + 2 * HY][2 * HY + 1], vu[C][LS + 2 * HU][2 * HU + 1];
#pragma unroll
                for (int c = 0; c < C; ++c) {
#pragma unroll
                    for (int r = -HY; r < LS + HY; ++r)
#pragma unroll
                        for (int dx = -HY; dx <= HY; ++dx)
                            if (wg_needed<HY, LS>(r, dx)) ve[c][r + HY][dx + HY] = (float)U[at(c, ys + r, x + dx)];
#pragma unroll
                    for (int r = -HU; r < LS + HU; ++r)
#pragma unroll
                        for (int dx = -HU; dx <= HU; ++dx)
                            if (wg_needed<HU, LS>(r, dx)) vu[c][r + HU][dx + HU] = Ub[at(c, ys + r, x + dx)];
                }
                double W[C][LS];
#pragma unroll
                for (int i = 0; i < LS; ++i) {
                    float Wi[C], r[C];
#pragma unroll
                    for (int c = 0; c < C; ++c) r[c] = (float)own[c][s0 + i];
                    eval_Ftilde<EQ>(s, [&](int c, int dy, int dx) { return ve[c][i + dy + HY][dx + HY]; },
                                    [&](int c, int dy, int dx) { return vu[c][i + dy + HU][dx + HU]; }, r, Wi);
#pragma unroll
                    for (int c = 0; c < C; ++c) {
                        W[c][i] = q[c][s0 + i] + om1 * (T)Wi[c];
                        q[c][s0 + i] += (T)Wi[c];
                        acc[c] += (double)Wi[c] * (double)Wi[c];
                    }
                }
#pragma unroll
                for (int c = 0; c < C; ++c) store_w(c, ys, x, W[c]);
            }
        }
        block_sum<C, NT7>(acc, red);
        if (tid == 0) {
            double res = 0.0;
#pragma unroll
            for (int c = 0; c < C; ++c) res += sqrt(acc[c]);
            stl = decide<K_INNER32>(stl, rule, res / s.ht, 0.0);
        }
        __syncthreads();
    };

    // ---- G^-1 Z in place (Z in S as packed row pairs on entry; on exit the complex
    // slot pos(x) of region c H + y / 2 holds G^-1 Z of rows y, y + 1 as re, im)
    auto precond = [&]() {
        wg_fft_r8<T, LOGN, -1, NREG, NT7, RowMap<LOGN>>(S, twr);
        rows_post_forward<T, LOGN, BC, NREG, NT7>(S, twd);
        wg_fft_r8<T, LOGN, -1, NREG, NT7, ColMap<LOGN, BC>>(S, twc);
        cols_symbol_mapped<T, LOGN, BC, NREG, ColMap<LOGN, BC>>(S, sym, twd);
        wg_fft_r8<T, LOGN, +1, NREG, NT7, ColMap<LOGN, BC>>(S, twc);
        rows_pre_inverse<T, LOGN, BC, NREG, NT7>(S, twd);
        wg_fft_r8<T, LOGN, +1, NREG, NT7, RowMap<LOGN>>(S, twr);
    };
    // ---- primal descent U_{n+1} = U_n - tau_u grad F(U_n)^T P~, P~ = tau_p G^-1 Z
    // (the first iteration: (1 + omega) tau_p G^-1 W_0), in place on U (the adjoint
    // reads U only at its own point); mixed: on e, with f' at U_b + e.
    auto primal = [&](bool first) {
        const T tu = (T)s.tau_u * (T)s.tau_p * (first ? om1 : (T)1);
        if (tid < STRIP_THREADS) {
            const int x = tid % N, y0 = (tid / N) * L;
#pragma unroll
            for (int s0 = 0; s0 < L; s0 += LS) {
                const int ys = y0 + s0;
                T pt[C][LS + 2 * HY][2 * HY + 1];
#pragma unroll
                for (int c = 0; c < C; ++c)
#pragma unroll
                    for (int dx = -HY; dx <= HY; ++dx) {
                        const int px = pos(wrap<BC>(x + dx, N));
                        if constexpr (LS >= 2) {
                            // the strip's own rows, two per complex slot
#pragma unroll
                            for (int h = 0; h < LS / 2; ++h) {
                                const cplx<T> z = S[rix<LOGN>(c * H + (ys >> 1) + h, px)];
                                pt[c][2 * h + HY][dx + HY] = z.re;
                                pt[c][2 * h + 1 + HY][dx + HY] = z.im;
                            }
                        } else {
                            pt[c][HY][dx + HY] = rreal<T, LOGN>(S, c * H + (ys >> 1), 2 * px + (ys & 1));
                        }
                        // halo rows, through the boundary map
#pragma unroll
                        for (int r = -HY; r < LS + HY; ++r) {
                            if (r >= 0 && r < LS) continue;
                            if (!wg_needed<HY, LS>(r, dx)) continue;
                            const int yy = wrap<BC>(ys + r, N);
                            pt[c][r + HY][dx + HY] = rreal<T, LOGN>(S, c * H + (yy >> 1), 2 * px + (yy & 1));
                        }
                    }
#pragma unroll
                for (int i = 0; i < LS; ++i) {
                    const int g = (ys + i) * N + x;
                    T un[C], Uc[C], adj[C];
#pragma unroll
                    for (int c = 0; c < C; ++c) {
                        if constexpr (MODE == MODE_F64) {
                            un[c] = U[c * NN + g];
                            Uc[c] = un[c];
                        } else {
                            un[c] = first ? (T)0 : U[c * NN + g];
                            Uc[c] = (T)Ub[c * NN + g] + un[c];
                        }
                    }
                    eval_adjoint<EQ, T>(s, [&](int c, int dy, int dx) { return pt[c][i + dy + HY][dx + HY]; }, Uc,
                                        adj);
#pragma unroll
                    for (int c = 0; c < C; ++c) U[c * NN + g] = un[c] - tu * adj[c];
                }
            }
        }
        __syncthreads();
    };

    // ---- the initial state U_0 = U^k (or the pointwise reaction prox of U^k)
    auto initial = [&](auto *Ui) {
        for (int g = tid; g < NN; g += NT7) {
            if constexpr (EQ == EQ_SCHNAK) {
                double u = src[g], v = src[NN + g];
                if (s.init != 0) prox_schnak(src[g], src[NN + g], s.ht, s.sa, s.sb, s.kappa, u, v);
                Ui[g] = u;
                Ui[NN + g] = v;
            } else {
                Ui[g] = (s.init != 0 && EQ == EQ_LAP5) ? prox_ac(src[g], s.ht, s.b) : src[g];
            }
        }
        __syncthreads();
    };

    if constexpr (MODE == MODE_F64) {
        initial(U);
        residual64(U, true, [&](double res, double m) { stl = decide<K_INIT64>(stl, rule, res, m); });
        while (!stl.done) {
            const bool first = stl.iters == 0;
            precond();
            primal(first);
            residual64(U, false, [&](double res, double m) { stl = decide<K_ITER64>(stl, rule, res, m); });
        }
        // the result where the batched path leaves it: U[iters & 1]
        double *out = (double *)s.U[stl.iters & 1];
        if ((void *)out != (void *)U)
            for (int g = tid; g < C * NN; g += NT7) out[g] = U[g];
    } else {
        // outer initial pass: U = U^k (or its prox) in FP64
        initial(U64);
        residual64(U64, true, [&](double res, double m) { stl = decide<K_OUTER_INIT>(stl, rule, res, m); });
        while (!stl.outer_done) {
            // inner FP32 loop on the correction e (e_0 = 0, P_0 = 0) from W = r
            while (!stl.done) {
                const bool first = stl.iters == 0;
                precond();
                primal(first);
                residual32();
            }
            // outer update U += e, then r = F(U) in FP64 and the outer decision
            if (stl.iters > 0) {
                for (int g = tid; g < C * NN; g += NT7) U64[g] += (double)U[g];
                __syncthreads();
            }
            residual64(U64, true, [&](double res, double m) { stl = decide<K_OUTER_UPD>(stl, rule, res, m); });
        }
        double *out = s.U64[stl.outer & 1];
        if (out != U64)
            for (int g = tid; g < C * NN; g += NT7) out[g] = U64[g];
    }
    if (tid == 0) store_state(s.st, stl);
}

}  // namespace rdk
