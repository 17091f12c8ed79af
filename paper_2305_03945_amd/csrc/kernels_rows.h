// The three row-parallel steps of an iteration in one launch (2-D grids).
//
// G^-1 is linear, so the dual variable need not be formed: with Q_n = W_0 + ... +
// W_{n-1} (P_n = tau_p G^-1 Q_n, P_0 = 0),
//
//   P~ = P_{n+1} + omega (P_{n+1} - P_n) = tau_p G^-1 (Q_n + (1 + omega) W_n),
//
// so the row pass transforms Z_n = Q_n + (1 + omega) W_n and what comes back from
// the column pass is P~ itself (eqs. 21-22 in one inverse transform):
//
//   inverse row transform                                    -> P~
//   U_{n+1} = U_n - tau_u grad F(U_n)^T P~                                 (eq. 23)
//   W_{n+1} = F(U_{n+1}) (mixed: F~(e_{n+1})), its partial norms
//   Q_{n+2} = Q_{n+1} + W_{n+1};  forward row transform of Z_{n+1}
//
// A workgroup owns the R rows of one spectrum tile and computes all they need
// itself: P~ on the R + 4 HY rows and U_{n+1} on the R + 2 HY rows that the two
// stencils (reach HY) chain to, with no exchange between workgroups.  P~ never
// leaves LDS, the iterate is read and written once, and Q is touched on the
// workgroup's own rows only.  The spectrum is read on rows that other workgroups
// write, so the column pass moves it from S to S2 and this pass from S2 to S.
//
// What bounds it: on small grids the launches and each workgroup's serial chain (two
// launches an iteration fewer), on large ones the bytes (FP64 56 instead of 80 per
// point and iteration, mixed 32 instead of 48: P~ and the second reads of U_n and P
// are gone) and the transforms of the halo rows, which the four-row tiles double.
// Row-parallel steps of one iteration, us, three launches -> one: 128^2 FCH FP64
// 15.4 -> 8.2, 512^2 Neumann Cahn-Hilliard FP64 17.8 -> 12.3, 1024^2 Schnakenberg
// 45.4 -> 34.6 (FP64) and 28.9 -> 22.8 (mixed), 2048^2 Allen-Cahn 66.8 -> 60.4 and
// 43.8 -> 39.7, 4096^2 mixed 166 -> 160.
#pragma once
#include "kernels.h"

namespace rdk {

// Q consecutive values (Q = 1, 2 or 4), aligned to Q values.
template <typename T, int Q> struct QV { T v[Q]; };
template <int Q, typename T> __device__ __forceinline__ QV<T, Q> load_q(gptr_t<const T> p) {
    QV<T, Q> r;
    if constexpr (Q == 1) {
        r.v[0] = *p;
    } else {
        typedef T vq __attribute__((ext_vector_type(Q)));
        const vq m = *(const gptr_t<const vq>)p;
#pragma unroll
        for (int k = 0; k < Q; ++k) r.v[k] = m[k];
    }
    return r;
}
template <int Q, typename T> __device__ __forceinline__ void store_q(gptr_t<T> p, const QV<T, Q> &r) {
    if constexpr (Q == 1) {
        *p = r.v[0];
    } else {
        typedef T vq __attribute__((ext_vector_type(Q)));
        vq m;
#pragma unroll
        for (int k = 0; k < Q; ++k) m[k] = r.v[k];
        *(gptr_t<vq>)p = m;
    }
}

// Stencil window of M adjacent rows of Q points, reach HY (the diamond
// |dy| + |dx| <= HY around each of them): at(j, k, dy, dx) is the value at row j,
// point k, offset (dy, dx).
template <typename T, int HY, int M, int Q> struct WinQ {
    T v[M + 2 * HY][Q + 2 * HY];
    __device__ __forceinline__ T at(int j, int k, int dy, int dx) const { return v[j + dy + HY][HY + dx + k]; }
    // x reach that row d (relative to the first of the M rows) needs
    __host__ __device__ static constexpr int reach(int d) { return HY - (d < 0 ? -d : d >= M ? d - M + 1 : 0); }
    template <class Get> __device__ __forceinline__ void load(Get get) {
#pragma unroll
        for (int d = -HY; d < M + HY; ++d)
#pragma unroll
            for (int dx = -reach(d); dx < Q + reach(d); ++dx) v[d + HY][dx + HY] = get(d, dx);
    }
};

template <typename T, int LOGN, int BC, int EQ>
__device__ __forceinline__ void rows_iteration(SlotRef s, StateRef sst, cplx<T> *buf, double *scratch) {
    using Pl = RowsPlan<T, LOGN, EQ>;
    constexpr int C = Pl::C, N = Pl::N, H = N / 2, HY = Pl::HY, R = Pl::R, RU = Pl::RU, RP = Pl::RP;
    constexpr int NRI = Pl::NRI, NRF = Pl::NRF, NTH = Pl::NTH, V = Pl::V, QU = Pl::QU, QW = Pl::QW;
    constexpr bool F64 = sizeof(T) == 8;
    constexpr size_t NN = (size_t)N * N;
    const int tid = threadIdx.x;
    const int tile = xcd_tile(blockIdx.x, gridDim.x);
    const int y0 = tile * R;
    const int yp = y0 - 2 * HY, yu = y0 - HY;   // first row of P~, of U_{n+1}
    const int it = sst.iters;
    const auto Q = gp((T *)s.P);
    const auto Un = gp((const T *)s.U[it & 1]);
    const auto Un1 = gp((T *)s.U[(it + 1) & 1]);
    const cplx<T> *S = (const cplx<T> *)s.S2;
    const cplx<T> *twd = (const cplx<T> *)s.twd;
    Tw16<T, LOGN, V> twr;
    load_tw16<T, LOGN, V>(twr, (const cplx<T> *)s.tw);

    // grid row of local pair p of the P~ rows (its first row).  Neumann pairs
    // outside the grid are never used; they load their mirror image.
    auto pair_row = [&](int p) {
        const int y = yp + 2 * p;
        if (BC == BC_P) return y & (N - 1);
        return y < 0 ? -2 - y : y >= N ? 2 * N - 2 - y : y;
    };

    // ---- spectrum rows -> packed pair spectra in LDS
    {
        constexpr int TOT = NRI * H;
#pragma unroll
        for (int i = 0; i < (TOT + NTH - 1) / NTH; ++i) {
            const int idx = tid + i * NTH;
            if (TOT % NTH != 0 && idx >= TOT) break;
            const int reg = idx / H, l = idx % H;
            const cplx<T> *p = &S[spec_off<R>(reg / (RP / 2), pair_row(reg % (RP / 2)), l, N)];
            cplx<T> v[2];
            if constexpr (spec_vec<T>() == 2) {
                spec_load<T>(p, v);
            } else {
                spec_load<T>(p, v);
                spec_load<T>(p + 1, v + 1);
            }
            const cplx<T> a = v[0], b = v[1];
            if constexpr (BC == BC_P) {
                if (l == 0) {
                    buf[rix<LOGN>(reg, 0)] = {a.re, b.re};   // Z_0 = A_0 + i B_0
                    buf[rix<LOGN>(reg, H)] = {a.im, b.im};   // Z_{N/2}
                } else {
                    buf[rix<LOGN>(reg, l)] = {a.re - b.im, a.im + b.re};
                    buf[rix<LOGN>(reg, N - l)] = {a.re + b.im, b.re - a.im};
                }
            } else {
                buf[rix<LOGN>(reg, l)] = a;
                buf[rix<LOGN>(reg, H + l)] = b;
            }
        }
        __syncthreads();
        if constexpr (BC == BC_N) rows_pre_inverse<T, LOGN, BC, NRI, NTH>(buf, twd);
    }
    wg_fft16<T, LOGN, +1, NRI, NTH, V>(buf, twr);

    auto pos = [](int x) { return BC == BC_P ? x : dct_pos(x, N); };
    auto wx = [](int x) { return wrap<BC>(x, N); };

    // ---- U_{n+1} on rows yu .. yu + RU - 1 (Neumann: those inside the grid)
    constexpr int TOTU = RU * N / QU, IU = (TOTU + NTH - 1) / NTH;
    QV<T, QU> un1[IU][C];
    {
        // the transform returns G^-1 Z; the first one W_0, not (1 + omega) W_0, was transformed
        const T tu = (T)s.tau_u * (T)s.tau_p * (it == 0 ? (T)1 + (T)s.omega : (T)1);
        const auto Ub = gp((const float *)s.Ub32);
#pragma unroll
        for (int i = 0; i < IU; ++i) {
            const int idx = tid + i * NTH;
            if (TOTU % NTH != 0 && idx >= TOTU) break;
            const int r = idx / (N / QU), x0 = (idx % (N / QU)) * QU;
            const int y = yu + r;
            if (BC == BC_N && (y < 0 || y >= N)) continue;
            const int yg = BC == BC_P ? y & (N - 1) : y;
            const size_t g = (size_t)yg * N + x0;
            WinQ<T, HY, 1, QU> wp[C];
#pragma unroll
            for (int c = 0; c < C; ++c)
                wp[c].load([&](int d, int dx) -> T {
                    const int rl = (BC == BC_P ? y + d : wrap<BC>(y + d, N)) - yp;
                    return rreal<T, LOGN>(buf, c * (RP / 2) + rl / 2, 2 * pos(wx(x0 + dx)) + (rl & 1));
                });
            if constexpr (EQ == EQ_FCH) {
                // the adjoint reads U on the 5-point neighbourhood (mixed: U_b + e)
                WinQ<T, 1, 1, QU> wu, we;
                auto at = [&](auto f) {
                    return [=](int d, int dx) { return f[(size_t)wrap<BC>(yg + d, N) * N + wx(x0 + dx)]; };
                };
                if constexpr (F64) {
                    wu.load(at(Un));
                    we = wu;
                } else {
                    WinQ<float, 1, 1, QU> wub;
                    wub.load(at(Ub));
                    if (it > 0) we.load(at(Un));
                    else we.load([](int, int) { return (T)0; });
                    wu.load([&](int d, int dx) { return (T)wub.v[d + 1][dx + 1] + we.v[d + 1][dx + 1]; });
                }
#pragma unroll
                for (int k = 0; k < QU; ++k)
                    un1[i][0].v[k] =
                        we.at(0, k, 0, 0) -
                        tu * eval_adjoint_fch<T>(s, [&](int, int dy, int dx) { return wp[0].at(0, k, dy, dx); },
                                                 [&](int, int dy, int dx) { return wu.at(0, k, dy, dx); });
            } else {
                QV<T, QU> un[C];
                T Uc[QU][C];
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    if constexpr (F64) {
                        un[c] = load_q<QU, T>(Un + c * NN + g);
#pragma unroll
                        for (int k = 0; k < QU; ++k) Uc[k][c] = un[c].v[k];
                    } else {
                        un[c] = QV<T, QU>{};
                        if (it > 0) un[c] = load_q<QU, T>(Un + c * NN + g);
                        const QV<float, QU> ub = load_q<QU, float>(Ub + c * NN + g);
#pragma unroll
                        for (int k = 0; k < QU; ++k) Uc[k][c] = (T)ub.v[k] + un[c].v[k];
                    }
                }
#pragma unroll
                for (int k = 0; k < QU; ++k) {
                    T adj[C];
                    eval_adjoint<EQ, T>(s, [&](int c, int dy, int dx) { return wp[c].at(0, k, dy, dx); }, Uc[k], adj);
#pragma unroll
                    for (int c = 0; c < C; ++c) un1[i][c].v[k] = un[c].v[k] - tu * adj[c];
                }
            }
            if (r >= HY && r < HY + R) {
#pragma unroll
                for (int c = 0; c < C; ++c) store_q<QU, T>(Un1 + c * NN + g, un1[i][c]);
            }
        }
    }
    __syncthreads();
    // U_{n+1} replaces P~ in LDS, rows in natural order
    T *ul = (T *)buf;
#pragma unroll
    for (int i = 0; i < IU; ++i) {
        const int idx = tid + i * NTH;
        if (TOTU % NTH != 0 && idx >= TOTU) break;
#pragma unroll
        for (int c = 0; c < C; ++c)
#pragma unroll
            for (int k = 0; k < QU; ++k) ul[c * (RU * N) + idx * QU + k] = un1[i][c].v[k];
    }
    __syncthreads();

    // ---- W = F(U_{n+1}) (mixed: F~(e_{n+1})) on the workgroup's own row pairs
    constexpr int TOTW = R / 2 * N / QW, IW = (TOTW + NTH - 1) / NTH;
    T w[IW][C][2][QW];   // Z_{n+1}
    const T om1 = (T)1 + (T)s.omega;
    double acc[2 * C];
#pragma unroll
    for (int k = 0; k < 2 * C; ++k) acc[k] = 0.0;
#pragma unroll
    for (int i = 0; i < IW; ++i) {
        const int idx = tid + i * NTH;
        if (TOTW % NTH != 0 && idx >= TOTW) break;
        const int p = idx / (N / QW), x0 = (idx % (N / QW)) * QW;
        const int y = y0 + 2 * p;
        const size_t g = (size_t)y * N + x0;
        WinQ<T, HY, 2, QW> wu[C];
#pragma unroll
        for (int c = 0; c < C; ++c)
            wu[c].load([&](int d, int dx) -> T {
                const int rl = (BC == BC_P ? y + d : wrap<BC>(y + d, N)) - yu;
                return ul[(c * RU + rl) * N + wx(x0 + dx)];
            });
        QV<T, QW> q[2][C];   // Q_{n+1}; mixed: Q_1 = r
        if (F64 || it > 0) {
#pragma unroll
            for (int c = 0; c < C; ++c)
#pragma unroll
                for (int j = 0; j < 2; ++j) q[j][c] = load_q<QW, T>((gptr_t<const T>)Q + c * NN + g + j * N);
        }
        if constexpr (F64) {
            QV<double, QW> uk[2][C];
#pragma unroll
            for (int c = 0; c < C; ++c)
#pragma unroll
                for (int j = 0; j < 2; ++j) uk[j][c] = load_q<QW, double>(gp((const double *)s.Uk) + c * NN + g + j * N);
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int k = 0; k < QW; ++k) {
                    double W[C], Uc[C], ukc[C];
#pragma unroll
                    for (int c = 0; c < C; ++c) ukc[c] = uk[j][c].v[k];
                    eval_F<EQ, double>(s, [&](int c, int dy, int dx) { return wu[c].at(j, k, dy, dx); }, ukc, W, Uc);
#pragma unroll
                    for (int c = 0; c < C; ++c) {
                        acc[c] += W[c] * W[c];
                        acc[C + c] += Uc[c] - ukc[c];
                        w[i][c][j][k] = q[j][c].v[k] + om1 * W[c];
                        q[j][c].v[k] += W[c];
                    }
                }
        } else {
            constexpr int HU = ftilde_hu<EQ>();
            const auto Ub = gp((const float *)s.Ub32);
            WinQ<float, HU, 2, QW> wub[C];
            QV<float, QW> r4[2][C];
#pragma unroll
            for (int c = 0; c < C; ++c) {
#pragma unroll
                for (int d = -HU; d < 2 + HU; ++d) {
                    constexpr int HX = HU;
                    const auto row = Ub + c * NN + (size_t)wrap<BC>(y + d, N) * N;
                    const QV<float, QW> m = load_q<QW, float>(row + x0);
#pragma unroll
                    for (int k = 0; k < QW; ++k) wub[c].v[d + HU][HX + k] = m.v[k];
#pragma unroll
                    for (int h = 1; h <= WinQ<float, HU, 2, QW>::reach(d); ++h) {
                        wub[c].v[d + HU][HX - h] = row[wx(x0 - h)];
                        wub[c].v[d + HU][HX + QW - 1 + h] = row[wx(x0 + QW - 1 + h)];
                    }
                }
#pragma unroll
                for (int j = 0; j < 2; ++j) r4[j][c] = load_q<QW, float>(gp((const float *)s.r32) + c * NN + g + j * N);
            }
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int k = 0; k < QW; ++k) {
                    float rc[C], W[C];
#pragma unroll
                    for (int c = 0; c < C; ++c) {
                        rc[c] = r4[j][c].v[k];
                        if (it == 0) q[j][c].v[k] = rc[c];
                    }
                    eval_Ftilde<EQ>(s, [&](int c, int dy, int dx) { return wu[c].at(j, k, dy, dx); },
                                    [&](int c, int dy, int dx) { return wub[c].at(j, k, dy, dx); }, rc, W);
#pragma unroll
                    for (int c = 0; c < C; ++c) {
                        acc[c] += (double)W[c] * (double)W[c];
                        w[i][c][j][k] = q[j][c].v[k] + om1 * W[c];
                        q[j][c].v[k] += W[c];
                    }
                }
        }
#pragma unroll
        for (int c = 0; c < C; ++c)
#pragma unroll
            for (int j = 0; j < 2; ++j) store_q<QW, T>(Q + c * NN + g + j * N, q[j][c]);
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < IW; ++i) {
        const int idx = tid + i * NTH;
        if (TOTW % NTH != 0 && idx >= TOTW) break;
        const int p = idx / (N / QW), x0 = (idx % (N / QW)) * QW;
#pragma unroll
        for (int c = 0; c < C; ++c)
#pragma unroll
            for (int k = 0; k < QW; ++k)
                buf[rix<LOGN>(c * (R / 2) + p, pos(x0 + k))] = {w[i][c][0][k], w[i][c][1][k]};
    }
    __syncthreads();
    wg_fft16<T, LOGN, -1, NRF, NTH, V>(buf, twr);
    rows_store_spectrum<T, LOGN, BC, C, R, NTH>(buf, (cplx<T> *)s.S, y0, twd);
    write_partials<C, NTH>(s, tile, acc, scratch);
}

// One iteration's row-parallel steps; mixed: the FP64 outer update instead once
// the inner loop has stopped (K_MIXED of k_row_forward).
template <typename T, int LOGN, int BC, int EQ>
__global__ __launch_bounds__((RowsPlan<T, LOGN, EQ>::NTH), (RowsPlan<T, LOGN, EQ>::WPE)) void k_rows(Slot *const *slots) {
    using Pl = RowsPlan<T, LOGN, EQ>;
    __shared__ cplx<T> buf[Pl::NRI * lds_region<LOGN>()];
    __shared__ double scratch[2 * Pl::C * (Pl::NTH / 64)];
    SlotRef s = slot_of(slots);
    StateRef sst = state_of(s);
    if constexpr (sizeof(T) == 8) {
        if (sst.done) return;
        rows_iteration<T, LOGN, BC, EQ>(s, sst, buf, scratch);
    } else {
        if (sst.outer_done) return;
        if (sst.done) row_forward_pass<T, LOGN, BC, EQ, K_OUTER_UPD, Pl::NTH>(s, sst, buf, scratch);
        else rows_iteration<T, LOGN, BC, EQ>(s, sst, buf, scratch);
    }
}

}  // namespace rdk
