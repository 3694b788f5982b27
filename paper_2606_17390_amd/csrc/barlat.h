// barlat.h -- Barlat Yld2004-18p yield function (Eq. Phi_barlat, App. A) and
// its closest-point return map (App. B line search, App. C Alg. C2) for one
// Gauss point, FP64, in the material frame.
//
// phi(T) = [1/4 sum_ij |s'_i - s''_j|^m]^(1/m), s'_i, s''_j the principal
// values of s' = C' : P : T and s'' = C'' : P : T (P the deviatoric
// projector).  Flow N = dphi/dT and dN/dT come from the principal-value
// derivatives lifted to tensors (spectral gradient and Hessian with divided
// differences; coincident values take their limit).  Unlike Hill-48, the
// closest-point equations have no closed-form reduction: a Newton iteration
// on (T, dgamma) (alpha = alpha_n + dgamma) solves the symmetric bordered
// system [[E^-1 + dgamma dN/dT, N], [N^T, -sigma_y']] by a 6x6 Cholesky
// factorisation, damped by the line search of App. B.
#pragma once

#include "fem_device.h"

namespace fem {

// 18 coefficients c'12 c'13 c'21 c'23 c'31 c'32 c'44 c'55 c'66, the same nine
// for c'', and the exponent m; mi = m - 2 when m is an integer in [2, 64]
// (the published fits use m = 8), else -1
struct BarlatCoef {
    double c[2][9];
    double m;
    int mi;
};

__device__ inline void load_barlat(const double* __restrict__ p, BarlatCoef& b) {
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        b.c[0][k] = p[k];
        b.c[1][k] = p[9 + k];
    }
    b.m = p[18];
    b.mi = (b.m >= 2.0 && b.m <= 64.0 && b.m == floor(b.m)) ? (int)b.m - 2 : -1;
}

// |d|^(m-2): by repeated squaring for an integer exponent (the same for every
// lane, so the branch is uniform), else pow; 1 at d = 0 for m = 2
__device__ inline double abs_pow_m2(double ad, const BarlatCoef& b) {
    if (b.mi >= 0) {
        double r = 1.0, x = ad;
        for (int k = b.mi; k; k >>= 1) {
            if (k & 1) r *= x;
            x *= x;
        }
        return r;
    }
    return pow(ad, b.m - 2.0);
}

// s = C : P : t as a symmetric 3x3 (t Mandel)
__device__ inline void barlat_apply(const double* c, const double t[6], double S[3][3]) {
    const double tr = (t[0] + t[1] + t[2]) * (1.0 / 3.0);
    const double s0 = t[0] - tr, s1 = t[1] - tr, s2 = t[2] - tr;
    S[0][0] = -c[0] * s1 - c[1] * s2;
    S[1][1] = -c[2] * s0 - c[3] * s2;
    S[2][2] = -c[4] * s0 - c[5] * s1;
    S[1][2] = S[2][1] = c[6] * t[3] * kInvSqrt2;
    S[0][2] = S[2][0] = c[7] * t[4] * kInvSqrt2;
    S[0][1] = S[1][0] = c[8] * t[5] * kInvSqrt2;
}

// Mandel vector of (C : P)^T : X for a symmetric X = Mandel x
__device__ inline void barlat_apply_T(const double* c, const double x[6], double out[6]) {
    // C^T x (normal block transposed, shear diagonal), then the deviator
    const double y0 = -c[2] * x[1] - c[4] * x[2];
    const double y1 = -c[0] * x[0] - c[5] * x[2];
    const double y2 = -c[1] * x[0] - c[3] * x[1];
    const double tr = (y0 + y1 + y2) * (1.0 / 3.0);
    out[0] = y0 - tr;
    out[1] = y1 - tr;
    out[2] = y2 - tr;
    out[3] = c[6] * x[3];
    out[4] = c[7] * x[4];
    out[5] = c[8] * x[5];
}

// Phi^(1/m); the published fits' m = 8 by three square roots
__device__ inline double barlat_root(double Phi, const BarlatCoef& b) {
    if (b.mi == 6 && Phi > 1e-280 && Phi < 1e280) {
        double r = Phi;
#pragma unroll
        for (int k = 0; k < 3; ++k) r *= rsqrt_nr(r);
        return r;
    }
    return exp(log(Phi) / b.m);
}

// Principal values of both transformed deviators, their eigenvectors, and the
// gradient g / Hessian h of phi with respect to lam = (s'_1..3, s''_1..3).
struct BarlatState {
    double lam[6];
    double P[2][3][3];  // eigenvectors (columns)
    double g[6];
    double phi;
};

// Symmetric 3x3 eigen-decomposition started from an orthonormal basis Q
// (columns) close to the eigenvectors: cyclic Jacobi on Q^T S Q, which is
// nearly diagonal, then Q <- Q Q'.  Between Newton iterates and line-search
// trials the transformed deviators turn little, so one or two sweeps replace
// the four to six of a start from the identity.
__device__ __forceinline__ void eig_sym3_from(const double S[3][3], double mu[3], double Q[3][3]) {
    double W[3][3], B[3][3], Qs[3][3];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int q = 0; q < 3; ++q) W[i][q] = S[i][0] * Q[0][q] + S[i][1] * Q[1][q] + S[i][2] * Q[2][q];
#pragma unroll
    for (int p = 0; p < 3; ++p)
#pragma unroll
        for (int q = p; q < 3; ++q) {
            const double v = Q[0][p] * W[0][q] + Q[1][p] * W[1][q] + Q[2][p] * W[2][q];
            B[p][q] = v;
            B[q][p] = v;
        }
    eig_sym3<double>(B, mu, Qs);
    double Qn[3][3];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) Qn[i][j] = Q[i][0] * Qs[0][j] + Q[i][1] * Qs[1][j] + Q[i][2] * Qs[2][j];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) Q[i][j] = Qn[i][j];
}

// st.P on entry: orthonormal bases to start from (the identity, or the
// eigenvectors of nearby deviators)
__device__ __forceinline__ double barlat_principal(const BarlatCoef& b, const double t[6], BarlatState& st) {
#pragma unroll
    for (int a = 0; a < 2; ++a) {
        double S[3][3], mu[3];
        barlat_apply(b.c[a], t, S);
        eig_sym3_from(S, mu, st.P[a]);
        st.lam[3 * a] = mu[0];
        st.lam[3 * a + 1] = mu[1];
        st.lam[3 * a + 2] = mu[2];
    }
    double Phi = 0.0, dPhi[6] = {0, 0, 0, 0, 0, 0};
    const double m = b.m;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const double d = st.lam[i] - st.lam[3 + j], ad = fabs(d);
            const double p2 = abs_pow_m2(ad, b);  // |d|^(m-2)
            Phi += 0.25 * p2 * ad * ad;
            const double t1 = 0.25 * m * d * p2;
            dPhi[i] += t1;
            dPhi[3 + j] -= t1;
        }
    st.phi = barlat_root(Phi, b);
    const double f = st.phi / (m * Phi);
#pragma unroll
    for (int a = 0; a < 6; ++a) st.g[a] = f * dPhi[a];
    return st.phi;
}

// N = dphi/dt (Mandel) = sum_a L_a^T (sum_i g_ai p_ai p_ai^T)
__device__ __forceinline__ void barlat_flow(const BarlatCoef& b, const BarlatState& st, double N[6]) {
#pragma unroll
    for (int k = 0; k < 6; ++k) N[k] = 0.0;
#pragma unroll
    for (int a = 0; a < 2; ++a) {
        double gp[3][3], n[6], o[6];
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int q = 0; q < 3; ++q) gp[i][q] = st.g[3 * a + q] * st.P[a][i][q];
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            const int i = mi(k), j = mj(k);
            n[k] = mw<double>(k) * (gp[i][0] * st.P[a][j][0] + gp[i][1] * st.P[a][j][1] + gp[i][2] * st.P[a][j][2]);
        }
        barlat_apply_T(b.c[a], n, o);
#pragma unroll
        for (int k = 0; k < 6; ++k) N[k] += o[k];
    }
}

// L_a^T of the Mandel unit tensor sym(p_i p_k^T) (i = k: p_i p_i^T; else
// scaled to unit norm), p_i the eigenvectors of block a
template <int a, int i, int k>
__device__ __forceinline__ void barlat_dyad(const BarlatCoef& b, const BarlatState& st, double o[6]) {
    double n[6];
#pragma unroll
    for (int t = 0; t < 6; ++t) {
        const int p = mi(t), q = mj(t);
        const double v = i == k ? st.P[a][p][i] * st.P[a][q][i]
                                : kInvSqrt2 * (st.P[a][p][i] * st.P[a][q][k] + st.P[a][p][k] * st.P[a][q][i]);
        n[t] = mw<double>(t) * v;
    }
    barlat_apply_T(b.c[a], n, o);
}

// Lower triangle of A = E^-1 + dg dN/dt (N = barlat_flow).  With
// n_ai = L_a^T (p_ai p_ai^T), m_aik the same of the unit shear dyads and
// d_ij = s'_i - s''_j,
//   dN/dt = f sum_ij t_ij (n_0i - n_1j)(n_0i - n_1j)^T + (1 - m) / phi N N^T
//           + sum theta_aik m_aik m_aik^T,
//   f = phi / (m Phi), t_ij = m (m - 1) / 4 |d_ij|^(m-2),
// and theta the divided differences of the gradient in the principal values
// (for coincident ones f sum t): 700 multiply-adds.  Column by column through
// the spectral derivative of a unit stress it took 3,600, three quarters of a
// Newton iteration.
__device__ __forceinline__ void barlat_matrix(const BarlatCoef& b, const BarlatState& st, const Modes& md, double dg,
                                     const double N[6], double A[6][6]) {
    auto rank_one = [&](double w, const double v[6]) {
#pragma unroll
        for (int p = 0; p < 6; ++p) {
            const double wv = w * v[p];
#pragma unroll
            for (int q = 0; q <= p; ++q) A[p][q] = m_fma(wv, v[q], A[p][q]);
        }
    };
    const double im = recip(md.mu2), ih = (recip(md.k3) - im) * (1.0 / 3.0);
#pragma unroll
    for (int i = 0; i < 6; ++i)
#pragma unroll
        for (int j = 0; j <= i; ++j) A[i][j] = (i < 3 ? ih : 0.0) + (i == j ? im : 0.0);
    // f t_ij and their sums over i and j; Phi as barlat_principal forms it
    double t[3][3], Phi = 0.0;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const double ad = fabs(st.lam[i] - st.lam[3 + j]);
            t[i][j] = 0.25 * abs_pow_m2(ad, b);
            Phi += t[i][j] * ad * ad;
        }
    const double f = st.phi * (b.m - 1.0) / Phi;
    double ts[6] = {0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            t[i][j] *= f;
            ts[i] += t[i][j];
            ts[3 + j] += t[i][j];
        }
    static_for<0, 2>([&](auto AA) {
        constexpr int a = decltype(AA)::value;
        const double* l = st.lam + 3 * a;
        const double scale = fabs(l[0]) + fabs(l[1]) + fabs(l[2]) + 1e-300;
        static_for<0, 3>([&](auto KK) {
            constexpr int i = decltype(KK)::value < 2 ? 0 : 1, k = decltype(KK)::value == 0 ? 1 : 2;
            const double dl = l[i] - l[k];
            const double th = fabs(dl) > 1e-9 * scale ? (st.g[3 * a + i] - st.g[3 * a + k]) / dl : ts[3 * a + i];
            double m[6];
            barlat_dyad<a, i, k>(b, st, m);
            rank_one(dg * th, m);
        });
    });
    double n[6][6];
    barlat_dyad<0, 0, 0>(b, st, n[0]);
    barlat_dyad<0, 1, 1>(b, st, n[1]);
    barlat_dyad<0, 2, 2>(b, st, n[2]);
    barlat_dyad<1, 0, 0>(b, st, n[3]);
    barlat_dyad<1, 1, 1>(b, st, n[4]);
    barlat_dyad<1, 2, 2>(b, st, n[5]);
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            double v[6];
#pragma unroll
            for (int q = 0; q < 6; ++q) v[q] = n[i][q] - n[3 + j][q];
            rank_one(dg * t[i][j], v);
        }
    rank_one(dg * (1.0 - b.m) / st.phi, N);
}

// Cholesky factor of a symmetric positive definite 6x6 given by its lower
// triangle, in place, with the reciprocals of the diagonal on the diagonal
// (1/0 and the root of a negative pivot keep their infinity and NaN)
__device__ __forceinline__ void chol6(double A[6][6]) {
#pragma unroll
    for (int j = 0; j < 6; ++j) {
        double s = A[j][j];
#pragma unroll
        for (int k = 0; k < j; ++k) s -= A[j][k] * A[j][k];
        const double id = s > 1e-280 && s < 1e280 ? rsqrt_nr(s) : 1.0 / sqrt(s);
        A[j][j] = id;
#pragma unroll
        for (int i = j + 1; i < 6; ++i) {
            double x = A[i][j];
#pragma unroll
            for (int k = 0; k < j; ++k) x -= A[i][k] * A[j][k];
            A[i][j] = x * id;
        }
    }
}

__device__ __forceinline__ void chol6_solve(const double L[6][6], double x[6]) {
#pragma unroll
    for (int i = 0; i < 6; ++i) {
        double s = x[i];
#pragma unroll
        for (int k = 0; k < i; ++k) s -= L[i][k] * x[k];
        x[i] = s * L[i][i];
    }
#pragma unroll
    for (int i = 5; i >= 0; --i) {
        double s = x[i];
#pragma unroll
        for (int k = i + 1; k < 6; ++k) s -= L[k][i] * x[k];
        x[i] = s * L[i][i];
    }
}

// Result of the Barlat local update (material frame); the algorithmic
// tangent goes to the caller's array cep[21] (upper triangle, row by row)
struct LocalB {
    double T[6];
    double hist[7];
    double ftr, sy_n;
    int plastic, converged;
};

// E^-1 x for isotropic elasticity (Mandel)
__device__ inline void elastic_compliance(const Modes& h, const double x[6], double y[6]) {
    const double hm = (x[0] + x[1] + x[2]) * (1.0 / 3.0);
    const double im = recip(h.mu2), ik = recip(h.k3);
#pragma unroll
    for (int k = 0; k < 6; ++k) y[k] = (k < 3 ? (x[k] - hm) : x[k]) * im;
#pragma unroll
    for (int k = 0; k < 3; ++k) y[k] += hm * ik;  // (3 kappa)^-1 on the spherical part
}

// E : x for isotropic elasticity (Mandel)
__device__ inline void elastic_stiffness(const Modes& h, const double x[6], double y[6]) {
    const double tr = x[0] + x[1] + x[2];
#pragma unroll
    for (int k = 0; k < 6; ++k) y[k] = h.mu2 * x[k] + (k < 3 ? h.lam * tr : 0.0);
}

// Local update.  The reduced closest-point equations at (T, dg), alpha =
// alpha_n + dg, are
//   G1 = E^-1 (T - t_tr) + dg N(T)  (strain),  G3 = phi(T) - sigma_y(alpha_n + dg),
// and the merit of Eq. (merit) is psi = 1/2 G^T G with the stress rows
// T - t_tr + dg E : N = E : G1 and the yield row G3 (both in stress units).
//
// One loop holds the yield check, the Newton steps and the line search: every
// pass evaluates the yield function, its flow and the residual at one stress,
// and each lane then takes up its own next step.  The code for each part is
// there once (with a call per use the compiler kept them as functions, with
// their states passed through scratch memory), lanes in a line search do not
// hold up the others, and an accepted trial is the next iterate without being
// evaluated again.  Bound by FP64 issue and latency at one wave per SIMD; the
// pass over 127,000 elements (half the Gauss points plastic) took 3.59 ms,
// 1.40 ms with the closed form of the system matrix.
__device__ __forceinline__ void local_update_barlat(const double eps[6], const double* hist_n, const Mat& m, const Modes& md,
                                           const BarlatCoef& b, LocalB& o, double* __restrict__ cep) {
    double ee[6];
    ee[0] = eps[0] - hist_n[0];
    ee[1] = eps[1] - hist_n[1];
    ee[2] = eps[2] - hist_n[2];
    ee[3] = eps[3] - kSqrt2 * hist_n[3];
    ee[4] = eps[4] - kSqrt2 * hist_n[4];
    ee[5] = eps[5] - kSqrt2 * hist_n[5];
    const double tr = ee[0] + ee[1] + ee[2];
    double t_tr[6];
#pragma unroll
    for (int i = 0; i < 6; ++i) t_tr[i] = md.mu2 * ee[i] + (i < 3 ? md.lam * tr : 0.0);
    const double alpha_n = hist_n[6];
    double dsig;
    o.sy_n = hardening(m, alpha_n, dsig);
    o.plastic = 0;
    o.converged = 1;
    BarlatState st;
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = 0; j < 3; ++j) st.P[a][i][j] = i == j ? 1.0 : 0.0;
    enum { kTrial, kStart, kFull, kGuess, kSearch };
    int state = kTrial, it = 0, ls = 0;
    double T[6], Tt[6], dT[6], N[6];  // iterate, evaluated stress, Newton direction, flow at Tt
    double dg = 0.0, dgt = 0.0, ddg = 0.0, psi = 0.0, zeta = 0.0, prev = __builtin_inf();
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        Tt[k] = t_tr[k];
        T[k] = dT[k] = 0.0;
    }
    for (;;) {
        barlat_principal(b, Tt, st);
        barlat_flow(b, st, N);
        if (state == kTrial) {
            o.ftr = st.phi - o.sy_n;
            if (!(o.ftr > 0.0)) break;
            o.plastic = 1;
            // start on the current yield surface: phi is homogeneous of degree
            // one, so T0 = t_tr sigma_y(alpha_n) / phi(t_tr), with the flow and
            // eigenvectors of t_tr and r times its principal values, and
            // dgamma0 from the flow rule projected on N(T0) (the root is
            // unique, the start only saves iterations)
            const double r = o.sy_n / st.phi;
            double c[6], nc = 0.0, nn = 0.0;
            elastic_compliance(md, t_tr, c);
#pragma unroll
            for (int i = 0; i < 6; ++i) {
                Tt[i] = r * t_tr[i];
                st.lam[i] *= r;
                nc += N[i] * c[i];
                nn += N[i] * N[i];
            }
            st.phi = o.sy_n;
            dgt = (1.0 - r) * nc / nn;
            if (!(dgt > 0.0)) dgt = 0.0;
            state = kStart;
        }
        // residual and merit
        double G[7], psi_t = 0.0, gn = 0.0;
        {
            double c[6], Eg[6];
#pragma unroll
            for (int k = 0; k < 6; ++k) c[k] = Tt[k] - t_tr[k];
            elastic_compliance(md, c, G);
#pragma unroll
            for (int k = 0; k < 6; ++k) G[k] += dgt * N[k];
            elastic_stiffness(md, G, Eg);
            const double i2 = 2.0 * recip(md.mu2);
#pragma unroll
            for (int k = 0; k < 6; ++k) {
                psi_t += Eg[k] * Eg[k];
                gn = fmax(gn, fabs(Eg[k]) * i2);
            }
            G[6] = st.phi - hardening(m, alpha_n + dgt, dsig);
            psi_t = 0.5 * (psi_t + G[6] * G[6]);
            gn = fmax(gn, fabs(G[6]) / o.sy_n);
        }
        // line search of App. B on the merit
        if (state != kStart) {
            bool next = false;  // another trial along dT
            if (state == kFull) {
                if (!(psi_t < (1.0 - 2.0 * 1e-4) * psi)) {
                    zeta = psi / (psi + psi_t);
                    if (!(zeta == zeta)) zeta = 0.1;
                    ls = 0;
                    state = kGuess;
                    next = true;
                }
            } else if (state == kGuess) {
                zeta = fmax(0.1 * zeta, psi / (psi + psi_t));
                state = kSearch;
                next = true;
            } else if (!(psi_t < (1.0 - 2.0 * 1e-4 * zeta) * psi) && ls < 20) {
                ++ls;
                state = kGuess;
                next = true;
            }
            if (next) {
#pragma unroll
                for (int k = 0; k < 6; ++k) Tt[k] = T[k] + zeta * dT[k];
                dgt = dg + zeta * ddg;
                continue;
            }
        }
#pragma unroll
        for (int k = 0; k < 6; ++k) T[k] = Tt[k];
        dg = dgt;
        psi = psi_t;
        // gn: the scaled residual, stress rows E : G1 over mu, the yield row
        // over sigma_y(alpha_n); converged at 1e-14, or at the rounding floor (a
        // step below 1e-9 that does not halve it; the floor grows with the
        // stress, so no fixed level detects it).  A residual that is not a
        // number (fmax passes it over, the merit keeps it) ends the iteration
        // without convergence
        const bool number = psi == psi;
        const bool conv = number && it < 60 && (gn <= 1e-14 || (gn <= 1e-9 && gn >= 0.5 * prev));
        const bool last = conv || it >= 60 || !number;
        prev = gn;
        // the bordered system at the iterate
        double A[6][6], w[6];
        barlat_matrix(b, st, md, dg, N, A);
        chol6(A);
#pragma unroll
        for (int k = 0; k < 6; ++k) w[k] = N[k];
        chol6_solve(A, w);  // Xi N = A^-1 N
        double NAw = 0.0;
#pragma unroll
        for (int k = 0; k < 6; ++k) NAw += N[k] * w[k];
        if (last) {
            o.converged = conv ? 1 : 0;
            // algorithmic tangent Xi - Xi N (Xi N)^T / (N Xi N + sigma_y'),
            // Xi = A^-1 = Y^T Y with Y the inverse of the factor
            const double den = 1.0 / (NAw + dsig);
            double Y[6][6];
#pragma unroll
            for (int j = 0; j < 6; ++j) {
                Y[j][j] = A[j][j];
#pragma unroll
                for (int i = j + 1; i < 6; ++i) {
                    double v = 0.0;
#pragma unroll
                    for (int k = j; k < i; ++k) v -= A[i][k] * Y[k][j];
                    Y[i][j] = v * A[i][i];
                }
            }
            int c = 0;
#pragma unroll
            for (int i = 0; i < 6; ++i)
#pragma unroll
                for (int j = i; j < 6; ++j) {
                    double v = 0.0;
#pragma unroll
                    for (int k = j; k < 6; ++k) v += Y[k][i] * Y[k][j];
                    cep[c++] = v - w[i] * w[j] * den;
                }
            break;
        }
        // Newton step
        double NAu = 0.0;
        chol6_solve(A, G);  // A^-1 G1 (the first six)
#pragma unroll
        for (int k = 0; k < 6; ++k) NAu += N[k] * G[k];
        ddg = (G[6] - NAu) / (NAw + dsig);
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            dT[k] = -G[k] - w[k] * ddg;
            Tt[k] = T[k] + dT[k];
        }
        dgt = dg + ddg;
        state = kFull;
        ++it;
    }
    if (!o.plastic) {
#pragma unroll
        for (int i = 0; i < 6; ++i) o.T[i] = t_tr[i];
#pragma unroll
        for (int i = 0; i < 7; ++i) o.hist[i] = hist_n[i];
        int c = 0;
#pragma unroll
        for (int i = 0; i < 6; ++i)
#pragma unroll
            for (int j = i; j < 6; ++j) cep[c++] = ((i < 3 && j < 3) ? md.lam : 0.0) + ((i == j) ? md.mu2 : 0.0);
        return;
    }
#pragma unroll
    for (int k = 0; k < 6; ++k) o.T[k] = T[k];
    // eps^p_{n+1} = eps^p_n + dg N (tensor components), alpha_{n+1} = alpha_n + dg
#pragma unroll
    for (int k = 0; k < 6; ++k) o.hist[k] = hist_n[k] + dg * N[k] / mw<double>(k);
    o.hist[6] = alpha_n + dg;
}

}  // namespace fem
