// iod_sens.hip -- gfx950 kernels of libiod's sensitivities and local
// refinement: the discrete adjoint of the RK4 propagation and the residual
// cost (cost gradient), the forward tangent (state transition matrix) for
// the Gauss-Newton normal equations, and the damped Gauss-Newton step and
// acceptance that refine the swarm's best (in place of the paper's
// Levenberg-Marquardt Local Minimization, eqs. non:linear:lsq and
// nonlinlsq:cost).
#include <algorithm>

#include "iod_device.h"
#include "iod_launch.h"

namespace iodk {

// ---------------------------------------------------------------------------
// Sensitivities: discrete adjoint (reverse sweep) and forward tangent of the
// RK4 map, for the cost gradient and the Gauss-Newton polish that refines
// the swarm's best (the paper's Local Minimization step).
// ---------------------------------------------------------------------------

// Thread placement of the sensitivity kernels: SINGLE and BATCH as locate
// (one problem per workgroup); PACKED, one (problem, particle) pair per
// thread from L, so that a wave can hold the candidates of several problems.
// Returns false for a thread with nothing to do (past the lanes, or its
// problem inactive; uniform over the workgroup unless PACKED). blk is the
// PACKED workgroup's index among the lanes' workgroups.
enum { PLACE_SINGLE = 0, PLACE_BATCH = 1, PLACE_PACKED = 2 };

template <int BS, int PLACE>
__device__ __forceinline__ bool place(const ProbDesc &d0, const SwarmArrays &B, const Lanes &L,
                                      int64_t blk, int64_t &p, int64_t &i, const ProbDesc *&D)
{
    if (PLACE == PLACE_PACKED) {
        const int64_t q = blk * BS + threadIdx.x;
        if (q >= (L.count ? *L.count : L.n)) return false;
        p = L.pairs[2 * q];
        i = L.pairs[2 * q + 1];
        D = &B.desc[p];
    } else {
        int64_t tile;
        D = &locate<PLACE == PLACE_SINGLE>(d0, B, p, tile);
        i = tile * BS + threadIdx.x;
    }
    return !(B.active && !B.active[p]);
}

// Gravity-plus-centrifugal block of the Jacobian at s, in factored form:
// d a/d r = diag(1, 1, 0) - cs I + e1 p1 p1^T + e2 p2 p2^T with
// p_j = (x - x_j, y, z), cs = c1 + c2, e_j = 3 c_j / r_j^2.
struct JacData {
    double cs, e1, e2, d1, d2, y, z;
};

// 1 / b from the hardware's reciprocal: the instruction sequence the compiler
// emits for the division, without operand rescaling and special-value fixups
// (two Newton steps and a corrected quotient).
__device__ __forceinline__ double rcp_inrange(double b)
{
    double r = __builtin_amdgcn_rcp(b);
    double e = fma(-b, r, 1.0);
    r = fma(r, e, r);
    e = fma(-b, r, 1.0);
    r = fma(r, e, r);
    e = fma(-b, r, 1.0);
    return fma(e, r, r);
}

// f(s) exactly as the propagation's right-hand side computes it (rhs: one
// reciprocal R = 1/(D1 D2), D_j = r_j^2 sqrt(r_j^2), correctly rounded sqrt
// and reciprocal; INRANGE selects the in-range sequences; returns the mark
// for their certificate), and the Jacobian data at s from the same intermediates:
// c1 = (1-mu) D2 R, c2 = mu D1 R, and, since D2 R = 1 / (r1^2 sqrt(r1^2)),
// 1 / r1^2 = sqrt(r1^2) D2 R, so e1 = 3 c1 sqrt(r1^2) (D2 R) and likewise
// e2, with no further square root or division. ROOTS: the reciprocal from the
// inverse roots (as rhs), else from the hardware's seed, which frees the roots
// early: the one-thread tangent sweep, at its register limit, is 3% faster
// with it (65,536 particles over 2,000 steps: 4.20 against 4.35 ms). That one is
// the compiler's own sequence for every D in the range, so its mark carries no
// residual; a D below the range shows in its NaN (Cert).
template <bool INRANGE, bool ROOTS>
__device__ __forceinline__ Mark rhs_jac(double mu, double mu1, const double s[6], double f[6],
                                        JacData &J)
{
    const double x = s[0], y = s[1], z = s[2], vx = s[3], vy = s[4];
    const double d1 = x + mu;
    const double d2 = x - mu1;
    const double q = fma(z, z, y * y);
    const double r1s = fma(d1, d1, q);
    const double r2s = fma(d2, d2, q);
    double h1 = 0.0, h2 = 0.0;
    const double q1 = INRANGE ? sqrt_inrange(r1s, h1) : sqrt(r1s);
    const double q2 = INRANGE ? sqrt_inrange(r2s, h2) : sqrt(r2s);
    const double D1 = r1s * q1;
    const double D2 = r2s * q2;
    const double D = D1 * D2;
    double e = 0.0;
    const double R = !INRANGE ? 1.0 / D : ROOTS ? rcp_from_roots(D, h1, h2, e) : rcp_inrange(D);
    const double i1 = D2 * R, i2 = D1 * R;
    const double c1 = mu1 * i1;
    const double c2 = mu * i2;
    const double cs = c1 + c2;
    f[0] = s[3];
    f[1] = s[4];
    f[2] = s[5];
    f[3] = fma(-c2, d2, fma(-c1, d1, fma(2.0, vy, x)));
    f[4] = fma(-cs, y, fma(-2.0, vx, y));
    f[5] = -(cs * z);
    J.cs = cs;
    J.e1 = 3.0 * c1 * (q1 * i1);
    J.e2 = 3.0 * c2 * (q2 * i2);
    J.d1 = d1;
    J.d2 = d2;
    J.y = y;
    J.z = z;
    return {D, e};
}

// G u for the symmetric gravity block.
__device__ __forceinline__ void gmul(const JacData &J, const double u[3], double out[3])
{
    const double p1 = fma(J.d1, u[0], fma(J.y, u[1], J.z * u[2]));
    const double p2 = fma(J.d2, u[0], fma(J.y, u[1], J.z * u[2]));
    const double a1 = J.e1 * p1, a2 = J.e2 * p2, a12 = a1 + a2;
    out[0] = fma(a1, J.d1, fma(a2, J.d2, u[0] - J.cs * u[0]));
    out[1] = fma(a12, J.y, u[1] - J.cs * u[1]);
    out[2] = fma(a12, J.z, -J.cs * u[2]);
}

// A(s) u (tangent) and A(s)^T v (cotangent); A = [[0, I], [G, W]], W the
// Coriolis block [[0, 2, 0], [-2, 0, 0], [0, 0, 0]].
__device__ __forceinline__ void amul(const JacData &J, const double u[6], double out[6])
{
    double g[3];
    gmul(J, u, g);
    out[0] = u[3];
    out[1] = u[4];
    out[2] = u[5];
    out[3] = fma(2.0, u[4], g[0]);
    out[4] = fma(-2.0, u[3], g[1]);
    out[5] = g[2];
}

__device__ __forceinline__ void atmul(const JacData &J, const double v[6], double out[6])
{
    double g[3];
    gmul(J, v + 3, g);
    out[0] = g[0];
    out[1] = g[1];
    out[2] = g[2];
    out[3] = fma(-2.0, v[4], v[0]);
    out[4] = fma(2.0, v[3], v[1]);
    out[5] = v[2];
}

// Jacobian data at the four stage inputs X, s2, s3, s4 of one RK4 step of
// size h from X, and optionally the stepped state Y. INRANGE as in rhs_jac;
// the stage inputs are those of the propagation bit for bit wherever the
// result is certified.
template <bool INRANGE, bool ROOTS>
__device__ __forceinline__ void stages_jac(double mu, double mu1, double h, double h2, double h6,
                                           const double X[6], JacData J[4], double *Y, Cert &cert)
{
    double k[6], a[6], s[6];
    Mark m = rhs_jac<INRANGE, ROOTS>(mu, mu1, X, k, J[0]);
#pragma unroll
    for (int d = 0; d < 6; ++d) {
        a[d] = k[d];
        s[d] = fma(h2, k[d], X[d]);
    }
    cert.add(m, rhs_jac<INRANGE, ROOTS>(mu, mu1, s, k, J[1]));
#pragma unroll
    for (int d = 0; d < 6; ++d) {
        a[d] = fma(2.0, k[d], a[d]);
        s[d] = fma(h2, k[d], X[d]);
    }
    m = rhs_jac<INRANGE, ROOTS>(mu, mu1, s, k, J[2]);
#pragma unroll
    for (int d = 0; d < 6; ++d) {
        a[d] = fma(2.0, k[d], a[d]);
        s[d] = fma(h, k[d], X[d]);
    }
    cert.add(m, rhs_jac<INRANGE, ROOTS>(mu, mu1, s, k, J[3]));
    if (Y) {
#pragma unroll
        for (int d = 0; d < 6; ++d) Y[d] = fma(h6, a[d] + k[d], X[d]);
    }
}

// The same with the in-range sequences where the whole wave is certified,
// else on the IEEE path (as rk4 does).
template <bool ROOTS = true>
__device__ __forceinline__ void stages_jac(double mu, double mu1, bool fast, double h, double h2,
                                           double h6, const double X[6], JacData J[4], double *Y)
{
    bool ok = false;
    if (fast) {
        Cert cert;
        stages_jac<true, ROOTS>(mu, mu1, h, h2, h6, X, J, Y, cert);
        // (a NaN of stage 1 or 2 reaches the position of stage 3 or 4)
        ok = cert.ok(Y ? Y[5] : J[2].cs + J[3].cs);
    }
    if (!__all(ok)) {
        Cert ieee;
        stages_jac<false, ROOTS>(mu, mu1, h, h2, h6, X, J, Y, ieee);
    }
}

// Reverse (transposed tangent) of one RK4 step with stage Jacobians J:
// lam <- (dX'/dX)^T lam.
// X' = X + h/6 (k1 + 2 k2 + 2 k3 + k4), s2 = X + h/2 k1, s3 = X + h/2 k2, s4 = X + h k3.
__device__ __forceinline__ void rk4_vjp_apply(const JacData J[4], double h, double h2, double h6,
                                              double lam[6])
{
    double kb[6], sb[6], xb[6];
#pragma unroll
    for (int d = 0; d < 6; ++d) kb[d] = h6 * lam[d];
    atmul(J[3], kb, sb);
#pragma unroll
    for (int d = 0; d < 6; ++d) {
        xb[d] = lam[d] + sb[d];
        kb[d] = fma(2.0 * h6, lam[d], h * sb[d]);
    }
    atmul(J[2], kb, sb);
#pragma unroll
    for (int d = 0; d < 6; ++d) {
        xb[d] += sb[d];
        kb[d] = fma(2.0 * h6, lam[d], h2 * sb[d]);
    }
    atmul(J[1], kb, sb);
#pragma unroll
    for (int d = 0; d < 6; ++d) {
        xb[d] += sb[d];
        kb[d] = fma(h6, lam[d], h2 * sb[d]);
    }
    atmul(J[0], kb, sb);
#pragma unroll
    for (int d = 0; d < 6; ++d) lam[d] = xb[d] + sb[d];
}

// The same for a step taken from X.
__device__ __forceinline__ void rk4_vjp(double mu, double mu1, bool fast, double h,
                                        const double X[6], double lam[6])
{
    const double h2 = 0.5 * h, h6 = h / 6.0;
    JacData J[4];
    stages_jac(mu, mu1, fast, h, h2, h6, X, J, nullptr);
    rk4_vjp_apply(J, h, h2, h6, lam);
}

// Residuals and their gradients with respect to rho at one observation row;
// returns false when rho = 0 (no line of sight).
//   d(da)/d rho = (rho_y, -rho_x, 0) / rho_xy^2
//   d(db)/d rho = (rho_z rho_x / rho_xy, rho_z rho_y / rho_xy, -rho_xy) / |rho|^2
//   d(dr)/d rho = -rho / |rho|   (range residual dr = observed - |rho|, only
//                                 when the problem has ranges)
__device__ __forceinline__ bool residual_and_grad(const double *row, const double S[6],
                                                  double &da, double &db, double ga[3],
                                                  double gb[3], bool ranged, double &dr,
                                                  double gr[3])
{
    const double rx = S[0] - row[TAB_RC + 0];
    const double ry = S[1] - row[TAB_RC + 1];
    const double rz = S[2] - row[TAB_RC + 2];
    if (rx == 0.0 && ry == 0.0 && rz == 0.0) return false;
    const double sa = row[TAB_SA], ca = row[TAB_CA], sb = row[TAB_SB], cb = row[TAB_CB];
    const double rxy2 = fma(rx, rx, ry * ry);
    const double rxy = sqrt(rxy2);
    double na = sa, nd = ca;
    if (rxy != 0.0) {
        na = fma(sa, rx, -(ca * ry));
        nd = fma(ca, rx, sa * ry);
    }
    da = atan2(na, nd);
    db = atan2(fma(sb, rxy, -(cb * rz)), fma(cb, rxy, sb * rz));
    const double r2 = fma(rz, rz, rxy2);
    ga[0] = ry / rxy2;
    ga[1] = -rx / rxy2;
    ga[2] = 0.0;
    gb[0] = rz * rx / rxy / r2;
    gb[1] = rz * ry / rxy / r2;
    gb[2] = -rxy / r2;
    if (ranged) {
        const double r = sqrt(fma(rx, rx, fma(ry, ry, rz * rz)));
        dr = row[TAB_RANGE] - r;
        gr[0] = -rx / r;
        gr[1] = -ry / r;
        gr[2] = -rz / r;
    }
    return true;
}

// Cotangent of observation k's cost term with respect to the state the
// observation is taken from (X on the grid; a partial step tau is reversed).
__device__ __forceinline__ void obs_cotangent(const KArgs &A, const double *row, const double X[6],
                                              double add[6])
{
    const double tau = row[TAB_TAU];
    double S[6];
#pragma unroll
    for (int d = 0; d < 6; ++d) S[d] = X[d];
    if (tau != 0.0) rk4<false>(A.mu, A.mu1, A.fast, tau, 0.5 * tau, tau / 6.0, S);
    double da = 0, db = 0, ga[3], gb[3], dr = 0, gr[3] = {0, 0, 0};
    double sbar[6] = {0, 0, 0, 0, 0, 0};
    const bool ranged = A.wr != 0.0;
    if (residual_and_grad(row, S, da, db, ga, gb, ranged, dr, gr)) {
        double e = A.w * fma(da, da, db * db);
        if (ranged) e = fma(A.wr * dr, dr, e);
        const double gp = (A.mode == 1 ? 1.0 : 2.0 * e) * 2.0;
#pragma unroll
        for (int d = 0; d < 3; ++d)
            sbar[d] = gp * fma(A.wr * dr, gr[d], A.w * fma(da, ga[d], db * gb[d]));
    } else {
#pragma unroll
        for (int d = 0; d < 3; ++d) sbar[d] = NAN;
    }
    if (tau != 0.0) rk4_vjp(A.mu, A.mu1, A.fast, tau, X, sbar);
#pragma unroll
    for (int d = 0; d < 6; ++d) add[d] = sbar[d];
}

constexpr int CKPT = ADJ_CKPT;   // steps between adjoint checkpoints (the host sizes the scratch with it)

// Cost and its gradient by the discrete adjoint. Forward: the certified
// propagation and cost (same bits as k_eval), checkpoints X_{64 j}. Reverse:
// per 64-step segment, recompute the states from the checkpoint into
// scratch, then sweep back applying the transposed RK4 step and adding each
// observation's cotangent at its grid index. Scratch per lane (column g of
// a [rows][6][wld] array): rows [0, nseg) checkpoints, [nseg, nseg + 64)
// segment states. mode >= 0 overrides the cost mode.
template <int BS, int PLACE>
__device__ __forceinline__ void grad_body(int64_t blk, const ProbDesc &d0, const SwarmArrays &B,
                                          const Lanes &L, double *__restrict__ grad,
                                          double *__restrict__ work, int64_t wld, int32_t mode)
{
    int64_t p, i;
    const ProbDesc *Dp;
    if (!place<BS, PLACE>(d0, B, L, blk, p, i, Dp)) return;
    const ProbDesc &D = *Dp;
    KArgs A = D.k;
    if (mode >= 0) A.mode = mode;
    const bool valid = i < D.m;
    const int64_t g = D.off + (valid ? i : D.m - 1);
    const int32_t S = A.ns[A.K - 1];
    const int32_t nseg = (S + CKPT - 1) / CKPT;
    // private scratch column: invalid lanes alias the last valid particle's
    // column but only ever read what they wrote themselves in lockstep
    double *ck = work;
    double *seg = work + (int64_t)nseg * 6 * wld;
    double X[6];
    load_state(B.x, B.ld, g, X);
    double J = 0.0;
    CostAcc acc{0.0, A.w, A.mode, A.wr};
    // k: next observation, nk: the step it is taken after (-1 past the last)
    int32_t k = 0, nk = A.ns[0];
    for (int32_t n = 0; n <= S; ++n) {
        if (n < S && n % CKPT == 0 && valid) {
#pragma unroll
            for (int d = 0; d < 6; ++d) ck[((int64_t)(n / CKPT) * 6 + d) * wld + g] = X[d];
        }
        while (nk == n) {
            const double *row = A.tab + (int64_t)k * TAB_W;
            double Sx[6];
#pragma unroll
            for (int d = 0; d < 6; ++d) Sx[d] = X[d];
            const double tau = row[TAB_TAU];
            if (tau != 0.0) rk4<false>(A.mu, A.mu1, A.fast, tau, 0.5 * tau, tau / 6.0, Sx);
            acc(row, Sx);
            ++k;
            nk = k < A.K ? A.ns[k] : -1;
        }
        if (n < S) rk4<true>(A.mu, A.mu1, A.fast, A.h, A.h2, A.h6, X);
    }
    J = acc.J;
    // reverse sweep
    double lam[6] = {0, 0, 0, 0, 0, 0};
    k = A.K - 1;
    nk = A.ns[k];
    while (nk == S) {
        double add[6];
        obs_cotangent(A, A.tab + (int64_t)k * TAB_W, X, add);
#pragma unroll
        for (int d = 0; d < 6; ++d) lam[d] += add[d];
        --k;
        nk = k >= 0 ? A.ns[k] : -1;
    }
    for (int32_t sg = nseg - 1; sg >= 0; --sg) {
        const int32_t a = sg * CKPT, b = min(a + CKPT, S);
        double Y[6];
#pragma unroll
        for (int d = 0; d < 6; ++d) Y[d] = valid ? ck[((int64_t)sg * 6 + d) * wld + g] : X[d];
        // the segment's states, stored as they are reached: the in-range
        // sequences with one certification vote for the segment (as
        // rk4_steps), and the whole segment again on the IEEE path if a lane
        // is not certified
        bool ok = false;
        if (A.fast) {
            double Z[6];
#pragma unroll
            for (int d = 0; d < 6; ++d) Z[d] = Y[d];
            Cert cert;
#pragma unroll 2
            for (int32_t j = a; j < b; ++j) {
                if (valid) {
#pragma unroll
                    for (int d = 0; d < 6; ++d) seg[((int64_t)(j - a) * 6 + d) * wld + g] = Z[d];
                }
                if (j + 1 < b) {
                    double q[6];
                    rk4_sum<true>(A.mu, A.mu1, A.h, A.h2, Z, q, cert);
#pragma unroll
                    for (int d = 0; d < 6; ++d) Z[d] = fma(A.h6, q[d], Z[d]);
                }
            }
            ok = b - a < 2 || cert.ok(Z[5]);
        }
        if (!__all(ok)) {
            for (int32_t j = a; j < b; ++j) {
                if (valid) {
#pragma unroll
                    for (int d = 0; d < 6; ++d) seg[((int64_t)(j - a) * 6 + d) * wld + g] = Y[d];
                }
                if (j + 1 < b) {
                    double q[6];
                    Cert ieee;
                    rk4_sum<false>(A.mu, A.mu1, A.h, A.h2, Y, q, ieee);
#pragma unroll
                    for (int d = 0; d < 6; ++d) Y[d] = fma(A.h6, q[d], Y[d]);
                }
            }
        }
        // each step's state is loaded one step ahead, while the step after it
        // is reversed, so the sweep does not wait for the load
        double Xn[6];
#pragma unroll
        for (int d = 0; d < 6; ++d) Xn[d] = valid ? seg[((int64_t)(b - 1 - a) * 6 + d) * wld + g] : X[d];
        for (int32_t j = b - 1; j >= a; --j) {
            double Xj[6];
#pragma unroll
            for (int d = 0; d < 6; ++d) Xj[d] = Xn[d];
            if (j > a) {
#pragma unroll
                for (int d = 0; d < 6; ++d)
                    Xn[d] = valid ? seg[((int64_t)(j - 1 - a) * 6 + d) * wld + g] : X[d];
            }
            rk4_vjp(A.mu, A.mu1, A.fast, A.h, Xj, lam);
            while (nk == j) {
                double add[6];
                obs_cotangent(A, A.tab + (int64_t)k * TAB_W, Xj, add);
#pragma unroll
                for (int d = 0; d < 6; ++d) lam[d] += add[d];
                --k;
                nk = k >= 0 ? A.ns[k] : -1;
            }
        }
    }
    if (valid) {
        B.cost[D.off + i] = J;
#pragma unroll
        for (int d = 0; d < 6; ++d) grad[d * B.ld + D.off + i] = lam[d];
    }
}

template <int BS, int PLACE>
__global__ __launch_bounds__(BS) void k_grad(ProbDesc d0, SwarmArrays B, Lanes L,
                                             double *__restrict__ grad, double *__restrict__ work,
                                             int64_t wld, int32_t mode)
{
    grad_body<BS, PLACE>(blockIdx.x, d0, B, L, grad, work, wld, mode);
}

// Forward tangent (6x6 state transition matrix of the discrete RK4 map) and
// the Gauss-Newton normal equations of the whitened residuals
// r = (da, db) / sigma: chi2 = sum r^2, N = J^T J (21 packed, row-major
// upper triangle), jtr = J^T r.
// The gravity-plus-centrifugal block G as a matrix (its six distinct
// entries), for products with the six columns of the tangent, where the
// factored form would repeat the projections p_j . u for every column.
struct GMat {
    double g00, g01, g02, g11, g12, g22;
};

__device__ __forceinline__ GMat gmat(const JacData &J)
{
    const double t1 = J.e1 * J.d1, t2 = J.e2 * J.d2;
    const double txy = t1 + t2, ey = J.e1 + J.e2, one_cs = 1.0 - J.cs;
    const double eyy = ey * J.y;
    GMat G;
    G.g00 = fma(t1, J.d1, fma(t2, J.d2, one_cs));
    G.g01 = txy * J.y;
    G.g02 = txy * J.z;
    G.g11 = fma(eyy, J.y, one_cs);
    G.g12 = eyy * J.z;
    G.g22 = fma(ey * J.z, J.z, -J.cs);
    return G;
}

// A(s) u with G given as a matrix.
__device__ __forceinline__ void amul(const GMat &G, const double u[6], double out[6])
{
    const double g0 = fma(G.g00, u[0], fma(G.g01, u[1], G.g02 * u[2]));
    const double g1 = fma(G.g01, u[0], fma(G.g11, u[1], G.g12 * u[2]));
    const double g2 = fma(G.g02, u[0], fma(G.g12, u[1], G.g22 * u[2]));
    out[0] = u[3];
    out[1] = u[4];
    out[2] = u[5];
    out[3] = fma(2.0, u[4], g0);
    out[4] = fma(-2.0, u[3], g1);
    out[5] = g2;
}

// One column u of the tangent through an RK4 step with stage blocks G.
__device__ __forceinline__ void tangent_column(const GMat G[4], double h, double h2, double h6,
                                               double u[6])
{
    double dk[6], acc[6], ds[6];
    amul(G[0], u, dk);
#pragma unroll
    for (int d = 0; d < 6; ++d) {
        acc[d] = dk[d];
        ds[d] = fma(h2, dk[d], u[d]);
    }
    amul(G[1], ds, dk);
#pragma unroll
    for (int d = 0; d < 6; ++d) {
        acc[d] = fma(2.0, dk[d], acc[d]);
        ds[d] = fma(h2, dk[d], u[d]);
    }
    amul(G[2], ds, dk);
#pragma unroll
    for (int d = 0; d < 6; ++d) {
        acc[d] = fma(2.0, dk[d], acc[d]);
        ds[d] = fma(h, dk[d], u[d]);
    }
    amul(G[3], ds, dk);
#pragma unroll
    for (int d = 0; d < 6; ++d) u[d] = fma(h6, acc[d] + dk[d], u[d]);
}

__device__ __forceinline__ void tangent_step(double mu, double mu1, bool fast, double h,
                                             double X[6], double Phi[36])
{
    const double h2 = 0.5 * h, h6 = h / 6.0;
    double Y[6];
    JacData J[4];
    stages_jac<false>(mu, mu1, fast, h, h2, h6, X, J, Y);
    const GMat G[4] = {gmat(J[0]), gmat(J[1]), gmat(J[2]), gmat(J[3])};
#pragma unroll
    for (int c = 0; c < 6; ++c) {
        double u[6];
#pragma unroll
        for (int d = 0; d < 6; ++d) u[d] = Phi[6 * d + c];
        tangent_column(G, h, h2, h6, u);
#pragma unroll
        for (int d = 0; d < 6; ++d) Phi[6 * d + c] = u[d];
    }
#pragma unroll
    for (int d = 0; d < 6; ++d) X[d] = Y[d];
}

template <int BS, int PLACE>
__device__ __forceinline__ void normal_body(int64_t blk, const ProbDesc &d0,
                                            const SwarmArrays &B, const Lanes &L,
                                            double *__restrict__ chi2, double *__restrict__ jtj,
                                            double *__restrict__ jtr, double *__restrict__ jrows,
                                            int64_t jstride, int64_t jld)
{
    int64_t p, i;
    const ProbDesc *Dp;
    if (!place<BS, PLACE>(d0, B, L, blk, p, i, Dp)) return;
    const ProbDesc &D = *Dp;
    const KArgs &A = D.k;
    const bool valid = i < D.m;
    const int64_t g = D.off + (valid ? i : D.m - 1);
    const double is = sqrt(A.w);   // 1 / sigma
    const bool ranged = A.wr != 0.0;
    const double isr = sqrt(A.wr); // 1 / sigma_range
    double X[6], Phi[36];
    load_state(B.x, B.ld, g, X);
#pragma unroll
    for (int d = 0; d < 36; ++d) Phi[d] = (d % 7 == 0) ? 1.0 : 0.0;
    double c2 = 0.0, N[21], gr[6];
#pragma unroll
    for (int d = 0; d < 21; ++d) N[d] = 0.0;
#pragma unroll
    for (int d = 0; d < 6; ++d) gr[d] = 0.0;
    const int32_t S = A.ns[A.K - 1];
    // k: next observation, nk: the step it is taken after (-1 past the last)
    int32_t k = 0, nk = A.ns[0];
    for (int32_t n = 0; n <= S; ++n) {
        while (nk == n) {
            const double *row = A.tab + (int64_t)k * TAB_W;
            double Sx[6], SP[36];
#pragma unroll
            for (int d = 0; d < 6; ++d) Sx[d] = X[d];
#pragma unroll
            for (int d = 0; d < 36; ++d) SP[d] = Phi[d];
            const double tau = row[TAB_TAU];
            if (tau != 0.0) tangent_step(A.mu, A.mu1, A.fast, tau, Sx, SP);
            double da, db, ga[3], gb[3], dr = 0, gq[3] = {0, 0, 0};
            if (!residual_and_grad(row, Sx, da, db, ga, gb, ranged, dr, gq)) {
                da = db = dr = NAN;
                ga[0] = ga[1] = ga[2] = gb[0] = gb[1] = gb[2] = gq[0] = gq[1] = gq[2] = NAN;
            }
            double ja[6], jb[6], jr[6];
#pragma unroll
            for (int c = 0; c < 6; ++c) {
                ja[c] = is * fma(ga[0], SP[c], fma(ga[1], SP[6 + c], ga[2] * SP[12 + c]));
                jb[c] = is * fma(gb[0], SP[c], fma(gb[1], SP[6 + c], gb[2] * SP[12 + c]));
                jr[c] = isr * fma(gq[0], SP[c], fma(gq[1], SP[6 + c], gq[2] * SP[12 + c]));
            }
            if (jrows && valid) {
                // rows of J for this observation: (k R + r) 6 + c, column p jstride + i
                const int R = ranged ? 3 : 2;
                double *q = jrows + (int64_t)k * R * 6 * jld + p * jstride + i;
#pragma unroll
                for (int c = 0; c < 6; ++c) {
                    q[c * jld] = ja[c];
                    q[(6 + c) * jld] = jb[c];
                    if (ranged) q[(12 + c) * jld] = jr[c];
                }
            }
            const double ra = da * is, rb = db * is, rr = dr * isr;
            c2 = fma(ra, ra, fma(rb, rb, c2));
            int t = 0;
#pragma unroll
            for (int r = 0; r < 6; ++r) {
                gr[r] = fma(ja[r], ra, fma(jb[r], rb, gr[r]));
#pragma unroll
                for (int c = r; c < 6; ++c, ++t) N[t] = fma(ja[r], ja[c], fma(jb[r], jb[c], N[t]));
            }
            if (ranged) {
                c2 = fma(rr, rr, c2);
                t = 0;
#pragma unroll
                for (int r = 0; r < 6; ++r) {
                    gr[r] = fma(jr[r], rr, gr[r]);
#pragma unroll
                    for (int c = r; c < 6; ++c, ++t) N[t] = fma(jr[r], jr[c], N[t]);
                }
            }
            ++k;
            nk = k < A.K ? A.ns[k] : -1;
        }
        if (n < S) tangent_step(A.mu, A.mu1, A.fast, A.h, X, Phi);
    }
    if (valid) {
        const int64_t o = D.off + i;
        chi2[o] = c2;
#pragma unroll
        for (int d = 0; d < 21; ++d) jtj[d * B.ld + o] = N[d];
#pragma unroll
        for (int d = 0; d < 6; ++d) jtr[d * B.ld + o] = gr[d];
    }
}

// The single problem's instances of the sweep are fastest when their step loop
// starts on a multiple of 8 bytes: 65,536 particles over 2,000 steps 4.05-4.08 ms,
// and 4.10-4.20 at the offsets between, with the same instructions; the padding
// puts them there (the placement test names one that has left).
template <int BS, int PLACE>
__global__ __launch_bounds__(BS) void k_normal(ProbDesc d0, SwarmArrays B, Lanes L,
                                               double *__restrict__ chi2, double *__restrict__ jtj,
                                               double *__restrict__ jtr, double *__restrict__ jrows,
                                               int64_t jstride, int64_t jld)
{
    if constexpr (PLACE == PLACE_SINGLE) entry_pad<1>();
    normal_body<BS, PLACE>(blockIdx.x, d0, B, L, chi2, jtj, jtr, jrows, jstride, jld);
}

// The normal equations (NB) and the adjoint gradient (GB) of the same packed
// lanes in one launch: even workgroups take the tangent sweep of lane block
// blockIdx.x / 2, odd ones the adjoint sweep of that block. When few lanes
// are live, the two sweeps of a block then run side by side on different
// SIMDs instead of one launch after the other.
__global__ __launch_bounds__(64) void k_normal_grad(ProbDesc d0, SwarmArrays NB, SwarmArrays GB,
                                                    Lanes L, double *__restrict__ chi2,
                                                    double *__restrict__ jtj,
                                                    double *__restrict__ jtr,
                                                    double *__restrict__ jrows, int64_t jstride,
                                                    int64_t jld, double *__restrict__ grad,
                                                    double *__restrict__ work, int64_t wld,
                                                    int32_t mode, Gate G)
{
    if (closed(G)) return;
    const int64_t blk = blockIdx.x >> 1;
    if (blockIdx.x & 1)
        grad_body<64, PLACE_PACKED>(blk, d0, GB, L, grad, work, wld, mode);
    else
        normal_body<64, PLACE_PACKED>(blk, d0, NB, L, chi2, jtj, jtr, jrows, jstride, jld);
}

// ---------------------------------------------------------------------------
// Pipelined sensitivities: the sweeps above for few particles. One thread per
// particle carries the state, its stage Jacobians and the six tangent columns
// (about 1,170 issue slots per RK4 step), or steps forward, again per segment,
// and once more per reversed step (1,460), while most SIMDs idle. Here a
// workgroup holds PIPE_P particles and its waves share the work of each step
// through LDS:
//   - wave 0 propagates the states, four lanes per particle: about 172 slots
//     per step, and 25 cycles for every LDS write, whatever its width;
//   - for the tangent it leaves the stages' positions (two writes a step), which
//     wave 3 turns into gravity blocks, one lane per particle and stage, a chunk
//     of steps behind, and two waves carry the tangent another chunk behind, one
//     lane per column (eight lanes per particle, six in use): about 75 slots;
//   - for the adjoint it leaves the stages' Jacobian data itself (six writes),
//     going back segment by segment: it recomputes the segment's steps from the
//     checkpoint while wave 1 applies the transposed steps of the segment after
//     it, in reverse order.
// Each operation on a particle is the one of the sweeps above, on the same
// operands, so the bits are the same. 96 particles over 2,520 steps: normal
// equations 5.02 -> 1.01 ms (1.13 with the Jacobian data from the producer and
// the blocks formed by every column); 1,000 over 2,000: cost gradient 5.03 ->
// 1.58 ms. Wave 0 bounds both, with its hand-over (a barrier every 8 steps and
// the wait for LDS); longer chunks, packed writes and reading a step ahead
// gained nothing. A workgroup's LDS (76 to 140 KB) lets one or two share a
// compute unit, so with more particles than the host's rule allows the other
// sweeps win.
// ---------------------------------------------------------------------------

// One step in LDS, PIPE_STEP double2: per stage the position (x, y), (z, cs) and
// (e1, e2) of each particle, then the velocity at the step's start.

// Stage data of the own stage, from the lanes of each particle.
struct PipeSink {
    static constexpr bool JAC = true;
    double2 *own;   // the particle's entry at the own stage of half 0
    int prim;
    __device__ __forceinline__ void operator()(int half, const double *q, const Attraction &o)
    {
        double2 *s = own + half * (6 * PIPE_P);
        s[0] = make_double2(q[0], q[1]);
        s[PIPE_P] = make_double2(q[2], o.cs);
        ((double *)(s + 2 * PIPE_P))[prim] = o.ej;
    }
};

// Positions of the own stage only: (x, y) by the lane of primary 1, z by the other.
struct PosSink {
    static constexpr bool JAC = false;
    double2 *own;   // the lane's entry at the own stage of half 0
    bool second;
    __device__ __forceinline__ void operator()(int half, const double *q, const Attraction &)
    {
        own[half * (6 * PIPE_P)] = make_double2(second ? q[2] : q[0], q[1]);
    }
};

// n steps from X by the producer wave of the tangent, the positions of their
// stages into slots ring + j PIPE_TSTEP; the vote and the redo as pipe_produce.
__device__ __forceinline__ void pipe_positions(const KArgs &A, int32_t n, double X[6],
                                               double2 *ring, int pp)
{
    if (A.fast) {
        double X0[6];
#pragma unroll
        for (int d = 0; d < 6; ++d) X0[d] = X[d];
        Cert cert;
        const int j = threadIdx.x & 1;
        PosSink sink{ring + (Quad<4>::is_late() ? 3 * PIPE_P : 0) + j * PIPE_P + pp, j != 0};
        auto step = [&]() __attribute__((always_inline)) {
            split_step<4>(A.mu, A.mu1, A.h, A.h2, A.h6, X, cert, sink);
            sink.own += PIPE_TSTEP;
        };
        int32_t i = 0;
        for (; i + 4 <= n; i += 4) {
            step();
            step();
            step();
            step();
        }
        for (; i < n; ++i) step();
        if (__all(cert.ok(X[5]))) return;
#pragma unroll
        for (int d = 0; d < 6; ++d) X[d] = X0[d];
    }
    for (int32_t j = 0; j < n; ++j) {
        double a[6], k[6], s[6];
#pragma unroll
        for (int d = 0; d < 6; ++d) s[d] = X[d];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            double2 *q = ring + j * PIPE_TSTEP + 3 * i * PIPE_P + pp;
            q[0] = make_double2(s[0], s[1]);
            q[PIPE_P] = make_double2(s[2], 0.0);
            rhs<false>(A.mu, A.mu1, s, k);
#pragma unroll
            for (int d = 0; d < 6; ++d) {
                a[d] = i == 0 ? k[d] : i < 3 ? fma(2.0, k[d], a[d]) : a[d] + k[d];
                if (i < 3) s[d] = fma(i == 2 ? A.h : A.h2, k[d], X[d]);
            }
        }
#pragma unroll
        for (int d = 0; d < 6; ++d) X[d] = fma(A.h6, a[d], X[d]);
    }
}

// The positions of n steps in ring become their gravity blocks in place, one
// lane per particle and stage: (g00, g01), (g02, g11), (g12, g22). A step with a
// lane that is not certified takes the IEEE path.
__device__ __forceinline__ void pipe_jacobians(const KArgs &A, int32_t n, double2 *ring)
{
    const int lane = (int)(threadIdx.x & 63);
    double2 *cell = ring + 3 * (lane / PIPE_P) * PIPE_P + lane % PIPE_P;
    for (int32_t j = 0; j < n; ++j, cell += PIPE_TSTEP) {
        const double2 xy = cell[0];
        const double s[6] = {xy.x, xy.y, cell[PIPE_P].x, 0.0, 0.0, 0.0};
        double f[6];
        JacData J;
        Cert cert;
        if (A.fast) {
            const Mark m = rhs_jac<true, true>(A.mu, A.mu1, s, f, J);
            cert.add(m, m);
        }
        if (!A.fast || !__all(cert.ok(J.cs))) rhs_jac<false, true>(A.mu, A.mu1, s, f, J);
        const GMat G = gmat(J);
        cell[0] = make_double2(G.g00, G.g01);
        cell[PIPE_P] = make_double2(G.g02, G.g11);
        cell[2 * PIPE_P] = make_double2(G.g12, G.g22);
    }
}

__device__ __forceinline__ void pipe_put_velocity(double2 *slot, int pp, const double X[6])
{
    if ((threadIdx.x & 3) == 0) {
        slot[12 * PIPE_P + pp] = make_double2(X[3], X[4]);
        ((double *)(slot + 13 * PIPE_P))[pp] = X[5];
    }
}

// n steps from X by the producer wave, their stage data into slots
// ring + j PIPE_STEP. As rk4_steps: one certification vote, and all n again on
// the IEEE path where a lane is not certified. vel: the steps' velocities are
// wanted too (by the partial steps of a reverse sweep).
__device__ __forceinline__ void pipe_produce(const KArgs &A, int32_t n, double X[6], double2 *ring,
                                             int pp, bool vel)
{
    if (A.fast) {
        double X0[6];
#pragma unroll
        for (int d = 0; d < 6; ++d) X0[d] = X[d];
        Cert cert;
        PipeSink sink{ring + (Quad<4>::is_late() ? 3 * PIPE_P : 0) + pp, (int)(threadIdx.x & 1)};
        double2 *slot = ring;
        auto step = [&]() __attribute__((always_inline)) {
            if (vel) pipe_put_velocity(slot, pp, X);
            split_step<4>(A.mu, A.mu1, A.h, A.h2, A.h6, X, cert, sink);
            sink.own += PIPE_STEP;
            slot += PIPE_STEP;
        };
        int32_t j = 0;
        for (; j + 4 <= n; j += 4) {
            step();
            step();
            step();
            step();
        }
        for (; j < n; ++j) step();
        if (__all(cert.ok(X[5]))) return;
#pragma unroll
        for (int d = 0; d < 6; ++d) X[d] = X0[d];
    }
    for (int32_t j = 0; j < n; ++j) {
        double2 *slot = ring + j * PIPE_STEP;
        JacData J[4];
        double Y[6];
        Cert ieee;
        stages_jac<false, true>(A.mu, A.mu1, A.h, A.h2, A.h6, X, J, Y, ieee);
        if (vel) pipe_put_velocity(slot, pp, X);
        // the stages' positions, stepped to once more
        double k[6], s[6];
#pragma unroll
        for (int d = 0; d < 6; ++d) s[d] = X[d];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            double2 *q = slot + 3 * i * PIPE_P + pp;
            q[0] = make_double2(s[0], s[1]);
            q[PIPE_P] = make_double2(s[2], J[i].cs);
            q[2 * PIPE_P] = make_double2(J[i].e1, J[i].e2);
            if (i < 3) {
                rhs<false>(A.mu, A.mu1, s, k);
#pragma unroll
                for (int d = 0; d < 6; ++d) s[d] = fma(i == 2 ? A.h : A.h2, k[d], X[d]);
            }
        }
#pragma unroll
        for (int d = 0; d < 6; ++d) X[d] = Y[d];
    }
}

// Stage data of a step in LDS, for particle pp.
struct PipeRow {
    double2 a[4], b[4], e[4];
    __device__ __forceinline__ void get(const double2 *slot, int pp)
    {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            a[i] = slot[3 * i * PIPE_P + pp];
            b[i] = slot[(3 * i + 1) * PIPE_P + pp];
            e[i] = slot[(3 * i + 2) * PIPE_P + pp];
        }
    }
    __device__ __forceinline__ void jac(const KArgs &A, JacData J[4]) const
    {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            J[i].cs = b[i].y;
            J[i].e1 = e[i].x;
            J[i].e2 = e[i].y;
            J[i].d1 = a[i].x + A.mu;
            J[i].d2 = a[i].x - A.mu1;
            J[i].y = a[i].y;
            J[i].z = b[i].x;
        }
    }
};

// Hand-over state `half` of particle pp.
__device__ __forceinline__ void pipe_put_state(double *xend, int half, int pp, const double X[6])
{
#pragma unroll
    for (int d = 0; d < 6; ++d) xend[(half * 6 + d) * PIPE_P + pp] = X[d];
}

__device__ __forceinline__ void pipe_get_state(const double *xend, int half, int pp, double X[6])
{
#pragma unroll
    for (int d = 0; d < 6; ++d) X[d] = xend[(half * 6 + d) * PIPE_P + pp];
}

// Buffers of the reverse sweep, PIPE_SUB steps each: the segment being
// reversed holds one per block of its steps, the segment before it fills the
// ones that become free. Both waves keep the same account (numbers of four
// bits in a word).
struct PipeBuffers {
    uint64_t cur = 0, next = 0, spare = 0;
    int nspare = 0;
    __device__ __forceinline__ void push(int id)
    {
        spare |= (uint64_t)id << (4 * nspare);
        ++nspare;
    }
    __device__ __forceinline__ int pop()
    {
        --nspare;
        const int id = (int)(spare >> (4 * nspare)) & 15;
        spare &= ~((uint64_t)15 << (4 * nspare));
        return id;
    }
    __device__ __forceinline__ int at(int block) const { return (int)(cur >> (4 * block)) & 15; }
};

// TAN: chi2, J^T J, J^T r (and the rows of J); ADJ: the cost and its gradient;
// either, not both. Outputs and arguments as normal_body and grad_body; Q.sub
// workgroups (block of them: this one) of PIPE_P particles per work entry (one
// problem: per launch). The checkpoints are Q's scratch rows, every Q.seg
// steps; STORED: they are there already (with the state at the last step after
// them), and only the gradient is formed, with no forward sweep.
template <bool SINGLE, bool TAN, bool ADJ, bool STORED = false>
__device__ __forceinline__ void pipe_body(int64_t block, const ProbDesc &d0, const SwarmArrays &B,
                                          const PipeArgs &Q)
{
    static_assert(TAN != ADJ && (ADJ || !STORED), "one sweep");
    extern __shared__ double2 pipe_lds[];
    double *xend = (double *)pipe_lds;
    double2 *ring = pipe_lds + PIPE_XEND;
    // with a gate, B.work lists the active problems
    if (closed(Q.gate) || (Q.gate.count && block >= (int64_t)*Q.gate.count * Q.sub)) return;
    int64_t p = 0, i0 = block * PIPE_P;
    if (!SINGLE) {
        const int64_t w = block / Q.sub;
        p = B.work[2 * w];
        i0 = B.work[2 * w + 1] * (Q.sub * PIPE_P) + (block % Q.sub) * PIPE_P;
    }
    const ProbDesc &D = SINGLE ? d0 : B.desc[p];
    if (i0 >= D.m || (B.active && !B.active[p])) return;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = (int)(threadIdx.x & 63);
    // particle of this thread, and whether its results are wanted
    auto wanted = [&](int64_t i) {
        return i < D.m && !(Q.done && Q.done[D.off + i]) && !(Q.stored && Q.stored[D.off + i] < 0);
    };
    if (!__any(wanted(i0 + (lane & (PIPE_P - 1))))) return;   // the same in every wave
    if (wave > (TAN ? 3 : 1)) return;
    const int pp = wave == 0 ? lane >> 2 : TAN ? (wave - 1) * 8 + (lane >> 3) : lane & (PIPE_P - 1);
    const int64_t i = i0 + pp;
    const int64_t g = D.off + (i < D.m ? i : D.m - 1);
    // column of its checkpoints
    const int64_t cg = STORED && Q.stored[g] >= 0 ? (int64_t)Q.stored[g] : g;
    KArgs A = D.k;
    if (Q.mode >= 0) A.mode = Q.mode;
    const int32_t S = A.ns[A.K - 1];
    const int32_t L = Q.seg, nseg = (S + L - 1) / L;

    // Forward sweep of the tangent: an interval between observations goes in equal
    // chunks of up to PIPE_FWD steps. The waves hand over in lockstep: while chunk
    // c is produced, c - 1 becomes Jacobians and c - 2 moves the tangent.
    struct Chunks {
        int32_t base, extra;
        __device__ __forceinline__ explicit Chunks(int32_t steps)
        {
            const int32_t parts = max(1, (steps + PIPE_FWD - 1) / PIPE_FWD);
            base = steps / parts;
            extra = steps - base * parts;
        }
        __device__ __forceinline__ int32_t next() { return base + (extra-- > 0 ? 1 : 0); }
    };
    auto tslot = [&](int c) { return ring + c * (PIPE_FWD * PIPE_TSTEP); };
    auto after = [](int c) { return c == PIPE_SLOTS - 1 ? 0 : c + 1; };
    if constexpr (STORED) {
        // no forward sweep
    } else if (wave == 0) {
        double X[6];
        load_state(B.x, B.ld, g, X);
        int32_t step = 0;
        int c = 0;
        for (int32_t k = 0; k < A.K; ++k) {
            const int32_t target = A.ns[k];
            Chunks chunks(TAN ? target - step : 0);
            while (step < target) {
                const int32_t n = TAN ? chunks.next() : min(target - step, L - step % L);
                if (ADJ && step % L == 0 && (lane & 3) == 0 && i < D.m) {
#pragma unroll
                    for (int d = 0; d < 6; ++d)
                        Q.work[((int64_t)(step / L) * 6 + d) * Q.wld + g] = X[d];
                }
                if (TAN) {
                    pipe_positions(A, n, X, tslot(c), pp);
                    if (step + n == target) pipe_put_state(xend, c, pp, X);
                    __syncthreads();
                    c = after(c);
                } else {
                    rk4_steps_split<4>(A, n, X);
                }
                step += n;
            }
            if (!TAN) {
                pipe_put_state(xend, k & 1, pp, X);
                __syncthreads();
            }
        }
        __syncthreads();   // (ADJ: the others are done with the forward sweep's data)
        if (!ADJ) return;
    } else if (TAN && wave == 3) {
        int32_t step = 0;
        int c = 0;
        __syncthreads();
        for (int32_t k = 0; k < A.K; ++k) {
            const int32_t target = A.ns[k];
            Chunks chunks(target - step);
            while (step < target) {
                const int32_t n = chunks.next();
                pipe_jacobians(A, n, tslot(c));
                __syncthreads();
                c = after(c);
                step += n;
            }
        }
        return;
    } else if (TAN) {
        const int cl = min(lane & 7, 5);   // column (lanes 6 and 7 repeat the last)
        const double is = sqrt(A.w);       // 1 / sigma
        const bool ranged = A.wr != 0.0;
        const double isr = sqrt(A.wr);     // 1 / sigma_range
        const bool write = wanted(i) && (lane & 7) < 6;
        double u[6], N[6], gr = 0.0, c2 = 0.0;
#pragma unroll
        for (int d = 0; d < 6; ++d) {
            u[d] = d == cl ? 1.0 : 0.0;
            N[d] = 0.0;
        }
        int32_t step = 0;
        int c = 0, last = 0;
        __syncthreads();
        for (int32_t k = 0; k < A.K; ++k) {
            const int32_t target = A.ns[k];
            Chunks chunks(target - step);
            while (step < target) {
                const int32_t n = chunks.next();
                __syncthreads();
                const double2 *slot = tslot(c) + pp;
                for (int32_t j = 0; j < n; ++j, slot += PIPE_TSTEP) {
                    GMat G[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const double2 a = slot[3 * i * PIPE_P], b = slot[(3 * i + 1) * PIPE_P],
                                      d = slot[(3 * i + 2) * PIPE_P];
                        G[i] = GMat{a.x, a.y, b.x, b.y, d.x, d.y};
                    }
                    tangent_column(G, A.h, A.h2, A.h6, u);
                }
                last = c;
                c = after(c);
                step += n;
            }
            // residuals and their rows of J at this observation
            double X[6], su[6];
            if (step == 0)
                load_state(B.x, B.ld, g, X);
            else
                pipe_get_state(xend, last, pp, X);
#pragma unroll
            for (int d = 0; d < 6; ++d) su[d] = u[d];
            const double *row = A.tab + (int64_t)k * TAB_W;
            const double tau = row[TAB_TAU];
            if (tau != 0.0) {
                const double t2 = 0.5 * tau, t6 = tau / 6.0;
                double Y[6];
                JacData J[4];
                stages_jac(A.mu, A.mu1, A.fast, tau, t2, t6, X, J, Y);
                const GMat G[4] = {gmat(J[0]), gmat(J[1]), gmat(J[2]), gmat(J[3])};
                tangent_column(G, tau, t2, t6, su);
#pragma unroll
                for (int d = 0; d < 6; ++d) X[d] = Y[d];
            }
            double da, db, ga[3], gb[3], dr = 0, gq[3] = {0, 0, 0};
            if (!residual_and_grad(row, X, da, db, ga, gb, ranged, dr, gq)) {
                da = db = dr = NAN;
                ga[0] = ga[1] = ga[2] = gb[0] = gb[1] = gb[2] = gq[0] = gq[1] = gq[2] = NAN;
            }
            const double ja = is * fma(ga[0], su[0], fma(ga[1], su[1], ga[2] * su[2]));
            const double jb = is * fma(gb[0], su[0], fma(gb[1], su[1], gb[2] * su[2]));
            const double jr = isr * fma(gq[0], su[0], fma(gq[1], su[1], gq[2] * su[2]));
            if (Q.jrows && write) {
                const int R = ranged ? 3 : 2;
                double *q = Q.jrows + ((int64_t)k * R * 6 + cl) * Q.jld + p * Q.jstride + i;
                q[0] = ja;
                q[6 * Q.jld] = jb;
                if (ranged) q[12 * Q.jld] = jr;
            }
            const double ra = da * is, rb = db * is, rr = dr * isr;
            c2 = fma(ra, ra, fma(rb, rb, c2));
            gr = fma(ja, ra, fma(jb, rb, gr));
#pragma unroll
            for (int r = 0; r < 6; ++r) {
                const int src = (lane & ~7) + r;
                N[r] = fma(__shfl(ja, src, 64), ja, fma(__shfl(jb, src, 64), jb, N[r]));
            }
            if (ranged) {
                c2 = fma(rr, rr, c2);
                gr = fma(jr, rr, gr);
#pragma unroll
                for (int r = 0; r < 6; ++r) N[r] = fma(__shfl(jr, (lane & ~7) + r, 64), jr, N[r]);
            }
        }
        if (write) {
            const int64_t o = D.off + i;
            if (cl == 0) Q.chi2[o] = c2;
            Q.jtr[cl * B.ld + o] = gr;
            // row r of the packed upper triangle starts at r (13 - r) / 2 - r
#pragma unroll
            for (int r = 0; r < 6; ++r)
                if (r <= cl) Q.jtj[(r * (13 - r) / 2 + cl - r) * B.ld + o] = N[r];
        }
        return;
    } else {
        // the cost, an observation behind the producer
        CostAcc acc{0.0, A.w, A.mode, A.wr};
        for (int32_t k = 0; k < A.K; ++k) {
            __syncthreads();
            double X[6];
            pipe_get_state(xend, k & 1, pp, X);
            const double *row = A.tab + (int64_t)k * TAB_W;
            const double tau = row[TAB_TAU];
            if (tau != 0.0) rk4<false>(A.mu, A.mu1, A.fast, tau, 0.5 * tau, tau / 6.0, X);
            acc(row, X);
        }
        if (wanted(i) && lane < PIPE_P) B.cost[D.off + i] = acc.J;
        __syncthreads();
    }
    if constexpr (ADJ) {
        // reverse sweep (waves 0 and 1): blocks of PIPE_SUB steps
        const int32_t nblk = L / PIPE_SUB;
        PipeBuffers F;
        const int32_t last = nseg > 0 ? (S - (nseg - 1) * L + PIPE_SUB - 1) / PIPE_SUB : 0;
        for (int j = nblk; j >= last; --j) F.push(j);
        for (int j = 0; j < last; ++j) F.cur |= (uint64_t)j << (4 * j);
        auto buffer = [&](int id) { return ring + id * (PIPE_SUB * PIPE_STEP); };
        if (wave == 0) {
            bool off = false;
            for (int32_t k = lane; k < A.K; k += 64) off |= A.tab[(int64_t)k * TAB_W + TAB_TAU] != 0.0;
            const bool offgrid = __any(off);
            double X[6];
            auto checkpoint = [&](int32_t sg) {
#pragma unroll
                for (int d = 0; d < 6; ++d) X[d] = Q.work[((int64_t)sg * 6 + d) * Q.wld + cg];
            };
            if (nseg > 0) {
                checkpoint(nseg - 1);
                const int32_t len = S - (nseg - 1) * L;
                for (int32_t j = 0; j < last; ++j)
                    pipe_produce(A, min(PIPE_SUB, len - j * PIPE_SUB), X, buffer(j), pp, offgrid);
            }
            __syncthreads();
            for (int32_t sg = nseg - 1; sg >= 0; --sg) {
                const int32_t nb = sg == nseg - 1 ? last : nblk, nn = sg > 0 ? nblk : 0;
                if (sg > 0) checkpoint(sg - 1);
                F.next = 0;
                for (int32_t t = 0; t < max(nb, nn); ++t) {
                    if (t < nn) {
                        const int id = F.pop();
                        F.next |= (uint64_t)id << (4 * t);
                        pipe_produce(A, PIPE_SUB, X, buffer(id), pp, offgrid);
                    }
                    if (t < nb) F.push(F.at(nb - 1 - t));
                    __syncthreads();
                }
                F.cur = F.next;
            }
            return;
        }
        // wave 1
        const int q = pp;
        double lam[6] = {0, 0, 0, 0, 0, 0};
        int32_t k = A.K - 1, nk = A.ns[k];
        auto observe = [&](int32_t n, const double X[6]) {
            while (nk == n) {
                double add[6];
                obs_cotangent(A, A.tab + (int64_t)k * TAB_W, X, add);
#pragma unroll
                for (int d = 0; d < 6; ++d) lam[d] += add[d];
                --k;
                nk = k >= 0 ? A.ns[k] : -1;
            }
        };
        double X[6];
        if (S == 0) {
            load_state(B.x, B.ld, D.off + (i0 + q < D.m ? i0 + q : D.m - 1), X);
        } else if (STORED) {
#pragma unroll
            for (int d = 0; d < 6; ++d) X[d] = Q.work[((int64_t)nseg * 6 + d) * Q.wld + cg];
        } else {
            // the state at S: the forward sweep's last hand-over
            pipe_get_state(xend, (A.K - 1) & 1, q, X);
        }
        observe(S, X);
        __syncthreads();
        for (int32_t sg = nseg - 1; sg >= 0; --sg) {
            const int32_t a = sg * L, len = min(L, S - a);
            const int32_t nb = sg == nseg - 1 ? last : nblk, nn = sg > 0 ? nblk : 0;
            F.next = 0;
            for (int32_t t = 0; t < max(nb, nn); ++t) {
                if (t < nn) F.next |= (uint64_t)F.pop() << (4 * t);
                if (t < nb) {
                    const int32_t blk = nb - 1 - t;
                    const double2 *buf = buffer(F.at(blk));
                    auto reverse = [&](const PipeRow &r, int32_t j) {
                        JacData J[4];
                        r.jac(A, J);
                        rk4_vjp_apply(J, A.h, A.h2, A.h6, lam);
                        const int32_t n = a + blk * PIPE_SUB + j;
                        if (nk == n) {
                            const double2 *slot = buf + j * PIPE_STEP;
                            // (written where some observation is off the grid)
                            const double2 v = slot[12 * PIPE_P + q];
                            X[0] = r.a[0].x;
                            X[1] = r.a[0].y;
                            X[2] = r.b[0].x;
                            X[3] = v.x;
                            X[4] = v.y;
                            X[5] = ((const double *)(slot + 13 * PIPE_P))[q];
                            observe(n, X);
                        }
                    };
                    for (int32_t j = min(PIPE_SUB, len - blk * PIPE_SUB) - 1; j >= 0; --j) {
                        PipeRow r;
                        r.get(buf + j * PIPE_STEP, q);
                        reverse(r, j);
                    }
                    F.push(F.at(blk));
                }
                __syncthreads();
            }
            F.cur = F.next;
        }
        if (lane < PIPE_P && wanted(i0 + q)) {
#pragma unroll
            for (int d = 0; d < 6; ++d) Q.grad[d * B.ld + D.off + i0 + q] = lam[d];
        }
    }
}

// (The padding: the single problem's tangent takes 1.012 ms instead of 1.033 for
// 96 particles over 2,520 steps with an odd number of s_nop at its entry, which
// moves the starts of its waves' step loops by 4 bytes modulo 8.)
template <bool SINGLE, bool TAN, bool ADJ>
__global__ __launch_bounds__(TAN ? 256 : 128) void k_sens_pipe(ProbDesc d0, SwarmArrays B, PipeArgs Q)
{
    if constexpr (SINGLE && TAN) entry_pad<1>();
    pipe_body<SINGLE, TAN, ADJ>(blockIdx.x, d0, B, Q);
}

// Both sweeps of the refinement, from the checkpoints that the evaluation of
// its trials left: the normal equations in even workgroups and, at the same
// time, the gradient in odd ones, so that a launch of few problems lasts as
// long as one sweep: one workgroup that went forward and then back took 2.13 ms
// over 2,500 steps, this takes 1.09. With more, two workgroups share a compute
// unit, its LDS (segments of 8 steps) and its registers (at most 256 to a lane:
// with 261, which the compiler took by itself, 384 problems' refinement was 5%
// longer): 384 problems 4.23 -> 1.77 ms.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_sens_stored(ProbDesc d0, SwarmArrays B, PipeArgs Q)
{
    if (blockIdx.x & 1)
        pipe_body<false, false, true, true>(blockIdx.x >> 1, d0, B, Q);
    else
        pipe_body<false, true, false>(blockIdx.x >> 1, d0, B, Q);
}

// Solve (N + l diag(N)) y = rhs by Cholesky, N = J^T J packed (row-major
// upper triangle) in column i of jtj [21][ld]. Returns false (y unusable)
// when the damped matrix is not positive definite.
__device__ __forceinline__ bool damped_solve(const double *__restrict__ jtj, int64_t ld, int64_t i,
                                             double l, const double rhs[6], double r[6])
{
    double M[6][6];
    int t = 0;
    for (int a = 0; a < 6; ++a)
        for (int b = a; b < 6; ++b, ++t) M[a][b] = M[b][a] = jtj[t * ld + i];
    for (int a = 0; a < 6; ++a) {
        M[a][a] = M[a][a] * (1.0 + l);
        r[a] = rhs[a];
    }
    // Cholesky M = L L^T in place (lower triangle)
    bool ok = true;
    for (int a = 0; a < 6; ++a) {
        double s = M[a][a];
        for (int c = 0; c < a; ++c) s -= M[a][c] * M[a][c];
        if (!(s > 0.0)) ok = false;
        const double da = sqrt(s);
        M[a][a] = da;
        for (int b = a + 1; b < 6; ++b) {
            double v = M[b][a];
            for (int c = 0; c < a; ++c) v -= M[b][c] * M[a][c];
            M[b][a] = v / da;
        }
    }
    for (int a = 0; a < 6; ++a) {
        double v = r[a];
        for (int c = 0; c < a; ++c) v -= M[a][c] * r[c];
        r[a] = v / M[a][a];
    }
    for (int a = 5; a >= 0; --a) {
        double v = r[a];
        for (int c = a + 1; c < 6; ++c) v -= M[c][a] * r[c];
        r[a] = v / M[a][a];
    }
    return ok;
}

// Damped Gauss-Newton step of column i: the right-hand side is -gscale g
// (gscale g = J^T r; the adjoint gives g = grad chi2 = 2 J^T r).
__device__ __forceinline__ bool damped_step(const double *__restrict__ jtj,
                                            const double *__restrict__ g, int64_t ld, int64_t i,
                                            double gscale, double l, double r[6])
{
    double rhs[6];
    for (int a = 0; a < 6; ++a) rhs[a] = -gscale * g[a * ld + i];
    return damped_solve(jtj, ld, i, l, rhs, r);
}

// Damped Gauss-Newton step per candidate (column o of B's layout) with its
// own damping lam[o]; writes the trial state x + dx (x where the step fails).
template <int BS, bool SINGLE>
__global__ __launch_bounds__(BS) void k_gn_solve(ProbDesc d0, SwarmArrays B,
                                                 const double *__restrict__ jtj,
                                                 const double *__restrict__ g, double gscale,
                                                 const double *__restrict__ lam,
                                                 double *__restrict__ xt)
{
    int64_t p, tile;
    const ProbDesc &D = locate<SINGLE>(d0, B, p, tile);
    const int64_t li = tile * BS + threadIdx.x;
    if (li >= D.m) return;
    const int64_t i = D.off + li, ld = B.ld;
    const double *x = B.x;
    double r[6];
    const bool ok = damped_step(jtj, g, ld, i, gscale, lam[i], r);
    for (int d = 0; d < 6; ++d) xt[d * ld + i] = x[d * ld + i] + (ok ? r[d] : 0.0);
}

// 10^e for a small integer e (exact for e >= 0; 1 / 10^-e below).
__device__ __forceinline__ double pow10i(int e)
{
    double f = 1.0;
    for (int k = 0; k < (e < 0 ? -e : e); ++k) f *= 10.0;
    return e < 0 ? 1.0 / f : f;
}

// n steps of every lane's state from step `from` of the grid, as rk4_steps; hook
// sees the state before every multiple of L steps, a power of two (again where
// the steps are repeated on the IEEE path).
template <int LPP, class Hook>
__device__ __forceinline__ void trial_steps(const KArgs &A, int32_t from, int32_t n, int32_t L,
                                            double X[6], Hook hook)
{
    const int32_t end = from + n;
    auto run = [&](auto step) __attribute__((always_inline)) {
        for (int32_t s = from; s < end;) {
            const int32_t at = s & (L - 1), m = min(end - s, L - at);
            if (at == 0) hook(s >> __builtin_ctz(L), X);
            int32_t j = 0;
            for (; j + 4 <= m; j += 4) {
                step();
                step();
                step();
                step();
            }
            for (; j < m; ++j) step();
            s += m;
        }
    };
    if (A.fast) {
        double X0[6];
#pragma unroll
        for (int d = 0; d < 6; ++d) X0[d] = X[d];
        Cert cert;
        run([&]() __attribute__((always_inline)) {
            if constexpr (LPP == 1) {
                double a[6];
                rk4_sum<true>(A.mu, A.mu1, A.h, A.h2, X, a, cert);
#pragma unroll
                for (int d = 0; d < 6; ++d) X[d] = fma(A.h6, a[d], X[d]);
            } else {
                NoSink none;
                split_step<LPP>(A.mu, A.mu1, A.h, A.h2, A.h6, X, cert, none);
            }
        });
        if (__all(cert.ok(X[5]))) return;
#pragma unroll
        for (int d = 0; d < 6; ++d) X[d] = X0[d];
    }
    for (int32_t s = from; s < end; ++s) {
        if ((s & (L - 1)) == 0) hook(s >> __builtin_ctz(L), X);
        double a[6];
        Cert ieee;
        rk4_sum<false>(A.mu, A.mu1, A.h, A.h2, X, a, ieee);
#pragma unroll
        for (int d = 0; d < 6; ++d) X[d] = fma(A.h6, a[d], X[d]);
    }
}

// Walk the observation schedule of a wave's trials, the table staged in LDS:
// steps(from, n, X), then obs(k, row, S) with the state at observation k.
template <class Steps, class Obs>
__device__ __forceinline__ void trial_walk(const KArgs &A, double X[6], double *lds,
                                           int32_t *lds_ns, Steps steps, Obs obs)
{
    int32_t step = 0;
    for (int32_t k0 = 0; k0 < A.K; k0 += OBS_CHUNK) {
        const int32_t nk = min(OBS_CHUNK, A.K - k0);
        WaveScope::sync();
        for (int32_t j = WaveScope::rank(); j < nk * TAB_W; j += 64)
            lds[j] = A.tab[(int64_t)k0 * TAB_W + j];
        for (int32_t j = WaveScope::rank(); j < nk; j += 64) lds_ns[j] = A.ns[k0 + j];
        WaveScope::sync();
        for (int32_t kk = 0; kk < nk; ++kk) {
            const double *row = lds + kk * TAB_W;
            const int32_t target = __builtin_amdgcn_readfirstlane(lds_ns[kk]);
            steps(k0 + kk, step, target - step, X);
            step = target;
            double S[6];
#pragma unroll
            for (int d = 0; d < 6; ++d) S[d] = X[d];
            const double tau = row[TAB_TAU];
            if (tau != 0.0) rk4<false>(A.mu, A.mu1, A.fast, tau, 0.5 * tau, tau / 6.0, S);
            obs(k0 + kk, row, S);
        }
    }
}

// One trial wave of the batched refinement stage: trial t = lane / LPP of this
// wave's share of problem p's trials is k = t % T of candidate j = t / T, its
// damping lam[j] 10^(k - T/2). Its step v, corrected by geodesic acceleration
// (Transtrum and Sethna, 2012, "Improvements to the Levenberg-Marquardt
// algorithm for nonlinear least-squares minimization"): with the directional
// second derivative of the residuals
// r_vv ~ (2 / hd) ((r(x + hd v) - r(x)) / hd - J v), the correction solves
// (N + l diag N) a = -J^T r_vv, and the trial becomes x + v + a / 2 when
// 2 |a| <= alpha |v|. J^T r(x + hd v) pairs the rows of J at x, stored by the
// normal equations' launch (jrows, column p jstride + j), with the residuals
// propagated from x + hd v; J^T r(x) and N are the normal equations' own. Then
// the trial's chi2, leaving the states every Q.seg steps and after the last
// one for the sweeps of the next iteration. A finished candidate (done)
// repeats its state.
template <int LPP>
__device__ __forceinline__ void trial_wave(const TrialArgs &Q, int64_t p, int part, double *lds,
                                           int32_t *lds_ns)
{
    const ProbDesc &D = Q.descs[p];
    const KArgs &A = D.k;
    const int lane = (int)(threadIdx.x & 63), T = Q.first ? 1 : Q.T, nt = (int)D.m * T;
    const int t0 = part * (64 / LPP) + lane / LPP;
    if (part * (64 / LPP) >= nt) return;   // whole wave
    const int t = min(t0, nt - 1), j = t / T, k = t % T;
    const bool writes = t0 < nt && lane % LPP == 0;
    const int64_t c = p * 64 + j, o = p * 64 + t, ld = Q.ld;
    double X[6], v[6], vn = 0.0;
    load_state(Q.x, ld, c, X);
    bool ok = false;
    const double l = Q.first ? 0.0 : Q.lam[c] * pow10i(k - T / 2);
    if (!Q.first && !Q.done[c]) ok = damped_step(Q.jtj, Q.grad, ld, c, 0.5, l, v);
#pragma unroll
    for (int d = 0; d < 6; ++d) {
        if (!ok) v[d] = 0.0;
        vn = fma(v[d], v[d], vn);
    }
    bool geo = vn > 0.0;
    if (__any(geo)) {
        const double is = sqrt(A.w);
        const bool ranged = A.wr != 0.0;
        const int R = ranged ? 3 : 2;
        const double isr = sqrt(A.wr);
        const double *rows = Q.jrows + p * Q.jstride + j;
        double Y[6], gy[6];
#pragma unroll
        for (int d = 0; d < 6; ++d) {
            Y[d] = fma(Q.hd, v[d], X[d]);
            gy[d] = 0.0;
        }
        double J[18];   // the observation's rows of J, loaded ahead of the steps to it
        trial_walk(A, Y, lds, lds_ns, [&](int32_t kk, int32_t, int32_t n, double *y) {
            const double *q = rows + (int64_t)kk * R * 6 * Q.jld;
#pragma unroll
            for (int e = 0; e < 18; ++e)
                if (e < 12 || ranged) J[e] = q[e * Q.jld];
            if constexpr (LPP == 1)
                rk4_steps(A, n, y);
            else
                rk4_steps_split<LPP>(A, n, y);
        }, [&](int32_t, const double *row, const double *Sy) {
            double ea, eb, fa[3], fb[3], er = 0, fq[3] = {0, 0, 0};
            // (no line of sight: the trial stays x + v)
            if (!residual_and_grad(row, Sy, ea, eb, fa, fb, ranged, er, fq)) geo = false;
            const double ra = ea * is, rb = eb * is, rr = er * isr;
#pragma unroll
            for (int cc = 0; cc < 6; ++cc) {
                gy[cc] = fma(J[cc], ra, fma(J[6 + cc], rb, gy[cc]));
                if (ranged) gy[cc] = fma(J[12 + cc], rr, gy[cc]);
            }
        });
        // J^T r_vv = (2 / hd) ((gy - J^T r) / hd - N v)
        double Nv[6] = {0, 0, 0, 0, 0, 0};
        {
            int qi = 0;
            for (int a = 0; a < 6; ++a)
                for (int b = a; b < 6; ++b, ++qi) {
                    const double nab = Q.jtj[qi * ld + c];
                    Nv[a] = fma(nab, v[b], Nv[a]);
                    if (b != a) Nv[b] = fma(nab, v[a], Nv[b]);
                }
        }
        double rhs[6], acc[6], an = 0.0;
#pragma unroll
        for (int d = 0; d < 6; ++d)
            rhs[d] = -(2.0 / Q.hd) * ((gy[d] - Q.jtr[d * ld + c]) / Q.hd - Nv[d]);
        geo = damped_solve(Q.jtj, ld, c, l, rhs, acc) && geo;
#pragma unroll
        for (int d = 0; d < 6; ++d) an = fma(acc[d], acc[d], an);
        geo = geo && 4.0 * an <= Q.alpha * Q.alpha * vn;
        if (geo) {
#pragma unroll
            for (int d = 0; d < 6; ++d) v[d] = fma(0.5, acc[d], v[d]);
        }
    }
#pragma unroll
    for (int d = 0; d < 6; ++d) {
        X[d] = X[d] + v[d];
        if (writes) Q.xt[d * ld + o] = X[d];
    }
    // the trial's chi2
    CostAcc cost{0.0, A.w, A.mode, A.wr};
    const int32_t S = A.ns[A.K - 1], L = Q.seg;
    auto store = [&](int32_t row, const double *y) {
        if (!writes || !Q.ckpt) return;
#pragma unroll
        for (int d = 0; d < 6; ++d) Q.ckpt[((int64_t)row * 6 + d) * ld + o] = y[d];
    };
    trial_walk(A, X, lds, lds_ns, [&](int32_t, int32_t from, int32_t n, double *y) {
        trial_steps<LPP>(A, from, n, L, y, store);
    }, [&](int32_t, const double *row, const double *Sx) { cost(row, Sx); });
    store((S + L - 1) / L, X);
    if (!writes) return;
    Q.chi2t[o] = cost.J;
    if (Q.first) Q.stored[o] = (int32_t)o;
}

// The trials of the active problems (Q.work, *Q.count of them), each problem's
// in up to LPP waves of 64 / LPP. A launch of few problems lasts as long as
// its longest wave, which more lanes to a trial shorten (see split_step), so
// they take as many as leave every wave a SIMD of its own. Four waves to a
// workgroup, since waves of smaller ones share SIMDs while others idle. The
// steps of both walks are most of the time: problems of up to 2,500 steps take
// 1.55 ms up to 128 of them, 1.65 at 256 and 1.85 at 384 (the corrections and
// the evaluations as two launches of one wave or one workgroup per problem, in
// their fixed order: 1.52, 2.2 and 2.5 ms).
__global__ __launch_bounds__(256) void k_gn_trials(TrialArgs Q)
{
    __shared__ double tab[4][OBS_CHUNK * TAB_W];
    __shared__ int32_t ns[4][OBS_CHUNK];
    const int64_t count = *Q.count;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int64_t w = (int64_t)blockIdx.x * 4 + wave;
    double *lds = tab[wave];
    int32_t *lds_ns = ns[wave];
    auto problem = [&](int64_t e) { return (int64_t)__builtin_amdgcn_readfirstlane(Q.work[2 * e]); };
    if (4 * count <= Q.simds) {
        if (w / 4 < count) trial_wave<4>(Q, problem(w / 4), (int)(w % 4), lds, lds_ns);
    } else if (2 * count <= Q.simds) {
        if (w / 2 < count) trial_wave<2>(Q, problem(w / 2), (int)(w % 2), lds, lds_ns);
    } else {
        if (w < count) trial_wave<1>(Q, problem(w), 0, lds, lds_ns);
    }
}

// Selection after the trials: each live candidate takes its lowest trial chi2
// (first trial on ties) if strictly below its own, and sets its damping to
// that trial's times 0.1; if none is lower, the damping grows to 10 x the
// largest tried. A candidate is done once its accepted step, or every trial
// step when none is accepted, is no larger than step_tol in every component,
// or its damping reaches the cap; the problem leaves the loop (active[p] = 0)
// when all its candidates are done. stored[c]: the trial taken, whose
// checkpoints are the candidate's now, or -1: it stays where it is, and its
// normal equations and gradient are those of the last iteration.
__global__ __launch_bounds__(64) void k_gn_select(double *__restrict__ x, double *__restrict__ chi2,
                                                  double *__restrict__ lam, int32_t *__restrict__ done,
                                                  int32_t *__restrict__ active,
                                                  const double *__restrict__ xt,
                                                  const double *__restrict__ chi2t,
                                                  const int32_t *__restrict__ n, int32_t T,
                                                  int64_t ld, double step_tol,
                                                  int32_t *__restrict__ stored)
{
    const int64_t p = blockIdx.x;
    if (!active[p]) return;   // whole workgroup (one wave)
    const int j = threadIdx.x;
    bool live = false;
    if (j < n[p]) {
        const int64_t c = p * 64 + j;
        if (!done[c]) {
            int kb = -1;
            double cb = chi2[c];
            for (int k = 0; k < T; ++k) {
                const double ct = chi2t[p * 64 + j * T + k];
                if (ct < cb) {
                    cb = ct;
                    kb = k;
                }
            }
            double step = 0.0;
            stored[c] = kb < 0 ? -1 : (int32_t)(p * 64 + j * T + kb);
            if (kb >= 0) {
                const int64_t o = p * 64 + j * T + kb;
                for (int d = 0; d < 6; ++d) {
                    step = fmax(step, fabs(xt[d * ld + o] - x[d * ld + c]));
                    x[d * ld + c] = xt[d * ld + o];
                }
                chi2[c] = cb;
                lam[c] = fmax(lam[c] * pow10i(kb - T / 2) * 0.1, 1e-12);
            } else {
                for (int k = 0; k < T; ++k)
                    for (int d = 0; d < 6; ++d)
                        step = fmax(step, fabs(xt[d * ld + p * 64 + j * T + k] - x[d * ld + c]));
                lam[c] = fmin(lam[c] * pow10i(T - 1 - T / 2) * 10.0, 1e12);
            }
            const bool fin = !(step > step_tol) || (kb < 0 && lam[c] >= 1e12);
            if (fin) done[c] = 1;
            live = !fin;
        }
    }
    if (!__any(live) && j == 0) active[p] = 0;
}

// Live lanes of the refinement's packed launches: the (problem, candidate)
// pairs of lanes [n][2] (problems with the most RK4 steps first, each with its
// candidates from 0) whose problem is active and whose candidate is not done,
// in the same order, into out, and the active problems as work entries
// (problem, 0) into work; *count and *problems receive their numbers. One
// 1024-thread workgroup walks the list in chunks, each wave compacting its
// lanes with ballots and the workgroup adding the waves' totals.
__global__ __launch_bounds__(1024) void k_live_lanes(const int32_t *__restrict__ lanes, int64_t n,
                                                     const int32_t *__restrict__ active,
                                                     const int32_t *__restrict__ done,
                                                     int32_t *__restrict__ out,
                                                     int64_t *__restrict__ count,
                                                     int32_t *__restrict__ work,
                                                     int32_t *__restrict__ problems)
{
    __shared__ int32_t wave_total[2][16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint64_t below = lane == 0 ? 0 : ~0ull >> (64 - lane);
    int64_t base[2] = {0, 0};
    for (int64_t c0 = 0; c0 < n; c0 += 1024) {
        const int64_t q = c0 + threadIdx.x;
        int32_t p = 0, j = 0;
        bool flag[2] = {false, false};
        if (q < n) {
            p = lanes[2 * q];
            j = lanes[2 * q + 1];
            const bool on = active[p] != 0;
            flag[0] = on && !done[(int64_t)p * 64 + j];
            flag[1] = on && j == 0;
        }
        const uint64_t mask[2] = {__ballot(flag[0]), __ballot(flag[1])};
        if (lane < 2) wave_total[lane][wave] = __popcll(mask[lane]);
        __syncthreads();
#pragma unroll
        for (int f = 0; f < 2; ++f) {
            int64_t off = base[f];
            for (int w = 0; w < wave; ++w) off += wave_total[f][w];
            for (int w = 0; w < 16; ++w) base[f] += wave_total[f][w];
            if (flag[f]) {
                int32_t *dst = (f ? work : out) + 2 * (off + __popcll(mask[f] & below));
                dst[0] = p;
                dst[1] = j;
            }
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        *count = base[0];
        *problems = (int32_t)base[1];
    }
}

// Final undamped Gauss-Newton step of the batched refinement, one 64-lane
// workgroup per problem, candidate j < n[p] in column p * 64 + j: solves
// J^T J dx = -J^T r and moves the candidate by dx if every component of dx
// is at most max_step (the quadratic region of the minimum, where a
// Gauss-Newton step is accurate). Near a least-squares minimum the binary64
// chi2 carries rounding noise (about 1e-8 of its value) above the decrease
// of a step along a weakly observed direction, so the damped iterations,
// which keep a trial only if its chi2 is lower, stop wherever the noise hides
// further progress; the normal equations' right-hand side J^T r is far less
// affected, so this step lands on the minimiser.
__global__ __launch_bounds__(64) void k_gn_final(double *__restrict__ x,
                                                 const double *__restrict__ jtj,
                                                 const double *__restrict__ jtr,
                                                 const int32_t *__restrict__ n, int64_t ld,
                                                 double max_step)
{
    const int64_t p = blockIdx.x;
    const int j = threadIdx.x;
    if (j >= n[p]) return;
    const int64_t c = p * 64 + j;
    double r[6];
    if (!damped_step(jtj, jtr, ld, c, 1.0, 0.0, r)) return;
    bool small = true;
#pragma unroll
    for (int d = 0; d < 6; ++d) small = small && fabs(r[d]) <= max_step;
    if (!small) return;
#pragma unroll
    for (int d = 0; d < 6; ++d) x[d * ld + c] += r[d];
}

// Candidate gather of the refinement: columns p * stride + j of dst, j <
// stride <= 64 (one wave per problem). Without rec, column j holds the
// personal best of particle cand[p][j]. With rec (each problem's final
// global-best record, [nprob][REC]), column 0 holds the global best itself,
// whatever rank its personal best has: in the mixed-precision swarm the
// global best is decided by FP64 costs while the personal bests rank by FP32
// costs, so it need not be among them. The next columns take the selected
// personal bests in rank order, skipping one whose state equals the global
// best's bit for bit; the count stays that of the selected candidates, so
// the lowest-ranked one drops out when the global best was not among them.
// Columns past the candidates repeat column 0, so every column holds a valid
// state.
__global__ __launch_bounds__(64) void k_gather(SwarmArrays B, const int32_t *__restrict__ cand,
                                               int32_t top_k, const double *__restrict__ rec,
                                               double *__restrict__ dst, int64_t dld,
                                               int64_t stride)
{
    const int64_t p = blockIdx.x;
    const ProbDesc &D = B.desc[p];
    const int j = threadIdx.x;
    const int32_t i = j < top_k ? cand[p * top_k + j] : -1;
    const bool has = i >= 0;
    int32_t i0 = cand[p * top_k];
    if (i0 < 0) i0 = 0;
    double s[6], s0[6];
#pragma unroll
    for (int d = 0; d < 6; ++d) {
        s[d] = B.p[d * B.ld + D.off + (has ? i : i0)];
        s0[d] = B.p[d * B.ld + D.off + i0];
    }
    const int nvalid = __popcll(__ballot(has));
    const double *r = rec ? rec + p * REC : nullptr;
    const bool use_rec = r && r[1] >= 0.0;
    int col = has ? j : -1;
    if (use_rec) {
        bool dup = has;
#pragma unroll
        for (int d = 0; d < 6; ++d) {
            s0[d] = r[2 + d];
            dup = dup && __double_as_longlong(s[d]) == __double_as_longlong(s0[d]);
        }
        const uint64_t keep = __ballot(has && !dup);
        const uint64_t below = j == 0 ? 0ull : (keep & (~0ull >> (64 - j)));
        col = (has && !dup) ? 1 + __popcll(below) : -1;
        if (col >= nvalid) col = -1;
    }
    if (col >= 0 && col < stride) {
#pragma unroll
        for (int d = 0; d < 6; ++d) dst[d * dld + p * stride + col] = s[d];
    }
    // column 0 (the global best) and the columns past the candidates
    if (j < stride && ((use_rec && j == 0) || j >= nvalid)) {
#pragma unroll
        for (int d = 0; d < 6; ++d) dst[d * dld + p * stride + j] = s0[d];
    }
}

// Per problem: the candidate column with the lowest (chi2, column) among its
// n[p] candidates at p * stride; writes its state (best [6][nprob]) and chi2.
__global__ __launch_bounds__(64) void k_pick_best(const double *__restrict__ x,
                                                  const double *__restrict__ chi2,
                                                  const int32_t *__restrict__ n, int64_t ld,
                                                  int64_t stride, double *__restrict__ best,
                                                  double *__restrict__ best_chi2)
{
    const int64_t nprob = gridDim.x;
    __shared__ double red[2];
    const int64_t p = blockIdx.x;
    double key = INFINITY, idx = INFINITY;
    for (int j = threadIdx.x; j < n[p]; j += blockDim.x) {
        const double k = cost_key(chi2[p * stride + j]);
        if (lex_less(k, (double)j, key, idx)) {
            key = k;
            idx = (double)j;
        }
    }
    block_argmin(key, idx, red);
    if (threadIdx.x < 6) {
        const int64_t j = idx < INFINITY ? (int64_t)idx : 0;
        best[threadIdx.x * nprob + p] = x[threadIdx.x * ld + p * stride + j];
    }
    if (threadIdx.x == 0) best_chi2[p] = idx < INFINITY ? key : NAN;
}

// Accept the trial where its chi2 is strictly lower (and finite); adapt the
// damping (/10 on success, *10 on failure). lam is initialised on the first
// iteration (first != 0).
template <int BS, bool SINGLE>
__global__ __launch_bounds__(BS) void k_gn_accept(ProbDesc d0, SwarmArrays B,
                                                  const double *__restrict__ xt,
                                                  double *__restrict__ chi2,
                                                  const double *__restrict__ chi2t,
                                                  double *__restrict__ lam)
{
    int64_t p, tile;
    const ProbDesc &D = locate<SINGLE>(d0, B, p, tile);
    const int64_t li = tile * BS + threadIdx.x;
    if (li >= D.m) return;
    const int64_t i = D.off + li, ld = B.ld;
    double *x = B.x;
    const double c = chi2[i], ct = chi2t[i];
    if (ct < c) {
        for (int d = 0; d < 6; ++d) x[d * ld + i] = xt[d * ld + i];
        chi2[i] = ct;
        lam[i] = fmax(lam[i] * 0.1, 1e-12);
    } else {
        lam[i] = fmin(lam[i] * 10.0, 1e12);
    }
}

// ---------------------------------------------------------------------------
// Launchers.
// ---------------------------------------------------------------------------

hipError_t launch_grad(const ProbDesc &d0, const SwarmArrays &B, int bs, int64_t grid,
                       double *grad, double *work, int64_t wld, int32_t mode, hipStream_t st)
{
    const Lanes L;
    if (B.desc == nullptr) {
        IOD_DISPATCH_BS(bs, hipLaunchKernelGGL((k_grad<BS_, PLACE_SINGLE>), dim3((unsigned)grid), dim3(BS_), 0, st, d0, B, L, grad, work, wld, mode));
    } else {
        IOD_DISPATCH_BS(bs, hipLaunchKernelGGL((k_grad<BS_, PLACE_BATCH>), dim3((unsigned)grid), dim3(BS_), 0, st, d0, B, L, grad, work, wld, mode));
    }
    return hipGetLastError();
}

hipError_t launch_normal(const ProbDesc &d0, const SwarmArrays &B, int bs, int64_t grid,
                         double *chi2, double *jtj, double *jtr, hipStream_t st, double *jrows,
                         int64_t jstride, int64_t jld, const Lanes &L)
{
    if (L.pairs) {
        if (bs != 64) return hipErrorInvalidValue;
        hipLaunchKernelGGL((k_normal<64, PLACE_PACKED>), dim3((unsigned)grid), dim3(64), 0, st, d0, B, L, chi2, jtj, jtr, jrows, jstride, jld);
    } else if (B.desc == nullptr) {
        IOD_DISPATCH_BS(bs, hipLaunchKernelGGL((k_normal<BS_, PLACE_SINGLE>), dim3((unsigned)grid), dim3(BS_), 0, st, d0, B, L, chi2, jtj, jtr, jrows, jstride, jld));
    } else {
        IOD_DISPATCH_BS(bs, hipLaunchKernelGGL((k_normal<BS_, PLACE_BATCH>), dim3((unsigned)grid), dim3(BS_), 0, st, d0, B, L, chi2, jtj, jtr, jrows, jstride, jld));
    }
    return hipGetLastError();
}

hipError_t launch_normal_grad(const ProbDesc &d0, const SwarmArrays &NB, const SwarmArrays &GB,
                              int64_t grid, double *chi2, double *jtj, double *jtr, double *jrows,
                              int64_t jstride, int64_t jld, double *grad, double *work,
                              int64_t wld, int32_t mode, hipStream_t st, const Lanes &L,
                              const Gate &G)
{
    if (!L.pairs || NB.desc != GB.desc) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_normal_grad, dim3((unsigned)(2 * grid)), dim3(64), 0, st, d0, NB, GB, L, chi2, jtj, jtr, jrows, jstride, jld, grad, work, wld, mode, G);
    return hipGetLastError();
}

hipError_t launch_sens_pipe(const ProbDesc &d0, const SwarmArrays &B, const PipeArgs &Q,
                            int64_t grid, bool tan, hipStream_t st)
{
    if (Q.seg < PIPE_SUB || Q.seg > PIPE_MAX_SEG || Q.seg % PIPE_SUB) return hipErrorInvalidValue;
    const unsigned lds = (unsigned)pipe_lds_bytes(Q.seg, tan, !tan);
    const dim3 g((unsigned)grid), b(tan ? 256 : 128);
    const bool single = B.desc == nullptr;
    if (tan) {
        if (single) hipLaunchKernelGGL((k_sens_pipe<true, true, false>), g, b, lds, st, d0, B, Q);
        else hipLaunchKernelGGL((k_sens_pipe<false, true, false>), g, b, lds, st, d0, B, Q);
    } else {
        if (single) hipLaunchKernelGGL((k_sens_pipe<true, false, true>), g, b, lds, st, d0, B, Q);
        else hipLaunchKernelGGL((k_sens_pipe<false, false, true>), g, b, lds, st, d0, B, Q);
    }
    return hipGetLastError();
}

hipError_t launch_sens_stored(const ProbDesc &d0, const SwarmArrays &B, const PipeArgs &Q,
                              int64_t grid, hipStream_t st)
{
    if (!B.desc || !Q.stored || Q.seg < PIPE_SUB || Q.seg > PIPE_MAX_SEG || Q.seg % PIPE_SUB)
        return hipErrorInvalidValue;
    const unsigned lds = (unsigned)pipe_lds_bytes(Q.seg, true, true);
    hipLaunchKernelGGL(k_sens_stored, dim3((unsigned)(2 * grid)), dim3(256), lds, st, d0, B, Q);
    return hipGetLastError();
}

hipError_t launch_gn_solve(const ProbDesc &d0, const SwarmArrays &B, int bs, int64_t grid,
                           const double *jtj, const double *g, double gscale, const double *lam,
                           double *xt, hipStream_t st)
{
    const bool single = B.desc == nullptr;
    IOD_DISPATCH_BS(bs, if (single) hipLaunchKernelGGL((k_gn_solve<BS_, true>), dim3((unsigned)grid), dim3(BS_), 0, st, d0, B, jtj, g, gscale, lam, xt);
                        else hipLaunchKernelGGL((k_gn_solve<BS_, false>), dim3((unsigned)grid), dim3(BS_), 0, st, d0, B, jtj, g, gscale, lam, xt));
    return hipGetLastError();
}

hipError_t launch_gn_trials(const TrialArgs &Q, int64_t nprob, hipStream_t st)
{
    if (Q.T < 1 || Q.T > 64 || Q.seg < 1 || (Q.seg & (Q.seg - 1)) || (!Q.first && !Q.jrows)) return hipErrorInvalidValue;
    // workgroups for whichever share the number of active problems calls for
    const int64_t four = std::min<int64_t>(nprob, Q.simds / 4), two = (std::min<int64_t>(nprob, Q.simds / 2) + 1) / 2;
    const int64_t grid = std::max({four, two, (nprob + 3) / 4});
    hipLaunchKernelGGL(k_gn_trials, dim3((unsigned)grid), dim3(256), 0, st, Q);
    return hipGetLastError();
}

hipError_t launch_gn_select(double *x, double *chi2, double *lam, int32_t *done, int32_t *active,
                            const double *xt, const double *chi2t, const int32_t *n, int32_t T,
                            int64_t nprob, int64_t ld, double step_tol, int32_t *stored,
                            hipStream_t st)
{
    if (T < 1 || T > 64) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_gn_select, dim3((unsigned)nprob), dim3(64), 0, st, x, chi2, lam, done, active, xt, chi2t, n, T, ld, step_tol, stored);
    return hipGetLastError();
}

hipError_t launch_live_lanes(const int32_t *lanes, int64_t n, const int32_t *active,
                            const int32_t *done, int32_t *out, int64_t *count, int32_t *work,
                            int32_t *problems, hipStream_t st)
{
    hipLaunchKernelGGL(k_live_lanes, dim3(1), dim3(1024), 0, st, lanes, n, active, done, out, count, work, problems);
    return hipGetLastError();
}

hipError_t launch_gn_final(double *x, const double *jtj, const double *jtr, const int32_t *n,
                          int64_t nprob, int64_t ld, double max_step, hipStream_t st)
{
    hipLaunchKernelGGL(k_gn_final, dim3((unsigned)nprob), dim3(64), 0, st, x, jtj, jtr, n, ld, max_step);
    return hipGetLastError();
}

hipError_t launch_gather(const SwarmArrays &B, const int32_t *cand, int32_t top_k,
                         const double *rec, double *dst, int64_t dld, int64_t stride,
                         hipStream_t st)
{
    if (stride > 64 || top_k > stride) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_gather, dim3((unsigned)B.nprob), dim3(64), 0, st, B, cand, top_k, rec, dst, dld, stride);
    return hipGetLastError();
}

hipError_t launch_pick_best(const double *x, const double *chi2, const int32_t *n, int64_t nprob,
                            int64_t ld, int64_t stride, double *best, double *best_chi2,
                            hipStream_t st)
{
    hipLaunchKernelGGL(k_pick_best, dim3((unsigned)nprob), dim3(64), 0, st, x, chi2, n, ld, stride, best, best_chi2);
    return hipGetLastError();
}

hipError_t launch_gn_accept(const ProbDesc &d0, const SwarmArrays &B, int bs, int64_t grid,
                            const double *xt, double *chi2, const double *chi2t, double *lam,
                            hipStream_t st)
{
    const bool single = B.desc == nullptr;
    IOD_DISPATCH_BS(bs, if (single) hipLaunchKernelGGL((k_gn_accept<BS_, true>), dim3((unsigned)grid), dim3(BS_), 0, st, d0, B, xt, chi2, chi2t, lam);
                        else hipLaunchKernelGGL((k_gn_accept<BS_, false>), dim3((unsigned)grid), dim3(BS_), 0, st, d0, B, xt, chi2, chi2t, lam));
    return hipGetLastError();
}

// lam[col] = value for the valid columns of the layout.
template <int BS, bool SINGLE>
__global__ __launch_bounds__(BS) void k_fill_cols(ProbDesc d0, SwarmArrays B, double *out,
                                                  double value)
{
    int64_t p, tile;
    const ProbDesc &D = locate<SINGLE>(d0, B, p, tile);
    const int64_t li = tile * BS + threadIdx.x;
    if (li < D.m) out[D.off + li] = value;
}

hipError_t launch_fill_cols(const ProbDesc &d0, const SwarmArrays &B, int bs, int64_t grid,
                            double *out, double value, hipStream_t st)
{
    const bool single = B.desc == nullptr;
    IOD_DISPATCH_BS(bs, if (single) hipLaunchKernelGGL((k_fill_cols<BS_, true>), dim3((unsigned)grid), dim3(BS_), 0, st, d0, B, out, value);
                        else hipLaunchKernelGGL((k_fill_cols<BS_, false>), dim3((unsigned)grid), dim3(BS_), 0, st, d0, B, out, value));
    return hipGetLastError();
}

}  // namespace iodk
