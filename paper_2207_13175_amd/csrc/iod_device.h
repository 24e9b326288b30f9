// iod_device.h -- device building blocks shared by the gfx950 kernels of
// libiod: the CR3BP right-hand side and RK4 step (eqs. cr3bp:x-z), the
// observation-schedule walk, the residual cost (eqs. rel:pos, meas:function,
// b:total, total:cost), Philox4x64-10, the particle-swarm update and
// initialisation (Algorithm 1 and its variants), Algorithm 2's test, and the
// deterministic argmin reductions. Included by iod_kernels.hip (FP64 swarm),
// iod_mixed.hip (mixed precision) and iod_sens.hip (sensitivities).
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "iod_internal.h"

namespace iodk {

// ---------------------------------------------------------------------------
// Dynamics: eqs. cr3bp:x-z in the rotating barycentric frame.
// ---------------------------------------------------------------------------

// In-range forms of the device's correctly rounded FP64 sqrt and reciprocal.
// The square root is the instruction sequence the compiler emits for sqrt(x)
// (hardware reciprocal-sqrt seed, one Goldschmidt step and two Markstein
// corrections) without the operand rescaling and special-value fixups, which
// are identities when x >= 2^-767 is finite. It also returns hh = 1/(2 sqrt x)
// to about 2^-47 relative (the seed's error, at most 5.3e-8 over the device's
// whole input range, enters as 1.5 times its square).
__device__ __forceinline__ double sqrt_inrange(double x, double &hh)
{
    const double y = __builtin_amdgcn_rsq(x);
    double g = x * y;
    hh = y * 0.5;
    const double r = fma(-hh, g, 0.5);
    g = fma(g, r, g);
    hh = fma(hh, r, hh);
    double d = fma(-g, g, x);
    g = fma(d, hh, g);
    d = fma(-g, g, x);
    return fma(d, hh, g);
}

// 1 / D for D = (x1 sqrt(x1)) (x2 sqrt(x2)), correctly rounded, from the
// halved inverse roots h1, h2 that the square roots leave behind: the seed
// 64 (h1 h2)^3 is within 2^-44 of it, one Newton step brings that within an
// ulp, and the last step then rounds correctly (Markstein's condition) unless
// D's mantissa is all ones. That one shows in the last residual e = 1 - D r,
// which is below 2^-53 for every other D and 2^-53 there (r = 2^k, whose
// neighbour is the right answer and ties with it). It takes eight
// instructions where the hardware reciprocal (four issue slots) and its two
// Newton steps took ten slots.
__device__ __forceinline__ double rcp_from_roots(double D, double h1, double h2, double &e)
{
    const double t = h1 * h2;
    double r = (64.0 * t) * (t * t);
    e = fma(-D, r, 1.0);
    r = fma(r, e, r);
    e = fma(-D, r, 1.0);
    return fma(e, r, r);
}

// What certifies in-range results, from every D = D1 D2 and the residual e of
// its reciprocal: D < 2^1000 and e < 2^-53, on the high words as integers
// (which order as the values do for numbers and infinities; a NaN's sign bit,
// set in those that this device makes, puts it below every positive number, so
// NaNs need a test of their own). A D too small for the reciprocal, whose seed overflows,
// and a zero D leave a NaN reciprocal where IEEE division gives an infinity. It
// makes every component of the acceleration NaN, and with it whatever the
// caller hands to ok(): a value that the accelerations of all certified stages
// have reached, such as a velocity after the steps. Two three-way maxima per
// two values, 4 issue slots per RK4 step, where two comparisons per value took
// 8, and one comparison per certified interval. With the reciprocal above a
// step takes 262 slots instead of 274: an iteration of the single large swarm
// went from 2.01 to 1.90 ms, and the uneven batch (two waves to a SIMD) gained 1-2%.
struct Mark {
    double D, e;
};

struct Cert {
    int32_t D = -0x7fffffff - 1, e = -0x7fffffff - 1;
    __device__ __forceinline__ void add(const Mark &a, const Mark &b)
    {
        D = max(max(__double2hiint(a.D), __double2hiint(b.D)), D);
        e = max(max(__double2hiint(a.e), __double2hiint(b.e)), e);
    }
    __device__ __forceinline__ bool ok(double reached) const
    {
        return D < ((1023 + 1000) << 20) && e < ((1023 - 53) << 20) && !isnan(reached);
    }
};

// f(s) for s = (x, y, z, vx, vy, vz):
//   ax =  2 vy + x - (1-mu)(x+mu)/r1^3 - mu (x-(1-mu))/r2^3
//   ay = -2 vx + y - ((1-mu)/r1^3 + mu/r2^3) y
//   az =           - ((1-mu)/r1^3 + mu/r2^3) z
// with both inverse cubes from one reciprocal: D_j = r_j^2 sqrt(r_j^2),
// R = 1/(D1 D2), c1 = (1-mu)(D2 R), c2 = mu (D1 R); sqrt and the reciprocal
// correctly rounded.
//
// INRANGE = true uses the in-range sequences; the result is certified equal
// to the IEEE one if the returned mark passes Cert. A reciprocal that is a
// number says that its seed neither overflowed nor lost bits
// below (D < 2^1000), so D >= 2^-1024 and x1 x2 = D^(2/3) >= 2^-683. Both
// radicands are then in range as well: r_j^2 < 2^-767 would need the other
// one above 2^84, but the primaries are one unit apart, so r_j ~ 0 puts the
// other at r ~ 1; an infinite or NaN radicand makes D1 D2 infinite or NaN. mu
// enters only through products, so every mu in [0, 0.5] takes the in-range
// path. INRANGE = false is the IEEE path (always valid).
template <bool INRANGE>
__device__ __forceinline__ Mark rhs(double mu, double mu1, const double s[6], double f[6])
{
    const double x = s[0], y = s[1], z = s[2], vx = s[3], vy = s[4];
    const double d1 = x + mu;
    const double d2 = x - mu1;
    const double q = fma(z, z, y * y);
    const double r1s = fma(d1, d1, q);
    const double r2s = fma(d2, d2, q);
    double h1 = 0.0, h2 = 0.0;
    const double D1 = r1s * (INRANGE ? sqrt_inrange(r1s, h1) : sqrt(r1s));
    const double D2 = r2s * (INRANGE ? sqrt_inrange(r2s, h2) : sqrt(r2s));
    const double D = D1 * D2;
    double e = 0.0;
    const double R = INRANGE ? rcp_from_roots(D, h1, h2, e) : 1.0 / D;
    const double c1 = mu1 * (D2 * R);
    const double c2 = mu * (D1 * R);
    const double cs = c1 + c2;
    f[0] = s[3];
    f[1] = s[4];
    f[2] = s[5];
    f[3] = fma(-c2, d2, fma(-c1, d1, fma(2.0, vy, x)));
    f[4] = fma(-cs, y, fma(-2.0, vx, y));
    f[5] = -(cs * z);
    return {D, e};
}

// Stage sum a = k1 + 2 k2 + 2 k3 + k4 of the classical RK4 step of size h
// (h2 = h/2) from X, accumulated as the stages are produced, so only X, a,
// the stage input and one derivative are live. cert takes in every stage.
template <bool INRANGE>
__device__ __forceinline__ void rk4_sum(double mu, double mu1, double h, double h2,
                                        const double X[6], double a[6], Cert &cert)
{
    double k[6], s[6];
    Mark m = rhs<INRANGE>(mu, mu1, X, k);
#pragma unroll
    for (int d = 0; d < 6; ++d) {
        a[d] = k[d];
        s[d] = fma(h2, k[d], X[d]);
    }
    cert.add(m, rhs<INRANGE>(mu, mu1, s, k));
#pragma unroll
    for (int d = 0; d < 6; ++d) {
        a[d] = fma(2.0, k[d], a[d]);
        s[d] = fma(h2, k[d], X[d]);
    }
    m = rhs<INRANGE>(mu, mu1, s, k);
#pragma unroll
    for (int d = 0; d < 6; ++d) {
        a[d] = fma(2.0, k[d], a[d]);
        s[d] = fma(h, k[d], X[d]);
    }
    cert.add(m, rhs<INRANGE>(mu, mu1, s, k));
#pragma unroll
    for (int d = 0; d < 6; ++d) a[d] = a[d] + k[d];
}

// One RK4 step in place, X <- X + h6 a (h6 = h/6). The stage sum runs with
// the in-range sequences; if any lane of the wave is not certified, the wave
// recomputes it from X on the IEEE path. Both give the same bits wherever the
// first is certified, so the result is always that of correctly rounded
// sqrt and division. X is updated only once the sum is final, so nothing
// needs a second copy of the state. VEL: the velocity is wanted too; otherwise
// only the position is certified, which the accelerations of stages 1 to 3
// reach, and the last stage's acceleration is not formed at all (11 instructions).
template <bool VEL>
__device__ __forceinline__ void rk4(double mu, double mu1, bool fast, double h, double h2,
                                    double h6, double X[6])
{
    double a[6];
    bool ok = false;
    if (fast) {
        Cert cert;
        rk4_sum<true>(mu, mu1, h, h2, X, a, cert);
        ok = cert.ok(a[VEL ? 5 : 2]);
    }
    if (!__all(ok)) {
        Cert ieee;
        rk4_sum<false>(mu, mu1, h, h2, X, a, ieee);
    }
#pragma unroll
    for (int d = 0; d < 6; ++d) X[d] = fma(h6, a[d], X[d]);
}

// n steps of size h in place. The in-range sequences run all n steps with no
// vote in between: each lane only accumulates the certificate of every stage
// of every step, and the wave votes once at the end. If some lane was
// not certified, the wave restores the state it started from and redoes the
// n steps on the IEEE path. Either way the result is that of correctly rounded sqrt and
// division, bit for bit, as with a vote per step; without a branch between
// steps the scheduler can overlap one step's distance chains with the end
// of the previous step. U steps per loop trip: a wave that has its SIMD to
// itself gains from a longer trip, while waves that share one hide each
// other's latency anyway (the callers choose).
template <int U = 2>
__device__ __forceinline__ void rk4_steps(const KArgs &A, int32_t n, double X[6])
{
    if (A.fast) {
        double X0[6];
#pragma unroll
        for (int d = 0; d < 6; ++d) X0[d] = X[d];
        Cert cert;
#pragma unroll U
        for (int32_t j = 0; j < n; ++j) {
            double a[6];
            rk4_sum<true>(A.mu, A.mu1, A.h, A.h2, X, a, cert);
#pragma unroll
            for (int d = 0; d < 6; ++d) X[d] = fma(A.h6, a[d], X[d]);
        }
        if (__all(cert.ok(X[5]))) return;
#pragma unroll
        for (int d = 0; d < 6; ++d) X[d] = X0[d];
    }
    for (int32_t j = 0; j < n; ++j) {
        double a[6];
        Cert ieee;
        rk4_sum<false>(A.mu, A.mu1, A.h, A.h2, X, a, ieee);
#pragma unroll
        for (int d = 0; d < 6; ++d) X[d] = fma(A.h6, a[d], X[d]);
    }
}

// ---------------------------------------------------------------------------
// Several lanes to a particle. A launch that leaves SIMDs idle is bound by one
// wave's instruction count (dependent FP64 instructions issue back to back,
// so there is no latency to hide), and more lanes per particle shorten it:
// the distance chains of stages 1 and 2 of an RK4 step do not depend on each
// other (stage 2's position is X + h/2 V), nor do those of stages 3 and 4
// once stage 2's acceleration is known. So the lanes of a particle take
// stage 1 or 2 (then 3 or 4), and with four lanes also one primary each.
// Every lane holds the whole state; values cross between adjacent lanes with
// quad permutations. Each operation is the one-lane form's, on the same
// operands, so the bits are the same. Per step 262 issue slots become 188
// with two lanes and 172 with four: 256 particles over 500 steps went from 243
// to 157 us, 5,001 over 2,257 from 1,098 to 727 us (four lanes), 32,768 over
// 500 from 243 to 184 us (two). A wave then holds 32 or 16 particles, so this
// pays only while the waves still have a SIMD each.
// ---------------------------------------------------------------------------

// x of another lane of the quad, two 32-bit moves (S0..S3: the source lane of
// lanes 0..3).
template <int S0, int S1, int S2, int S3>
__device__ __forceinline__ double quad_perm(double x)
{
    constexpr int CTRL = S0 | S1 << 2 | S2 << 4 | S3 << 6;
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}

// LPP lanes per particle, 2 or 4: lane = LPP/2 * stage + primary. early / late:
// the value of the lane that holds stage 1 or 3 / stage 2 or 4 (with four
// lanes, of the own primary's); first / second: the value of the own stage's
// lane for primary 1 / 2 (four lanes only); other: of its other primary's.
template <int LPP>
struct Quad {
    static __device__ __forceinline__ bool is_late() { return threadIdx.x & (LPP / 2); }
    static __device__ __forceinline__ double early(double x)
    {
        return LPP == 2 ? quad_perm<0, 0, 2, 2>(x) : quad_perm<0, 1, 0, 1>(x);
    }
    static __device__ __forceinline__ double late(double x)
    {
        return LPP == 2 ? quad_perm<1, 1, 3, 3>(x) : quad_perm<2, 3, 2, 3>(x);
    }
    static __device__ __forceinline__ double first(double x) { return quad_perm<0, 0, 2, 2>(x); }
    static __device__ __forceinline__ double second(double x) { return quad_perm<1, 1, 3, 3>(x); }
    static __device__ __forceinline__ double other(double x) { return quad_perm<1, 0, 3, 2>(x); }
};

// The position-dependent part of rhs<true> at p, shared by a particle's
// lanes: c1, c2, their sum and the offsets; returns the mark. xj, muj: with four
// lanes, mu or -mu1 and mu1 or mu by the lane's primary. JAC (four lanes): also
// the own primary's Jacobian factor e_j = 3 c_j / r_j^2 (rhs_jac).
struct Attraction {
    double d1, d2, c1, c2, cs, ej;
};

template <int LPP, bool JAC = false>
__device__ __forceinline__ Mark attraction(double mu, double mu1, double xj, double muj,
                                         const double p[3], Attraction &o)
{
    o.d1 = p[0] + mu;
    o.d2 = p[0] - mu1;
    const double q = fma(p[2], p[2], p[1] * p[1]);
    double D, e;
    if (LPP == 4) {
        const double dj = p[0] + xj;
        const double rs = fma(dj, dj, q);
        double hj;
        const double qj = sqrt_inrange(rs, hj);
        const double Dj = rs * qj;
        const double Do = Quad<4>::other(Dj);
        const double ho = Quad<4>::other(hj);
        D = Dj * Do;
        const double ij = Do * rcp_from_roots(D, hj, ho, e);
        const double cj = muj * ij;
        if (JAC) o.ej = 3.0 * cj * (qj * ij);
        o.c1 = Quad<4>::first(cj);
        o.c2 = Quad<4>::second(cj);
    } else {
        const double r1s = fma(o.d1, o.d1, q);
        const double r2s = fma(o.d2, o.d2, q);
        double h1, h2;
        const double D1 = r1s * sqrt_inrange(r1s, h1);
        const double D2 = r2s * sqrt_inrange(r2s, h2);
        D = D1 * D2;
        const double R = rcp_from_roots(D, h1, h2, e);
        o.c1 = mu1 * (D2 * R);
        o.c2 = mu * (D1 * R);
    }
    o.cs = o.c1 + o.c2;
    return {D, e};
}

// x and y of rhs's acceleration at p moving with (vx, vy).
__device__ __forceinline__ void accel_xy(const Attraction &o, const double p[3], double vx,
                                         double vy, double &ax, double &ay)
{
    ax = fma(-o.c2, o.d2, fma(-o.c1, o.d1, fma(2.0, vy, p[0])));
    ay = fma(-o.cs, p[1], fma(-2.0, vx, p[1]));
}

// What a particle's lanes see of the stages on the way: sink(half, p, o), the
// own stage's position and attraction (stages 1 and 2 in half 0, 3 and 4 in 1).
struct NoSink {
    static constexpr bool JAC = false;
    __device__ __forceinline__ void operator()(int, const double *, const Attraction &) {}
};

// One RK4 step on the in-range path by the LPP lanes of each particle. In each
// half of the step the lanes evaluate their own stage's attraction, then the
// earlier stage's acceleration (with the velocity all lanes know) passes to
// the later stage's lanes, whose velocity and acceleration it completes.
template <int LPP, class Sink>
__device__ __forceinline__ void split_step(double mu, double mu1, double h, double h2, double h6,
                                           double X[6], Cert &cert, Sink &sink)
{
    using Q = Quad<LPP>;
    const bool is_late = Q::is_late(), second = LPP == 4 && (threadIdx.x & 1);
    const double ha = is_late ? h2 : 0.0, hb = is_late ? h : h2;
    const double xj = second ? -mu1 : mu, muj = second ? mu : mu1;
    const double *V = X + 3;
    double p[3], a[3], w[3], k1[3], k2[3], k3[3], v2[3], v3[3], v4[3];
    Attraction o;
    // stages 1 and 2
#pragma unroll
    for (int d = 0; d < 3; ++d) p[d] = fma(ha, V[d], X[d]);
    const Mark m = attraction<LPP, Sink::JAC>(mu, mu1, xj, muj, p, o);
    sink(0, p, o);
    double ax, ay;
    accel_xy(o, p, V[0], V[1], ax, ay);
    k1[0] = Q::early(ax);
    k1[1] = Q::early(ay);
    // the own stage's velocity: V, or stage 2's V + h/2 k1
    accel_xy(o, p, fma(ha, k1[0], V[0]), fma(ha, k1[1], V[1]), a[0], a[1]);
    a[2] = -(o.cs * p[2]);
    k1[2] = Q::early(a[2]);
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        // the next stage's velocity: stage 2's (early) or stage 3's (late)
        w[d] = fma(h2, a[d], V[d]);
        k2[d] = Q::late(a[d]);
        v2[d] = fma(h2, k1[d], V[d]);
        v3[d] = fma(h2, k2[d], V[d]);
    }
    // stages 3 and 4
#pragma unroll
    for (int d = 0; d < 3; ++d) p[d] = fma(hb, w[d], X[d]);
    cert.add(m, attraction<LPP, Sink::JAC>(mu, mu1, xj, muj, p, o));
    sink(1, p, o);
    accel_xy(o, p, v3[0], v3[1], ax, ay);
    k3[0] = Q::early(ax);
    k3[1] = Q::early(ay);
    a[2] = -(o.cs * p[2]);
    k3[2] = Q::early(a[2]);
#pragma unroll
    for (int d = 0; d < 3; ++d) v4[d] = fma(h, k3[d], V[d]);
    accel_xy(o, p, v4[0], v4[1], a[0], a[1]);
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const double sx = fma(2.0, v3[d], fma(2.0, v2[d], V[d])) + v4[d];
        const double sv = fma(2.0, k3[d], fma(2.0, k2[d], k1[d])) + Q::late(a[d]);
        X[d] = fma(h6, sx, X[d]);
        X[3 + d] = fma(h6, sv, X[3 + d]);
    }
}

// n steps as rk4_steps, by the LPP lanes of each particle.
template <int LPP>
__device__ __forceinline__ void rk4_steps_split(const KArgs &A, int32_t n, double X[6])
{
    if (A.fast) {
        double X0[6];
#pragma unroll
        for (int d = 0; d < 6; ++d) X0[d] = X[d];
        Cert cert;
        NoSink none;
        auto step = [&]() __attribute__((always_inline)) {
            split_step<LPP>(A.mu, A.mu1, A.h, A.h2, A.h6, X, cert, none);
        };
        // (written out: the compiler does not unroll a loop of lane exchanges
        // whose trip count it does not know)
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
        double a[6];
        Cert ieee;
        rk4_sum<false>(A.mu, A.mu1, A.h, A.h2, X, a, ieee);
#pragma unroll
        for (int d = 0; d < 6; ++d) X[d] = fma(A.h6, a[d], X[d]);
    }
}

// Who stages the observation table into LDS together: the whole workgroup
// (with barriers), or one wave on its own. A wave's lanes run in lockstep and
// its LDS accesses complete in issue order, so a wave needs only a fence
// that keeps the compiler from moving accesses across the hand-over.
struct BlockScope {
    static __device__ __forceinline__ int32_t rank() { return threadIdx.x; }
    static __device__ __forceinline__ int32_t size() { return blockDim.x; }
    static __device__ __forceinline__ void sync() { __syncthreads(); }
};
struct WaveScope {
    static __device__ __forceinline__ int32_t rank() { return threadIdx.x & 63; }
    static __device__ __forceinline__ int32_t size() { return 64; }
    static __device__ __forceinline__ void sync()
    {
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
};

// Walk the observation schedule: advance X on the grid, and at each
// observation hand the state there (a side copy advanced by the partial step
// when the time is off the grid) to `obs(row, S)`, which reads S's velocity
// only if Obs::VEL. Every thread of the scope
// (the workgroup, or the wave) must call this: it stages the table through
// LDS in chunks. LPP adjacent lanes hold the same particle (1, 2 or 4).
template <class Scope = BlockScope, int U = 2, int LPP = 1, class Obs>
__device__ __forceinline__ void walk(const KArgs &A, double X[6], double *lds, int32_t *lds_ns,
                                     Obs &obs)
{
    int32_t step = 0;
    for (int32_t k0 = 0; k0 < A.K; k0 += OBS_CHUNK) {
        const int32_t nk = min(OBS_CHUNK, A.K - k0);
        Scope::sync();
        for (int32_t j = Scope::rank(); j < nk * TAB_W; j += Scope::size())
            lds[j] = A.tab[(int64_t)k0 * TAB_W + j];
        for (int32_t j = Scope::rank(); j < nk; j += Scope::size()) lds_ns[j] = A.ns[k0 + j];
        Scope::sync();
        for (int32_t kk = 0; kk < nk; ++kk) {
            const double *row = lds + kk * TAB_W;
            const int32_t target = __builtin_amdgcn_readfirstlane(lds_ns[kk]);
            if (target > step) {
                if constexpr (LPP == 1)
                    rk4_steps<U>(A, target - step, X);
                else
                    rk4_steps_split<LPP>(A, target - step, X);
                step = target;
            }
            const double tau = row[TAB_TAU];
            double S[6];
#pragma unroll
            for (int d = 0; d < 6; ++d) S[d] = X[d];
            if (tau != 0.0) rk4<Obs::VEL>(A.mu, A.mu1, A.fast, tau, 0.5 * tau, tau / 6.0, S);
            obs(row, S);
        }
    }
}

// ---------------------------------------------------------------------------
// Measurement model and cost: eqs. rel:pos, meas:function, b:total,
// total:cost.
// ---------------------------------------------------------------------------

// Residual-squared accumulator. rho = r - r_chief; the azimuth and elevation
// residuals (observed - predicted, azimuth wrapped to (-pi, pi]) come from
// the angle-difference identities
//   |rho_xy| sin(da) = sa rho_x - ca rho_y,  |rho_xy| cos(da) = ca rho_x + sa rho_y
//   |rho|    sin(db) = sb rho_xy - cb rho_z, |rho|    cos(db) = cb rho_xy + sb rho_z
// so atan2 acts on the residual itself. rho_xy = 0 means the predicted
// azimuth is atan2(0, 0) = 0; rho = 0 has no line of sight and e = +inf.
// e_k = w (da^2 + db^2); J = sum e_k^2 (mode 0) or sum e_k (mode 1).
struct CostAcc {
    static constexpr bool VEL = false;
    double J, w;
    int32_t mode;
    double wr;   // range weight, 0 = angles only
    __device__ __forceinline__ void operator()(const double *row, const double S[6])
    {
        const double rx = S[0] - row[TAB_RC + 0];
        const double ry = S[1] - row[TAB_RC + 1];
        const double rz = S[2] - row[TAB_RC + 2];
        const double sa = row[TAB_SA], ca = row[TAB_CA], sb = row[TAB_SB], cb = row[TAB_CB];
        double e;
        if (rx == 0.0 && ry == 0.0 && rz == 0.0) {
            e = INFINITY;
        } else {
            const double rxy = sqrt(fma(rx, rx, ry * ry));
            double na, nd;
            if (rxy == 0.0) {
                na = sa;
                nd = ca;
            } else {
                na = fma(sa, rx, -(ca * ry));
                nd = fma(ca, rx, sa * ry);
            }
            const double da = atan2(na, nd);
            const double db = atan2(fma(sb, rxy, -(cb * rz)), fma(cb, rxy, sb * rz));
            e = w * fma(da, da, db * db);
            if (wr != 0.0) {
                // range residual: observed minus |rho|
                const double dr = row[TAB_RANGE] - sqrt(fma(rx, rx, fma(ry, ry, rz * rz)));
                e = fma(wr * dr, dr, e);
            }
        }
        J = (mode == 1) ? J + e : fma(e, e, J);
    }
};

template <class Scope = BlockScope, int U = 2, int LPP = 1>
__device__ __forceinline__ double eval_cost(const KArgs &A, const double x0[6], double *lds,
                                            int32_t *lds_ns)
{
    double X[6];
#pragma unroll
    for (int d = 0; d < 6; ++d) X[d] = x0[d];
    CostAcc acc{0.0, A.w, A.mode, A.wr};
    walk<Scope, U, LPP>(A, X, lds, lds_ns, acc);
    return acc.J;
}

// ---------------------------------------------------------------------------
// Philox4x64-10 (Salmon et al., SC'11).
// ---------------------------------------------------------------------------

__device__ __forceinline__ void philox4x64_10(uint64_t c[4], uint64_t k0, uint64_t k1)
{
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        if (r) {
            k0 += 0x9E3779B97F4A7C15ULL;
            k1 += 0xBB67AE8584CAA73BULL;
        }
        const uint64_t hi0 = __umul64hi(0xD2E7470EE14C6C93ULL, c[0]);
        const uint64_t lo0 = 0xD2E7470EE14C6C93ULL * c[0];
        const uint64_t hi1 = __umul64hi(0xCA5A826395121157ULL, c[2]);
        const uint64_t lo1 = 0xCA5A826395121157ULL * c[2];
        const uint64_t n0 = hi1 ^ c[1] ^ k0;
        const uint64_t n2 = hi0 ^ c[3] ^ k1;
        c[0] = n0;
        c[1] = lo1;
        c[2] = n2;
        c[3] = lo0;
    }
}

__device__ __forceinline__ double u01(uint64_t w) { return (double)(w >> 11) * 0x1.0p-53; }

// ---------------------------------------------------------------------------
// Particle swarm building blocks (Algorithm 1 and its variants).
// ---------------------------------------------------------------------------

// Initial position of particle j (its velocity is zero). With the grid
// initialisation, particles j < grid_g sit on the cell centres of a
// Cartesian grid over the box: j's mixed-radix digits (dimension 0 fastest)
// give u_d = (2 j_d + 1) / (2 n_d). Otherwise u is uniform, words 0-5 of
// Philox counters (0, j, problem, 0) and (1, j, problem, 0).
__device__ __forceinline__ void init_state(const ProbDesc &D, int64_t j, double X[6])
{
    double u[6];
    if (j < D.grid_g) {
        int64_t q = j;
#pragma unroll
        for (int d = 0; d < 6; ++d) {
            const int64_t nd = D.grid_n[d];
            const int64_t jd = q % nd;
            q /= nd;
            u[d] = (double)(2 * jd + 1) / (double)(2 * nd);
        }
    } else {
        uint64_t w[8] = {0, (uint64_t)j, D.problem, 0, 1, (uint64_t)j, D.problem, 0};
        philox4x64_10(w, D.seed, 0);
        philox4x64_10(w + 4, D.seed, 0);
#pragma unroll
        for (int d = 0; d < 6; ++d) u[d] = u01(w[d]);
    }
#pragma unroll
    for (int d = 0; d < 6; ++d) X[d] = D.lo[d] + (D.hi[d] - D.lo[d]) * u[d];
}

// Velocity and position update of particle j at iteration n towards its
// personal best Pb and the global best g:
//   v <- kappa (omega v + eta1 r1 (Pb - x) + eta2 r2 (g - x)),  x <- x + v,
// with kappa = 1 unless the constriction factor is on. r1, r2: words 0 and 1
// of Philox counter (n, j, problem, 1); per dimension, words 2d and 2d + 1
// of counters (n, j, problem, 2), (.., 3), (.., 4).
__device__ __forceinline__ void pso_update(const ProbDesc &D, int64_t n, int64_t j, double X[6],
                                           double V[6], const double Pb[6], const double g[6])
{
    double a1[6], a2[6];
    if (D.flags & PSO_PER_DIM_R) {
        uint64_t w[12];
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            w[4 * b + 0] = (uint64_t)n;
            w[4 * b + 1] = (uint64_t)j;
            w[4 * b + 2] = D.problem;
            w[4 * b + 3] = 2 + (uint64_t)b;
            philox4x64_10(w + 4 * b, D.seed, 0);
        }
#pragma unroll
        for (int d = 0; d < 6; ++d) {
            a1[d] = D.eta1 * u01(w[2 * d]);
            a2[d] = D.eta2 * u01(w[2 * d + 1]);
        }
    } else {
        uint64_t c[4] = {(uint64_t)n, (uint64_t)j, D.problem, 1};
        philox4x64_10(c, D.seed, 0);
        const double s1 = D.eta1 * u01(c[0]), s2 = D.eta2 * u01(c[1]);
#pragma unroll
        for (int d = 0; d < 6; ++d) {
            a1[d] = s1;
            a2[d] = s2;
        }
    }
#pragma unroll
    for (int d = 0; d < 6; ++d) {
        const double vn = D.kappa * (D.omega * V[d] + a1[d] * (Pb[d] - X[d]) + a2[d] * (g[d] - X[d]));
        V[d] = vn;
        X[d] = X[d] + vn;
    }
}

// Algorithm 2's test on the global-best costs of iterations n and n - L:
// K = |(jn - jl) / jn| < tau, with equal costs counted as K = 0.
__device__ __forceinline__ bool tolerance_met(double jn, double jl, double tau)
{
    const double K = (jn == jl) ? 0.0 : fabs((jn - jl) / jn);
    return K < tau;
}

// ---------------------------------------------------------------------------
// Argmin reductions: lexicographic (key, index), NaN ranked as +inf.
// ---------------------------------------------------------------------------

__device__ __forceinline__ double cost_key(double J) { return isnan(J) ? INFINITY : J; }

__device__ __forceinline__ bool lex_less(double ka, double ia, double kb, double ib)
{
    return ka < kb || (ka == kb && ia < ib);
}

// Wave-wide argmin by butterfly exchanges; every lane returns the minimum.
__device__ __forceinline__ void wave_argmin(double &key, double &idx)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const double ok = __shfl_xor(key, off, 64);
        const double oi = __shfl_xor(idx, off, 64);
        if (lex_less(ok, oi, key, idx)) {
            key = ok;
            idx = oi;
        }
    }
}

// Block-wide argmin; every thread returns the minimum. red: LDS [2 * waves].
__device__ __forceinline__ void block_argmin(double &key, double &idx, double *red)
{
    wave_argmin(key, idx);
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        red[2 * wave] = key;
        red[2 * wave + 1] = idx;
    }
    __syncthreads();
    key = red[0];
    idx = red[1];
    for (int w = 1; w < (int)(blockDim.x >> 6); ++w)
        if (lex_less(red[2 * w], red[2 * w + 1], key, idx)) {
            key = red[2 * w];
            idx = red[2 * w + 1];
        }
    __syncthreads();
}

// Workgroup argmin of (key(jp), i) over its valid particles (i counted within
// the problem), written with the winner's state to `slot` as
// [key, index, state[6]].
__device__ __forceinline__ void write_slot(double jp, int64_t i, bool valid, const double st[6],
                                           double *slot, double *red, double *wst)
{
    double key = valid ? cost_key(jp) : INFINITY;
    double idx = valid ? (double)i : INFINITY;
    block_argmin(key, idx, red);
    if (valid && (double)i == idx) {
#pragma unroll
        for (int d = 0; d < 6; ++d) wst[d] = st[d];
    }
    __syncthreads();
    if (threadIdx.x < REC)
        slot[threadIdx.x] = threadIdx.x == 0 ? key : threadIdx.x == 1 ? idx : wst[threadIdx.x - 2];
}

// Global best of one problem: merge(record, the problem's slots). The slot
// minimum replaces the record if the record is empty (index < 0) or the slot
// cost is strictly lower. Slot s holds the minimum of particles
// [s * per_slot, (s + 1) * per_slot). Every workgroup of the problem computes
// the same result.
__device__ __forceinline__ void reduce_global(const double *slots, int64_t nslots,
                                              int32_t per_slot, const double *prev, double g[6], double &gkey,
                                              double &gidx, double *red)
{
    double key = INFINITY, idx = INFINITY;
    for (int64_t s = threadIdx.x; s < nslots; s += blockDim.x) {
        const double k = slots[s * REC], i = slots[s * REC + 1];
        if (lex_less(k, i, key, idx)) {
            key = k;
            idx = i;
        }
    }
    block_argmin(key, idx, red);
    const double pk = prev[0], pi = prev[1];
    if (pi < 0.0 || key < pk) {
        const int64_t s = (int64_t)idx / per_slot;
        gkey = key;
        gidx = idx;
#pragma unroll
        for (int d = 0; d < 6; ++d) g[d] = slots[s * REC + 2 + d];
    } else {
        gkey = pk;
        gidx = pi;
#pragma unroll
        for (int d = 0; d < 6; ++d) g[d] = prev[2 + d];
    }
}

__device__ __forceinline__ void write_record(double *rec, const double g[6], double gkey,
                                             double gidx)
{
    if (threadIdx.x < REC)
        rec[threadIdx.x] = threadIdx.x == 0 ? gkey : threadIdx.x == 1 ? gidx : g[threadIdx.x - 2];
}

// ---------------------------------------------------------------------------
// Kernels. Swarm kernels serve one problem (SINGLE: the descriptor is a
// kernel argument, workgroup b is tile b) or a batch (the descriptors live in
// device memory and a work list maps workgroup b to (problem, tile), ordered
// longest problem first so the dispatcher's greedy placement balances the
// uneven work).
// ---------------------------------------------------------------------------

struct StoreStates {
    static constexpr bool VEL = true;
    double *out;
    int64_t ld, i;
    int32_t k;
    bool valid;
    __device__ __forceinline__ void operator()(const double *, const double S[6])
    {
        if (valid) {
#pragma unroll
            for (int d = 0; d < 6; ++d) out[((int64_t)k * 6 + d) * ld + i] = S[d];
        }
        ++k;
    }
};

struct StoreAngles {
    static constexpr bool VEL = false;
    double *out;
    int64_t ld, i;
    int32_t k;
    bool valid;
    __device__ __forceinline__ void operator()(const double *row, const double S[6])
    {
        // L = rho / |rho|, azimuth = atan2(L_y, L_x), elevation = asin(L_z)
        const double rx = S[0] - row[TAB_RC + 0];
        const double ry = S[1] - row[TAB_RC + 1];
        const double rz = S[2] - row[TAB_RC + 2];
        const double r = sqrt(rx * rx + ry * ry + rz * rz);
        double az = NAN, el = NAN;
        if (r != 0.0) {
            az = atan2(ry / r, rx / r);
            el = asin(rz / r);
        }
        if (valid) {
            out[((int64_t)k * 2 + 0) * ld + i] = az;
            out[((int64_t)k * 2 + 1) * ld + i] = el;
        }
        ++k;
    }
};

// Chief positions written into the observation table of each problem.
struct StoreChief {
    static constexpr bool VEL = false;
    double *tab;
    int32_t k;
    __device__ __forceinline__ void operator()(const double *, const double S[6])
    {
        if (threadIdx.x == 0) {
#pragma unroll
            for (int d = 0; d < 3; ++d) tab[(int64_t)k * TAB_W + TAB_RC + d] = S[d];
        }
        ++k;
    }
};

__device__ __forceinline__ void load_state(const double *x, int64_t ld, int64_t j, double X[6])
{
#pragma unroll
    for (int d = 0; d < 6; ++d) X[d] = x[d * ld + j];
}

template <bool SINGLE>
__device__ __forceinline__ const ProbDesc &locate(const ProbDesc &d0, const SwarmArrays &B,
                                                  int64_t &p, int64_t &tile)
{
    if (SINGLE) {
        p = 0;
        tile = blockIdx.x;
        return d0;
    }
    p = B.work[2 * (int64_t)blockIdx.x];
    tile = B.work[2 * (int64_t)blockIdx.x + 1];
    return B.desc[p];
}

// ---------------------------------------------------------------------------
// Launch helpers.
// ---------------------------------------------------------------------------

// N s_nop (4 bytes each) at a kernel's entry shift every later instruction of
// the kernel, and so where its loops start (each kernel's code starts on a
// 256-byte boundary, so a kernel's padding moves nothing else).
template <int N>
__device__ __forceinline__ void entry_pad()
{
    if constexpr (N > 0) {
        __asm__ volatile("s_nop 0");
        entry_pad<N - 1>();
    }
}

__device__ __forceinline__ bool closed(const Gate &g)
{
    return g.count && !(*g.count > g.above && *g.count <= g.upto);
}

static inline unsigned grid_for(int64_t m, int bs) { return (unsigned)((m + bs - 1) / bs); }

#define IOD_DISPATCH_BS(BSV, ...)                                  \
    switch (BSV) {                                                 \
    case 64: { constexpr int BS_ = 64; __VA_ARGS__; break; }       \
    case 128: { constexpr int BS_ = 128; __VA_ARGS__; break; }     \
    case 256: { constexpr int BS_ = 256; __VA_ARGS__; break; }     \
    default: return hipErrorInvalidValue;                          \
    }

#define IOD_DISPATCH_SPLIT(LPPV, ...)                              \
    switch (LPPV) {                                                \
    case 2: { constexpr int LPP_ = 2; __VA_ARGS__; break; }        \
    case 4: { constexpr int LPP_ = 4; __VA_ARGS__; break; }        \
    default: return hipErrorInvalidValue;                          \
    }

#define IOD_DISPATCH_LPP(LPPV, ...)                                \
    switch (LPPV) {                                                \
    case 1: { constexpr int LPP_ = 1; __VA_ARGS__; break; }        \
    case 2: { constexpr int LPP_ = 2; __VA_ARGS__; break; }        \
    case 4: { constexpr int LPP_ = 4; __VA_ARGS__; break; }        \
    default: return hipErrorInvalidValue;                          \
    }

}  // namespace iodk
