// lw_device.hpp -- device math of the Lienard-Wiechert path for gfx950.
//
// Retarded time (Eq. (ret_t)) by a safeguarded Newton iteration in FP64, the
// retarded kinematics of each trajectory family, and the Lienard-Wiechert
// potentials and fields (Eqs. (V), (A), (E), (ECoulomb), (Eradiation), (B)) in
// the working precision F (float for the mixed path, double for the FP64 path).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lw {

// CODATA 2018
constexpr double C_LIGHT = 299792458.0;
constexpr double INV_C = 1.0 / 299792458.0;
constexpr double EPS0 = 8.8541878128e-12;
constexpr double PI = 3.14159265358979323846;
constexpr double K_COUL = 1.0 / (4.0 * PI * EPS0);

enum { K_STATIONARY = 0, K_UNIFORM_VELOCITY = 1, K_LINEAR_OSC = 2, K_CIRCULAR = 3, K_ACCEL = 4 };
enum { F_TOTAL = 0, F_COULOMB = 1, F_RADIATION = 2 };
enum { FLAG_MASKED = 1u, FLAG_NOCONV = 2u };
enum { OUT_PHI = 1, OUT_A = 2, OUT_E = 4, OUT_B = 8, OUT_S = 16 };

// Exchanges a of the lanes whose index has bit K (16 or 32) with b of the lanes K below them:
// one v_permlane swap per 32-bit half.  (A host-only build compiles the device pass for
// a default architecture without these instructions, hence the second form.)
template <int K> __device__ __forceinline__ void lane_swap(double &a, double &b)
{
#if __has_builtin(__builtin_amdgcn_permlane32_swap) && __has_builtin(__builtin_amdgcn_permlane16_swap)
    auto swap = [](int x, int y) {
        if constexpr (K == 32) return __builtin_amdgcn_permlane32_swap((unsigned)x, (unsigned)y, false, false);
        else return __builtin_amdgcn_permlane16_swap((unsigned)x, (unsigned)y, false, false);
    };
    const auto lo = swap(__double2loint(a), __double2loint(b)), hi = swap(__double2hiint(a), __double2hiint(b));
    a = __hiloint2double((int)hi[0], (int)lo[0]);
    b = __hiloint2double((int)hi[1], (int)lo[1]);
#else
    const double from_b = __shfl_xor(b, K, 64), from_a = __shfl_xor(a, K, 64);
    if (threadIdx.x & K) a = from_b;
    else b = from_a;
#endif
}

// Per (time, charge) source record, written by the preparation kernel and read
// wave-uniformly (scalar loads) by the field kernels.
struct alignas(16) SrcRec {
    int32_t kind;
    float kqf;        // kq in FP32 (mixed path)
    double kq;        // q / (4 pi eps0)
    double t;         // observation time
    double c0[3];
    double e1[3];
    double e2[3];
    // circular, linear: omega / c, its square, 2 amp omega^2 / c^2 (geo_prepare_k)
    double koc, koc2, akoc;
    double amp, omega;  // uniform velocity: c^2 - |v|^2 and its reciprocal (rcp_steer)
    double cT, sT;    // cos, sin of Theta = omega t + phase
    double accel;     // circular, linear: ORBIT_TAB / (2 pi) omega / c
    double Lmax;      // accel: distance travelled along e1 by time t; circular, linear: 1 / omega
    double v[3];      // circular, linear: amp e1
    double rt[3];     // uniform velocity: position at time t; circular: amp e2; linear: rt[0] = (amp omega / c)^2
    // FP32 coefficients of beta and beta_dot (mixed path) in the orbit frame:
    // circular  beta = -s bw1 + c bw2,  beta_dot = -(c aw1 + s aw2);
    // linear    beta = -s bw1,          beta_dot = -c aw1;
    // bw = amp omega / c * e, aw = amp omega^2 / c * e; uniform velocity: bw1 = beta;
    // accel: bw1 = e1, aw1 = accel / c * e1
    float bw1[3], bw2[3], aw1[3], aw2[3];
    float omb;        // circular, uniform velocity: 1 - |beta|^2
};

// Retarded kinematics seen from the observation point: R = x - r(t'),
// velocity and acceleration of the charge at t' (Sec. 2.1).
struct Kin {
    double R[3];
    double v[3];        // FP64 path
    double a[3];
    float bf[3], df[3]; // mixed path: beta = v / c and beta_dot = a / c in FP32
    float omb;          // mixed path: 1 - |beta|^2
    double tp;          // retarded time t'
    double cph, sph;    // cos, sin of the phase at t' (oscillating families)
    uint32_t flags;
    int iters;          // solver iterations taken (ITER_FALLBACK set when the mixed path
                        // fell back to the safeguarded solver); read only by the
                        // iteration-histogram kernels, dead code elsewhere
};

constexpr int ITER_FALLBACK = 1 << 16;

// a * b + k with the constant k read from a scalar register pair.  Polynomial
// coefficients used this way stay out of vector registers: held there, every
// accumulate would first need a copy of its coefficient (the two-address form
// overwrites the addend), and the coefficients would take ~30 VGPRs.
__device__ __forceinline__ double fma_k(double a, double b, double k)
{
    double r;
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "s"(k));
    return r;
}

// sin and cos of a small angle from their Taylor series (terms through x^17 and x^16;
// the truncation error is below 1e-18 for |x| <= 0.75 and 9e-16 for |x| <= 1.1).
__device__ __forceinline__ void sincos_small(double x, double &s, double &c)
{
    const double x2 = x * x;
    double ps = fma_k(x2, -1.0 / 355687428096000.0, 1.0 / 1307674368000.0);   // -1/17!, 1/15!
    ps = fma_k(ps, x2, -1.0 / 6227020800.0);       // -1/13!
    ps = fma_k(ps, x2, 1.0 / 39916800.0);          //  1/11!
    ps = fma_k(ps, x2, -1.0 / 362880.0);           // -1/9!
    ps = fma_k(ps, x2, 1.0 / 5040.0);              //  1/7!
    ps = fma_k(ps, x2, -1.0 / 120.0);
    ps = fma_k(ps, x2, 1.0 / 6.0);
    // ps now holds 1/3! - x^2/5! + ...; sin x = x - x^3 * ps
    s = fma(-x * x2, ps, x);
    double pc = fma_k(x2, 1.0 / 20922789888000.0, -1.0 / 87178291200.0);       // 1/16!, -1/14!
    pc = fma_k(pc, x2, 1.0 / 479001600.0);         //  1/12!
    pc = fma_k(pc, x2, -1.0 / 3628800.0);          // -1/10!
    pc = fma_k(pc, x2, 1.0 / 40320.0);             //  1/8!
    pc = fma_k(pc, x2, -1.0 / 720.0);              // -1/6!
    pc = fma_k(pc, x2, 1.0 / 24.0);                //  1/4!
    pc = fma(pc, x2, -0.5);                        // -1/2!
    c = fma(pc, x2, 1.0);
}

// sin and cos for |x| < 2^30: x = k pi/2 + r with pi/2 split into three
// doubles (FMA Cody-Waite reduction, |r| <= pi/4), the Taylor kernel on r, then
// the quadrant's swap and signs.
__device__ __forceinline__ void sincos_reduced(double x, double &s, double &c)
{
    const double P1 = 0x1.921fb54442d18p+0;     // pi/2 = P1 + P2 + P3
    const double P2 = 0x1.1a62633145c07p-54;
    const double P3 = -0x1.f1976b7ed8fbcp-110;
    const double k = rint(x * 0x1.45f306dc9c883p-1);   // x * 2/pi
    double r = fma(-k, P1, x);
    r = fma(-k, P2, r);
    r = fma(-k, P3, r);
    double sr, cr;
    sincos_small(r, sr, cr);
    const int q = (int)k & 3;
    const double a = (q & 1) ? cr : sr;          // |sin x|, |cos x| up to sign
    const double b = (q & 1) ? sr : cr;
    s = (q & 2) ? -a : a;
    c = ((q + 1) & 2) ? -b : b;
}

// Square root for bounds and starting values only (v_sqrt_f64, relative error
// near 2^-22): callers widen what they derive from it.
__device__ __forceinline__ double sqrt_rough(double x) { return __builtin_amdgcn_sqrt(x); }

// Trig state (cos, sin) of theta' = Theta - omega*tau kept across Newton
// updates: small changes rotate it, large ones recompute it.
struct Phase {
    double c, s;
    // from cw, sw = cos, sin(omega tau)
    __device__ __forceinline__ void set_from(const SrcRec &S, double cw, double sw)
    {
        c = S.cT * cw + S.sT * sw;      // cos(Theta - w tau)
        s = S.sT * cw - S.cT * sw;      // sin(Theta - w tau)
    }
    __device__ __forceinline__ void set(const SrcRec &S, double tau)
    {
        double sw, cw;
        sincos_reduced(S.omega * tau, sw, cw);
        set_from(S, cw, sw);
    }
    __device__ __forceinline__ void advance(const SrcRec &S, double tau_new, double dtau)
    {
        const double ang = -S.omega * dtau;    // theta' moves by -omega * dtau
        if (fabs(ang) <= 0x1p-8) {
            // |ang| <= 2^-8: Taylor through x^7 and x^6 (truncation below 5e-25)
            const double a2 = ang * ang;
            const double sa = fma(-ang * a2, fma_k(fma_k(a2, -1.0 / 5040.0, 1.0 / 120.0), -a2, 1.0 / 6.0), ang);
            const double ca = fma(a2, fma(a2, fma_k(a2, -1.0 / 720.0, 1.0 / 24.0), -0.5), 1.0);
            const double cn = c * ca - s * sa;
            const double sn = s * ca + c * sa;
            c = cn;
            s = sn;
        } else if (fabs(ang) <= 0.75) {
            double sa, ca;
            sincos_small(ang, sa, ca);
            const double cn = c * ca - s * sa;
            const double sn = s * ca + c * sa;
            c = cn;
            s = sn;
        } else {
            set(S, tau_new);
        }
    }
};

// Root bracket of g(tau) = c tau - D(tau): g < 0 below the root, g > 0 above
// (g' >= c - |v| > 0).  The ends start as geometric bounds; an end is
// "evaluated" once an iterate has landed there.
struct Bracket {
    double lo, hi;
    bool lo_ev, hi_ev;
    __device__ __forceinline__ Bracket(double l, double h) : lo(l), hi(h), lo_ev(false), hi_ev(false) {}
};

// Reciprocal for derivative terms and step sizes (v_rcp_f64 refined by one
// Newton-Raphson step): these only steer the iteration, the root itself is
// decided by g = c tau - D, which is evaluated exactly.
__device__ __forceinline__ double rcp_steer(double x)
{
    const double r = __builtin_amdgcn_rcp(x);
    return fma(r, fma(-x, r, 1.0), r);
}

// |x| and 1/|x| from s = |x|^2 (s > 0 and normal): v_rsq_f64 refined by one
// Goldschmidt step (both the root and the half-reciprocal), then Newton
// corrections of the root on its residual s - r^2.  FULL takes two corrections
// (the root to about one ulp, for the FP64 tolerance), otherwise one (relative
// error far below the 2^-32 tolerance of the mixed path).  The reciprocal keeps
// the Goldschmidt step's accuracy, which is what steering terms need.
template <bool FULL>
__device__ __forceinline__ void root_rsqrt(double s, double &r, double &ir)
{
    const double y = __builtin_amdgcn_rsq(s);
    double g = s * y, h = 0.5 * y;
    const double e = fma(-g, h, 0.5);
    g = fma(g, e, g);
    h = fma(h, e, h);
    g = fma(fma(-g, g, s), h, g);
    if (FULL) g = fma(fma(-g, g, s), h, g);
    r = g;
    ir = 2.0 * h;
}

// One safeguarded Halley update of g(tau) = c tau - D(tau) with g' = c - D'
// and g'' = -D''.  An exact root, or a step below the rounding of tau, returns
// tau itself (converged).  The Halley step is used while its denominator stays
// above g'^2 (the step is then at most twice Newton's), else Newton's.  A step
// leaving the bracket goes to the nearer end if that end has not been
// evaluated yet (the geometric bounds are often close to the root), otherwise
// bisects; so does a step onto an end already evaluated.  `free_step` reports
// whether the returned iterate is the plain Halley/Newton step (not moved onto
// the bracket).
__device__ __forceinline__ double halley_step(double tau, double D, double dD, double ddD, Bracket &b,
                                              bool &free_step)
{
    free_step = true;
    const double g = C_LIGHT * tau - D;
    if (g == 0.0) return tau;
    if (g < 0.0) {
        b.lo = tau;
        b.lo_ev = true;
    } else {
        b.hi = tau;
        b.hi_ev = true;
    }
    const double gp = C_LIGHT - dD;
    const double gp2 = gp * gp;
    const double den = fma(2.0 * gp, gp, g * ddD);          // 2 g'^2 - g g''
    // Newton's step is the same formula with the denominator 2 g'^2
    double tn = tau - 2.0 * g * gp * rcp_steer((den > gp2) ? den : 2.0 * gp2);
    if (tn == tau) return tau;
    // landing on an evaluated end again would cycle: bisect instead
    if (tn <= b.lo) {
        tn = b.lo_ev ? 0.5 * (b.lo + b.hi) : b.lo;
        free_step = false;
    } else if (tn >= b.hi) {
        tn = b.hi_ev ? 0.5 * (b.lo + b.hi) : b.hi;
        free_step = false;
    }
    return tn;
}

// Converged when the last step is below tol_rel (relative), or when both
// bracket ends have been evaluated and lie within 4 tol_rel of each other
// (rounding noise in D can make the last steps alternate around the root).
__device__ __forceinline__ bool converged(double tn, double tau, double tol_rel, const Bracket &b)
{
    return fabs(tn - tau) <= tol_rel * tn || (b.lo_ev && b.hi_ev && b.hi - b.lo <= 4.0 * tol_rel * tn);
}

// A-posteriori stop for trajectories whose g is smooth in tau (circular and
// linear oscillation, either side of the start of uniform acceleration): from
// tau, Newton's step leaves an error of about |g''| / (2 g') dtau^2 and
// Halley's a smaller (cubic) one, so once that bound is below tol/4 the new
// iterate is accepted without evaluating D at it.  Only a free (unclamped)
// step qualifies; a clamped or bisection step ends the iteration once it is
// below tol (rounding noise near the root gives free steps of a few ulp, which
// the bound accepts).
__device__ __forceinline__ bool converged_smooth(double tn, double tau, double tol_rel, const Bracket &b,
                                                 bool free_step, double dD, double ddD)
{
    const double st = tn - tau;
    return fabs(st) <= tol_rel * tn || (free_step && fabs(ddD) * (st * st) <= 0.5 * tol_rel * tn * (C_LIGHT - dD));
}

// cos and sin of 2 pi k / ORBIT_TAB, the phases that starting values lie on.
constexpr int ORBIT_TAB = 128;
constexpr double TWO_PI = 6.28318530717958647692;

constexpr double series_sin(double x)       // |x| <= pi / 4, to rounding
{
    double term = x, sum = x;
    for (int n = 1; n < 12; ++n) {
        term *= -x * x / (2.0 * n * (2.0 * n + 1.0));
        sum += term;
    }
    return sum;
}
constexpr double series_cos(double x)
{
    double term = 1.0, sum = 1.0;
    for (int n = 1; n < 12; ++n) {
        term *= -x * x / (2.0 * n * (2.0 * n - 1.0));
        sum += term;
    }
    return sum;
}
struct OrbitTable {
    double cs[ORBIT_TAB][2];
    constexpr OrbitTable() : cs{}
    {
        for (int k = 0; k < ORBIT_TAB; ++k) {
            // nearest quadrant's axis plus a remainder of at most pi / 4
            const int q = (k + ORBIT_TAB / 8) / (ORBIT_TAB / 4);
            const double r = TWO_PI / ORBIT_TAB * (k - q * (ORBIT_TAB / 4));
            const double c = series_cos(r), s = series_sin(r);
            cs[k][0] = (q & 1) ? ((q & 2) ? s : -s) : ((q & 2) ? -c : c);
            cs[k][1] = (q & 1) ? ((q & 2) ? -c : c) : ((q & 2) ? -s : s);
        }
    }
};
__device__ const OrbitTable orbit_table{};

// Part of a source's retarded-time problem that does not depend on the
// observation time, for one observation point.  Field kernels build it once per
// (point, charge) and reuse it for every time.
//
// Circular and linear orbits: the retarded time is sought as a phase, T = omega
// tau = T0 + a, about a start T0: the light time from the orbit's RMS distance,
// beyond the near field moved to the grid of 2 pi / ORBIT_TAB.  With theta = Theta -
// T the condition (c tau)^2 = D^2, in units of c / omega, reads
//   g(a) = a (2 T0 + a) + G(theta) - K = 0,
// circular:  G = w1b cos theta + w2b sin theta,  K = (|w|^2 + A^2) (omega / c)^2 - T0^2,
// linear:    G = w1b cos theta - beta^2 cos^2 theta,  K = |w|^2 (omega / c)^2 - T0^2,
// with w1b = 2 beta (omega / c) w.e1, w2b likewise, beta = A omega / c.  g needs no
// square root, has the root of Eq. (ret_t) as its only root with tau > 0, and needs
// no division here.  A start on the grid costs one table entry instead of a sine
// and cosine (27 VALU instructions per (point, charge)) and moves |a| by at most
// pi / ORBIT_TAB.
struct Geo {
    double w[3];      // x - c0
    double w1, w2;    // accel: w along e1, distance^2 from the axis
    double T2;        // 2 T0
    double cw, sw;    // cos, sin of T0
    double w1b, w2b, K;
};

template <int KIND>
__device__ __forceinline__ void geo_prepare_k(const SrcRec &S, const double x[3], Geo &g)
{
    for (int i = 0; i < 3; ++i) g.w[i] = x[i] - S.c0[i];
    const double *w = g.w;
    if constexpr (KIND == K_CIRCULAR || KIND == K_LINEAR_OSC) {
        const double W = w[0] * w[0] + w[1] * w[1] + w[2] * w[2];
        const double w1 = w[0] * S.e1[0] + w[1] * S.e1[1] + w[2] * S.e1[2];
        const double A2 = S.amp * S.amp, WA = KIND == K_CIRCULAR ? W + A2 : W;
        // RMS distance to the orbit (omega = 0 gives T0 = 0 and a solve that is never
        // accepted; the safeguarded solver takes it)
        const double rms = sqrt_rough(KIND == K_CIRCULAR ? WA : fma(0.5, A2, W));
        const double kk = rint(rms * S.accel);
        if (fabs(kk) < 15.0) {
            // near field (|T0| < 0.72): the grid is coarse against T0 there
            const double T0 = rms * S.koc;
            g.T2 = T0 + T0;
            sincos_small(T0, g.sw, g.cw);
        } else {
            const uint32_t o = (uint32_t)(__builtin_amdgcn_fract(kk * (1.0 / ORBIT_TAB)) * (double)(ORBIT_TAB * 16));
            const double *cs = (const double *)((const char *)orbit_table.cs + o);
            g.cw = cs[0];
            g.sw = cs[1];
            g.T2 = kk * (2.0 * TWO_PI / ORBIT_TAB);
        }
        g.w1b = w1 * S.akoc;
        if constexpr (KIND == K_CIRCULAR)
            g.w2b = (w[0] * S.e2[0] + w[1] * S.e2[1] + w[2] * S.e2[2]) * S.akoc;
        g.K = fma(-0.25 * g.T2, g.T2, WA * S.koc2);
    } else if constexpr (KIND == K_ACCEL) {
        g.w1 = w[0] * S.e1[0] + w[1] * S.e1[1] + w[2] * S.e1[2];
        const double p0 = w[0] - g.w1 * S.e1[0], p1 = w[1] - g.w1 * S.e1[1], p2 = w[2] - g.w1 * S.e1[2];
        g.w2 = p0 * p0 + p1 * p1 + p2 * p2;
    }
}

// The point in the orbit's frame with the geometric bracket on tau and a start,
// for the safeguarded solvers (circular, linear).  The start is the RMS distance
// to the orbit over c: the mean of the squared distance lies between its least
// and greatest values, so the clamp to the bracket never moves it.
struct GeoSafe {
    double w[3];      // x - c0
    double w1, w2, w3;// circular: coordinates along e1, e2, e1 x e2; linear: w1 along e1, w2 = distance^2 from the axis
    double lo, hi;    // bracket on tau
    double tau0;      // starting value
    double cw, sw;    // cos, sin of omega tau0
};

template <int KIND>
__device__ __forceinline__ void geo_safe(const SrcRec &S, const double x[3], GeoSafe &g)
{
    for (int i = 0; i < 3; ++i) g.w[i] = x[i] - S.c0[i];
    const double *w = g.w;
    const double A = S.amp;
    g.w1 = w[0] * S.e1[0] + w[1] * S.e1[1] + w[2] * S.e1[2];
    const double w1 = g.w1;
    if constexpr (KIND == K_CIRCULAR) {
        const double w2 = w[0] * S.e2[0] + w[1] * S.e2[1] + w[2] * S.e2[2];
        const double w3 = w[0] * (S.e1[1] * S.e2[2] - S.e1[2] * S.e2[1]) +
                          w[1] * (S.e1[2] * S.e2[0] - S.e1[0] * S.e2[2]) +
                          w[2] * (S.e1[0] * S.e2[1] - S.e1[1] * S.e2[0]);
        g.w2 = w2;
        g.w3 = w3;
        const double rho = sqrt_rough(w1 * w1 + w2 * w2);
        // the distance to the orbit lies between these, so c tau does too
        // (widened by 1e-6 to cover the rough square roots; next to the orbit rho's
        // error is of the size of rho, not of rho - A)
        const double gap = fmax(fabs(rho - A) - 1e-6 * rho, 0.0);
        g.lo = sqrt_rough(w3 * w3 + gap * gap) * (INV_C * (1.0 - 1e-6));
        g.hi = sqrt_rough(w3 * w3 + (rho + A) * (rho + A)) * (INV_C * (1.0 + 1e-6));
        g.tau0 = fmin(fmax(sqrt_rough(w1 * w1 + w2 * w2 + w3 * w3 + A * A) * INV_C, g.lo), g.hi);
    } else {
        const double p0 = w[0] - w1 * S.e1[0], p1 = w[1] - w1 * S.e1[1], p2 = w[2] - w1 * S.e1[2];
        const double perp2 = p0 * p0 + p1 * p1 + p2 * p2;     // distance^2 from the axis line
        g.w2 = perp2;
        g.w3 = 0.0;
        const double W2 = perp2 + w1 * w1;
        const double u = fmin(fmax(w1, -A), A);
        g.lo = sqrt_rough(perp2 + (w1 - u) * (w1 - u)) * (INV_C * (1.0 - 1e-6));
        g.hi = sqrt_rough(W2 + A * A + 2.0 * A * fabs(w1)) * (INV_C * (1.0 + 1e-6));
        g.tau0 = fmin(fmax(sqrt_rough(W2 + 0.5 * A * A) * INV_C, g.lo), g.hi);
    }
    sincos_reduced(S.omega * g.tau0, g.sw, g.cw);
}

// --- circular orbit: r = c0 + amp (cos th e1 + sin th e2), th = Theta - w tau ---
template <bool FULL>
__device__ __forceinline__ void solve_circular(const SrcRec &S, const GeoSafe &g, int max_iter, double tol_rel, Kin &k)
{
    const double A = S.amp, om = S.omega;
    const double w1 = g.w1, w2 = g.w2, w3 = g.w3;
    Bracket b(g.lo, g.hi);
    double tau = g.tau0;
    Phase ph;
    ph.set_from(S, g.cw, g.sw);
    bool ok = (b.hi == b.lo);
    int n_it = 0;
    for (int it = 0; it < max_iter && !ok; ++it) {
        ++n_it;
        // R = x - r(t') in the orbit frame (no cancellation near the orbit)
        const double x1 = w1 - A * ph.c, x2 = w2 - A * ph.s;
        double D, iD;
        root_rsqrt<FULL>(fmax(x1 * x1 + x2 * x2 + w3 * w3, 1e-300), D, iD);
        const double Q = ph.c * x2 - ph.s * x1;              // D' = n . v = A w Q / D
        const double P = w1 * ph.c + w2 * ph.s;              // D'' = (A w^2 P - D'^2) / D
        const double dD = A * om * Q * iD;
        const double ddD = (A * om * om * P - dD * dD) * iD;
        bool free_step;
        const double tn = halley_step(tau, D, dD, ddD, b, free_step);
        ph.advance(S, tn, tn - tau);
        ok = converged_smooth(tn, tau, tol_rel, b, free_step, dD, ddD);
        tau = tn;
    }
    k.flags = ok ? 0u : FLAG_NOCONV;
    k.iters = n_it;
    k.tp = S.t - tau;
    k.cph = ph.c;
    k.sph = ph.s;
    if (FULL) {
        double ro[3], vo[3];
        for (int i = 0; i < 3; ++i) {
            ro[i] = A * (ph.c * S.e1[i] + ph.s * S.e2[i]);
            vo[i] = A * (-ph.s * S.e1[i] + ph.c * S.e2[i]);
            k.R[i] = g.w[i] - ro[i];
            k.v[i] = om * vo[i];
            k.a[i] = -om * om * ro[i];
        }
    } else {
        const float cf = (float)ph.c, sf = (float)ph.s;
        for (int i = 0; i < 3; ++i) {
            k.R[i] = g.w[i] - A * (ph.c * S.e1[i] + ph.s * S.e2[i]);
            k.bf[i] = cf * S.bw2[i] - sf * S.bw1[i];
            k.df[i] = -(cf * S.aw1[i] + sf * S.aw2[i]);
        }
        k.omb = S.omb;
    }
}

// --- linear oscillation: r = c0 + amp cos th e1 ---
template <bool FULL>
__device__ __forceinline__ void solve_linear(const SrcRec &S, const GeoSafe &g, int max_iter, double tol_rel, Kin &k)
{
    const double A = S.amp, om = S.omega;
    const double w1 = g.w1, perp2 = g.w2;
    Bracket b(g.lo, g.hi);
    double tau = g.tau0;
    Phase ph;
    ph.set_from(S, g.cw, g.sw);
    bool ok = (b.hi == b.lo);
    int n_it = 0;
    for (int it = 0; it < max_iter && !ok; ++it) {
        ++n_it;
        const double x1 = w1 - A * ph.c;                     // R . e1
        double D, iD;
        root_rsqrt<FULL>(fmax(perp2 + x1 * x1, 1e-300), D, iD);
        const double v1 = A * om * ph.s;                     // d x1 / d tau = -v1
        const double dD = -v1 * x1 * iD;
        const double ddD = (v1 * v1 + x1 * A * om * om * ph.c - dD * dD) * iD;
        bool free_step;
        const double tn = halley_step(tau, D, dD, ddD, b, free_step);
        ph.advance(S, tn, tn - tau);
        ok = converged_smooth(tn, tau, tol_rel, b, free_step, dD, ddD);
        tau = tn;
    }
    k.flags = ok ? 0u : FLAG_NOCONV;
    k.iters = n_it;
    k.tp = S.t - tau;
    k.cph = ph.c;
    k.sph = ph.s;
    if (FULL) {
        for (int i = 0; i < 3; ++i) {
            k.R[i] = g.w[i] - A * ph.c * S.e1[i];
            k.v[i] = -A * om * ph.s * S.e1[i];
            k.a[i] = -A * om * om * ph.c * S.e1[i];
        }
    } else {
        const float cf = (float)ph.c, sf = (float)ph.s;
        for (int i = 0; i < 3; ++i) {
            k.R[i] = g.w[i] - A * ph.c * S.e1[i];
            k.bf[i] = -sf * S.bw1[i];
            k.df[i] = -cf * S.aw1[i];
        }
        k.omb = fmaf(-(float)S.rt[0] * sf, sf, 1.f);
    }
}

// --- uniform acceleration from rest at t = 0 along e1 ---
template <bool FULL>
__device__ __forceinline__ void solve_accel(const SrcRec &S, const Geo &g, int max_iter, double tol_rel, Kin &k)
{
    const double acc = S.accel, L = S.Lmax, t = S.t;
    const double w1 = g.w1, perp2 = g.w2;
    const double W2 = perp2 + w1 * w1;
    // positions up to time t fill the segment [0, L] along e1
    const double u = fmin(fmax(w1, 0.0), L);
    const double Dnow = sqrt_rough(perp2 + (w1 - L) * (w1 - L));   // distance to the position at t
    Bracket b(sqrt_rough(perp2 + (w1 - u) * (w1 - u)) * (INV_C * (1.0 - 1e-6)),
              fmax(sqrt_rough(W2), Dnow) * (INV_C * (1.0 + 1e-6)));
    double tau = fmin(fmax(Dnow * INV_C, b.lo), b.hi);
    bool ok = (b.hi == b.lo);
    int n_it = 0;
    for (int it = 0; it < max_iter && !ok; ++it) {
        ++n_it;
        const double tp = t - tau;
        const double s = (tp > 0.0) ? 0.5 * acc * tp * tp : 0.0;   // distance along e1
        const double vel = (tp > 0.0) ? acc * tp : 0.0;
        const double x1 = w1 - s;
        double D, iD;
        root_rsqrt<FULL>(fmax(perp2 + x1 * x1, 1e-300), D, iD);
        const double dD = vel * x1 * iD;                      // d x1 / d tau = vel
        const double ddD = (vel * vel - ((tp > 0.0) ? acc * x1 : 0.0) - dD * dD) * iD;
        bool free_step;
        const double tn = halley_step(tau, D, dD, ddD, b, free_step);
        // g is smooth on either side of t' = 0 (the start of the motion), so the
        // a-posteriori stop applies to a step that stays on one side
        ok = converged_smooth(tn, tau, tol_rel, b, free_step && ((t - tn > 0.0) == (tp > 0.0)), dD, ddD);
        tau = tn;
    }
    k.flags = ok ? 0u : FLAG_NOCONV;
    k.iters = n_it;
    const double tp = t - tau;
    k.tp = tp;
    k.cph = 1.0;
    k.sph = 0.0;
    const double s = (tp >= 0.0) ? 0.5 * acc * tp * tp : 0.0;
    const double vel = (tp >= 0.0) ? acc * tp : 0.0;
    const double ac = (tp >= 0.0) ? acc : 0.0;
    for (int i = 0; i < 3; ++i) {
        k.R[i] = g.w[i] - s * S.e1[i];
        k.v[i] = vel * S.e1[i];
        k.a[i] = ac * S.e1[i];
    }
}

// --- uniform velocity: |wt + v tau| = c tau has a closed-form root ---
// FULL: correctly rounded square root and division; otherwise (the mixed path,
// whose field is FP32) the refined v_rsq_f64 root and v_rcp_f64 reciprocal,
// within a few ulp, which is all the mixed tolerance needs.
// The record holds den = c^2 - |v|^2 (amp) and its reciprocal (omega), which
// do not depend on the point.
template <bool FULL>
__device__ __forceinline__ void solve_uniform(const SrcRec &S, const double x[3], Kin &k)
{
    double wt[3];
    for (int i = 0; i < 3; ++i) wt[i] = x[i] - S.rt[i];
    const double wv = wt[0] * S.v[0] + wt[1] * S.v[1] + wt[2] * S.v[2];
    const double ww = wt[0] * wt[0] + wt[1] * wt[1] + wt[2] * wt[2];
    const double den = S.amp;
    const double disc = wv * wv + den * ww;
    double sq, isq;
    if (FULL) sq = sqrt(disc);
    else root_rsqrt<false>(fmax(disc, 1e-300), sq, isq);
    // the two algebraically equal forms, chosen to avoid cancellation
    const double tau = FULL ? ((wv >= 0.0) ? (wv + sq) / den : ww / (sq - wv))
                            : ((wv >= 0.0) ? (wv + sq) * S.omega : ww * rcp_steer(sq - wv));
    k.tp = S.t - tau;
    k.cph = 1.0;
    k.sph = 0.0;
    for (int i = 0; i < 3; ++i) {
        k.R[i] = wt[i] + S.v[i] * tau;
        k.v[i] = S.v[i];
        k.a[i] = 0.0;
    }
    k.flags = 0u;
    k.iters = 0;
}

// The next iterate's distance from a root of a function with Taylor coefficients
// F[0..N-1] (F[k] = f^(k) / k!): the root of the Pade approximant of 1 / f's
// series (Householder's method of order N), -F0 D_{N-2} / D_{N-1} with D_0 = 1,
// D_k = sum_i (-1)^(i-1) F0^(i-1) F_i D_{k-i}.  The error left is of the order of
// the N-th power of the error before.  Returns numerator and denominator.
template <int N, typename F>
__device__ __forceinline__ void pade_step(const F c[5], F &num, F &den)
{
    static_assert(N >= 3 && N <= 5, "");
    const F x2 = c[0] * c[2];
    const F d2 = c[1] * c[1] - x2;
    if constexpr (N == 3) {
        num = -c[0] * c[1];
        den = d2;
    } else {
        const F f2 = c[0] * c[0];
        const F x3 = f2 * c[3];
        const F d3 = c[1] * (d2 - x2) + x3;
        if constexpr (N == 4) {
            num = -c[0] * d2;
            den = d3;
        } else {
            const F x4 = f2 * c[0] * c[4];
            num = -c[0] * d3;
            den = c[1] * (d3 + x3) - x2 * d2 - x4;
        }
    }
}

// Taylor coefficients of g (Geo) at a, phase (c, s) = (cos, sin) theta, in precision
// F.  b2 = beta^2 (linear).
template <int KIND, int N, typename F>
__device__ __forceinline__ void orbit_taylor(F w1b, F w2b, F b2, F T2, F K, F a, F c, F s, F g[5])
{
    if constexpr (KIND == K_CIRCULAR) {
        const F P = w1b * c + w2b * s, Q = w2b * c - w1b * s;      // dP/da = -Q, dQ/da = P
        g[0] = a * (T2 + a) + (P - K);
        g[1] = (F)2 * a + (T2 - Q);
        g[2] = (F)-0.5 * P + (F)1;
        if constexpr (N >= 4) g[3] = Q * (F)(1.0 / 6.0);
        if constexpr (N >= 5) g[4] = P * (F)(1.0 / 24.0);
    } else {
        const F bc = b2 * c, bs = b2 * s, y = w1b - bc;            // y - bc = -dG / d cos theta
        const F cy = c * (y - bc) + (F)2 * bs * s;                 // -G''
        g[0] = a * (T2 + a) + (c * y - K);
        g[1] = (F)2 * a + (s * (y - bc) + T2);
        g[2] = (F)-0.5 * cy + (F)1;
        if constexpr (N >= 4) g[3] = s * ((F)7 * bc - y) * (F)(1.0 / 6.0);
        if constexpr (N >= 5) g[4] = (cy - (F)6 * (bc * c - bs * s)) * (F)(1.0 / 24.0);
    }
}

// (cos, sin) of theta0 - a from (c0, s0) = (cos, sin) theta0, |a| <= 0.75.  The polynomials'
// lowest terms are Taylor's, the others those of least maximal error over the range
// (Remez's exchange): sin through a^13 and cos through a^12 to 4.1e-17, for the mixed
// path (SHORT) through a^9 and a^10 to 1.5e-12, against FP32 outputs.  (Taylor's own
// coefficients through a^11 and a^12 leave 4e-12 at 0.75 and 2e-14 at 0.5.)
template <bool SHORT>
__device__ __forceinline__ void rot_phase(double c0, double s0, double a, double &c, double &s)
{
    const double a2 = a * a;
    double sa, ca;
    if constexpr (SHORT) {
        sa = fma_k(fma_k(fma_k(a2, 0x1.6d0107747315cp-19, -0x1.a0100f79c206ep-13), a2, 0x1.111108c357014p-7), a2,
                   -0x1.5555554c2328fp-3);
        ca = fma_k(fma_k(fma_k(a2, -0x1.247e88251427ap-22, 0x1.a0129e2b6279ap-16), a2, -0x1.6c16baba0e016p-10), a2,
                   0x1.5555555129dd0p-5);
    } else {
        sa = fma_k(fma_k(a2, 0x1.5db8f28b864f3p-33, -0x1.ae5ed1ace9646p-26), a2, 0x1.71de35e02ff18p-19);
        sa = fma_k(fma_k(fma_k(sa, a2, -0x1.a01a019c5e2e3p-13), a2, 0x1.111111110f91fp-7), a2, -0x1.5555555555548p-3);
        ca = fma_k(fma_k(a2, 0x1.1c0e6d755a142p-29, -0x1.27e0f99997faep-22), a2, 0x1.a019fc581f90fp-16);
        ca = fma_k(fma_k(ca, a2, -0x1.6c16c168dbc4dp-10), a2, 0x1.5555555553e74p-5);
    }
    sa = a * fma(a2, sa, 1.0);
    ca = fma(a2, fma(a2, ca, -0.5), 1.0);
    c = c0 * ca + s0 * sa;
    s = s0 * ca - c0 * sa;
}

// One step e of order N = 3 (mixed path) or 4 (FULL) towards the root of g (Geo) in FP64
// from a, whose phase is turned there from (c0, s0); (c, s) is that phase.  Returns whether
// a has settled:
//   |g| < E g',  |g g''| / 2 <= H (g'^2 - g g'' / 2).
// The second is Kantorovich's condition on Newton's step: met with H far below 1/4, a root
// lies about g / g' away, of which a step of order N leaves H^(N - 1).  So the error is
// relative to the root itself where g bends most: next to a slow orbit g is T^2 less the
// squared distance, g' = 2 T, and 2 H^N T is left, 4e-12 T or 4e-16 T.  The first bounds the
// step for the short rotation that follows, and demands g' > 0, which the mirror root at
// T < 0 does not have (omega < 0 turns both signs).  The step's own size would prove
// neither: it is an absolute phase, which next to a slow charge all of T is below, and it
// vanishes where its numerator does, root or not.  WIDE (the further steps): |a| up to 1.1, by
// longer series, which holds the roots of all but points close to the fastest orbits (|a|
// is at most beta away from the orbit, sqrt 2 beta on it, and pi / 128 for the grid);
// otherwise up to 0.75.
template <int KIND, bool FULL, bool WIDE>
__device__ __forceinline__ bool orbit_step(const SrcRec &S, const Geo &g, double c0, double s0, double a, double &c,
                                           double &s, double &e)
{
    constexpr int N = FULL ? 4 : 3;
    constexpr double H = 0x1p-13;
    const double E = copysign(0x1p-12, S.omega);
    double t[5], num, den;
    if constexpr (WIDE) {
        double sa, ca;
        sincos_small(a, sa, ca);
        c = c0 * ca + s0 * sa;
        s = s0 * ca - c0 * sa;
    } else {
        rot_phase<!FULL>(c0, s0, a, c, s);
    }
    orbit_taylor<KIND, N, double>(g.w1b, g.w2b, KIND == K_LINEAR_OSC ? S.rt[0] : 0.0, g.T2, g.K, a, c, s, t);
    pade_step<N, double>(t, num, den);
    // v_rcp_f64 unrefined (relative error below 2^-26) for the mixed path
    e = num * (FULL ? rcp_steer(den) : __builtin_amdgcn_rcp(den));
    const double x2 = t[0] * t[2], d2 = t[1] * t[1] - x2;
    return fabs(t[0]) < E * t[1] && fabs(x2) <= H * d2 && fabs(a) <= (WIDE ? 1.1 : 0.75);
}

// Circular and linear orbits: the root of g (Geo).  One step of order 5 in FP32 from a = 0,
// whose phase is known in FP64; then FP64 steps (orbit_step) until one settles, whose
// phase follows by a short rotation.  1 % of the waves of the grid workloads hold a lane
// that takes a second FP64 step, most waves beyond 0.7 c, where |a| leaves the first step's
// range; one that has not settled after four takes the safeguarded solver (false is
// returned).  512^2 x 16 x 16 orbits at 0.9 c, mixed, 0.37 ms, 0.72 with those lanes left to
// the safeguarded solver.
//
// VALU issue bounds the grid kernels, where an FP64 instruction costs as much as an
// FP32 one (v_rcp_f64 four, v_rcp_f32 two).  So steps of high order, whose extra
// terms cost two or three instructions each, replace further low-order steps,
// each of which evaluates the phase anew (about 36).  512^2 x 64 x 16 mixed grid, against
// FP32 Halley steps until one was below 2^-7 and one FP64 Newton step: 1.47 -> 1.22 to
// 1.26 ms per call by its mix of charges, FP64 75^3 x 5 x 16 volume 0.292 -> 0.226 ms.  The
// first FP64 step stands before the loop: as the loop's own first turn 1.32 ms on that
// grid, 1.29 so (both with steps of order 4).
template <int KIND, bool FULL>
__device__ __forceinline__ bool solve_orbit(const SrcRec &S, const Geo &g, Kin &k)
{
    // phase at T0 for this observation time (FP64)
    const double c0 = S.cT * g.cw + S.sT * g.sw;
    const double s0 = S.sT * g.cw - S.cT * g.sw;
    float t32[5], n32, d32;
    orbit_taylor<KIND, 5, float>((float)g.w1b, (float)g.w2b, KIND == K_LINEAR_OSC ? (float)S.rt[0] : 0.f, (float)g.T2,
                                 (float)g.K, 0.f, (float)c0, (float)s0, t32);
    pade_step<5, float>(t32, n32, d32);
    double a = (double)(n32 * __builtin_amdgcn_rcpf(d32));
    double c, s, e;
    int it = 1;
    bool ok = orbit_step<KIND, FULL, false>(S, g, c0, s0, a, c, s, e);
    while (!ok && it < 4) {
        ++it;
        a += e;
        ok = orbit_step<KIND, FULL, true>(S, g, c0, s0, a, c, s, e);
    }
    if (!ok) return false;
    a += e;
    {
        // to fourth order (truncation e^5 / 120 below 1e-19), mixed to second (e^3 / 6
        // below 3e-12)
        const double e2 = e * e;
        double ce, se;
        if constexpr (FULL) {
            ce = fma(e2, fma(e2, 1.0 / 24.0, -0.5), 1.0);
            se = e * fma(e2, -1.0 / 6.0, 1.0);
        } else {
            ce = fma(-0.5, e2, 1.0);
            se = e;
        }
        const double cn = c * ce + s * se, sn = s * ce - c * se;
        c = cn;
        s = sn;
    }
    k.flags = 0u;
    k.iters = 1 + it;
    k.tp = S.t - fma(0.5, g.T2, a) * S.Lmax;
    k.cph = c;
    k.sph = s;
    if constexpr (FULL) {
        const double A = S.amp, om = S.omega;
        const double vw = om * A, aw = -om * om;
        for (int i = 0; i < 3; ++i) {
            const double ro = KIND == K_CIRCULAR ? c * S.v[i] + s * S.rt[i] : c * S.v[i];
            k.R[i] = g.w[i] - ro;
            k.v[i] = KIND == K_CIRCULAR ? vw * (c * S.e2[i] - s * S.e1[i]) : -vw * s * S.e1[i];
            k.a[i] = aw * ro;
        }
    } else {
        const float cf = (float)c, sf = (float)s;
        for (int i = 0; i < 3; ++i) {
            if (KIND == K_CIRCULAR) {
                k.R[i] = fma(-s, S.rt[i], fma(-c, S.v[i], g.w[i]));
                k.bf[i] = cf * S.bw2[i] - sf * S.bw1[i];
                k.df[i] = -(cf * S.aw1[i] + sf * S.aw2[i]);
            } else {
                k.R[i] = fma(-c, S.v[i], g.w[i]);
                k.bf[i] = -sf * S.bw1[i];
                k.df[i] = -cf * S.aw1[i];
            }
        }
        k.omb = KIND == K_CIRCULAR ? S.omb : fmaf(-(float)S.rt[0] * sf, sf, 1.f);
    }
    return true;
}

// Uniform acceleration from rest at t = 0: where the point is at least c t away
// from the rest position, the retarded time lies before the start and tau = |w| / c.
// Elsewhere the charge sits at L - m along e1 at t - tau, with L = a t^2 / 2 and
// m = a tau (2t - tau) / 2, and with tau = tau0 (1 + u), tau0 = D0 / c the light time
// from its position at t, X = w1 - L, in units of D0:
//   f(u) = u (2 + u) - m (2 X + m) - K0h,  m = (a / 2c)(1 + u)(2t - tau),
// K0h = (perp^2 + X^2 - D0^2) / D0^2: a polynomial in u whose root is the retarded
// time's.  One step of order 5 in FP32 from u = 0, then in FP64 steps of order N = 4
// (mixed) or 5 (FULL) from where the last one led until that point has settled,
//   |f| < E f',  |f f''| / 2 <= H (f'^2 - f f'' / 2),
// as for the orbits (orbit_step): about a root of the physical sign only, of which the
// step leaves H^(N - 1), 2^-36 or 2^-44, of a distance below H.  (Behind a charge beyond
// 0.6 c f has inflections next to no root, where a step is small all the same.)  One
// such step on 99 % of the pairs of the grid workloads.  Returns false (the caller takes
// the safeguarded solver) when they do not settle.
template <typename F>
__device__ __forceinline__ void accel_taylor(F Xh, F K0h, F gh, F t, F tau0, F u, F f[5])
{
    const F tau = tau0 * u + tau0;
    const F gd = gh * (t - tau);
    // m and its derivatives in u
    const F m = (gh * ((F)1 + u)) * (t + (t - tau)), mp = gd + gd, mpp = (F)-2 * gh * tau0, xm = Xh + m;
    f[0] = u * ((F)2 + u) - (m * (Xh + xm) + K0h);
    f[1] = (F)-2 * mp * xm + ((F)2 + (F)2 * u);
    f[2] = (F)1 - (mpp * xm + mp * mp);
    f[3] = -mp * mpp;
    f[4] = (F)-0.25 * mpp * mpp;
}

template <bool FULL>
__device__ __forceinline__ bool solve_accel_poly(const SrcRec &S, const Geo &g, Kin &k)
{
    const double t = S.t, acc = S.accel, L = S.Lmax;
    const double W2 = fma(g.w1, g.w1, g.w2);
    const double ct = C_LIGHT * t;
    k.flags = 0u;
    k.cph = 1.0;
    k.sph = 0.0;
    double tp = 0.0;
    bool ok = true;
    int it = 0;
    if (t > 0.0 && W2 < ct * ct) {
        const double X = g.w1 - L;
        const double Dn2 = fma(X, X, g.w2);
        const double D0 = sqrt_rough(Dn2);
        const double iD0 = rcp_steer(D0), tau0 = D0 * INV_C;
        const double Xh = X * iD0, K0h = fma(-D0, D0, Dn2) * (iD0 * iD0), gh = acc * (0.5 * INV_C);
        float f32[5], n32, d32;
        accel_taylor<float>((float)Xh, (float)K0h, (float)gh, (float)t, (float)tau0, 0.f, f32);
        pade_step<5, float>(f32, n32, d32);
        double u = (double)(n32 * __builtin_amdgcn_rcpf(d32));
        ok = false;
        if (!(u > -0.999 && u < 100.0)) u = 0.0;
        do {
            ++it;
            double f[5], num, den;
            accel_taylor<double>(Xh, K0h, gh, t, tau0, u, f);
            pade_step<FULL ? 5 : 4, double>(f, num, den);
            u += num * rcp_steer(den);
            const double x2 = f[0] * f[2], d2 = f[1] * f[1] - x2;
            ok = fabs(f[0]) < 0x1p-11 * f[1] && fabs(x2) <= (FULL ? 0x1p-11 : 0x1p-12) * d2;
        } while (!ok && it < 8);
        const double tau = fma(tau0, u, tau0);
        tp = t - tau;
        // the polynomial's other roots are not retarded times
        ok = ok && u > -1.0 && tp >= -0x1p-40 * t;
        if (FULL) k.tp = tp;
        tp = fmax(tp, 0.0);
    } else {
        k.tp = FULL ? t - sqrt(W2) * INV_C : 0.0;
    }
    k.iters = 1 + max(it, 1);
    const double sd = 0.5 * acc * tp * tp;
    for (int i = 0; i < 3; ++i) k.R[i] = g.w[i] - sd * S.e1[i];
    if constexpr (FULL) {
        const double vel = acc * tp, ac = (tp > 0.0) ? acc : 0.0;
        for (int i = 0; i < 3; ++i) {
            k.v[i] = vel * S.e1[i];
            k.a[i] = ac * S.e1[i];
        }
    } else {
        const float bf = (float)(acc * tp * INV_C);
        for (int i = 0; i < 3; ++i) {
            k.bf[i] = bf * S.bw1[i];
            k.df[i] = (tp > 0.0) ? S.aw1[i] : 0.f;
        }
        k.omb = fmaf(-bf, bf, 1.f);
    }
    return ok;
}

// The rare fallback of the correction solves (a solve that did not settle): the
// safeguarded solver, for the orbits on a geometry built here with its bracket,
// so that the main path neither builds the bracket nor keeps the frame
// coordinates live across the times.
template <bool FULL, int KIND>
__device__ __forceinline__ void retarded_fallback(const SrcRec &S, const Geo &g, const double x[3], int max_iter,
                                                  double tol_rel, Kin &k)
{
    if constexpr (KIND == K_ACCEL) {
        solve_accel<FULL>(S, g, max_iter, tol_rel, k);
        if constexpr (!FULL) {
            float bb = 0.f;
            for (int i = 0; i < 3; ++i) {
                k.bf[i] = (float)(k.v[i] * INV_C);
                k.df[i] = (float)(k.a[i] * INV_C);
                bb = fmaf(k.bf[i], k.bf[i], bb);
            }
            k.omb = 1.f - bb;
        }
    } else {
        GeoSafe gf;
        geo_safe<KIND>(S, x, gf);
        if constexpr (KIND == K_CIRCULAR) solve_circular<FULL>(S, gf, max_iter, tol_rel, k);
        else solve_linear<FULL>(S, gf, max_iter, tol_rel, k);
    }
    if (!FULL) k.iters |= ITER_FALLBACK;
}

// Retarded kinematics of a source S of family KIND (its record for the
// observation time) seen from point x, with g = geo_prepare_k<KIND>(record of any
// time of this source, x).  FULL: to FP64 rounding; otherwise for FP32 fields
// (phases good to about 5e-12).  Only the fallback can fail to converge: its flags
// are added to `flags` there, off the usual path.
template <bool FULL, int KIND>
__device__ __forceinline__ void retarded_kind(const SrcRec &S, const Geo &g, const double x[3], int max_iter,
                                              double tol_rel, Kin &k, uint32_t &flags)
{
    if constexpr (KIND == K_CIRCULAR || KIND == K_LINEAR_OSC) {
        if (!solve_orbit<KIND, FULL>(S, g, k)) {
            retarded_fallback<FULL, KIND>(S, g, x, max_iter, tol_rel, k);
            flags |= k.flags;
        }
    } else if constexpr (KIND == K_ACCEL) {
        if (!solve_accel_poly<FULL>(S, g, k)) {
            retarded_fallback<FULL, KIND>(S, g, x, max_iter, tol_rel, k);
            flags |= k.flags;
        }
    } else if constexpr (KIND == K_UNIFORM_VELOCITY) {
        solve_uniform<FULL>(S, x, k);
        if (!FULL) {
            for (int i = 0; i < 3; ++i) {     // beta from the record
                k.bf[i] = S.bw1[i];
                k.df[i] = 0.f;
            }
            k.omb = S.omb;
        }
    } else {
        for (int i = 0; i < 3; ++i) { k.R[i] = g.w[i]; k.v[i] = 0.0; k.a[i] = 0.0; k.bf[i] = 0.f; k.df[i] = 0.f; }
        k.omb = 1.f;
        k.tp = S.t - sqrt(g.w[0] * g.w[0] + g.w[1] * g.w[1] + g.w[2] * g.w[2]) * INV_C;
        k.cph = 1.0;
        k.sph = 0.0;
        k.flags = 0u;
        k.iters = 0;
    }
}

template <typename F> __device__ __forceinline__ F recip(F x);
template <> __device__ __forceinline__ float recip<float>(float x) { return __builtin_amdgcn_rcpf(x); }
// FP64: v_rcp_f64 and two Newton-Raphson steps (within about one ulp)
template <> __device__ __forceinline__ double recip<double>(double x)
{
    double r = __builtin_amdgcn_rcp(x);
    r = fma(r, fma(-x, r, 1.0), r);
    return fma(r, fma(-x, r, 1.0), r);
}

// Lienard-Wiechert outputs of one charge from its retarded kinematics, in
// precision F: out = (Phi, A, E, B).  With u = n - beta and kappa = 1 - n.beta,
// the radiation term's double cross product expands (BAC-CAB, n.u = kappa) to
//   n x (u x beta_dot) = u (n . beta_dot) - kappa beta_dot,
// so E = kq / (kappa^3 R) [u ((1 - beta^2)/R + n.beta_dot / c) - kappa beta_dot / c]
// for the total field (Eq. (E)); the Coulomb and radiation parts keep their
// own terms.  B = n x E / c (Eq. (B)), Phi = kq / (kappa R) (Eq. (V)),
// A = Phi beta / c (Eq. (A) in SI form).
// |R| and 1/|R| in precision F: FP32 through v_rsq_f32; FP64 from the refined
// v_rsq_f64 with one more Newton-Raphson step on the reciprocal (both within
// about one ulp).  |R| = 0 gives NaN, which the caller masks.
__device__ __forceinline__ void dist_inv(float R0, float R1, float R2, float &D, float &iD)
{
    const float D2 = R0 * R0 + R1 * R1 + R2 * R2;
    iD = __builtin_amdgcn_rsqf(D2);
    D = D2 * iD;
}
__device__ __forceinline__ void dist_inv(double R0, double R1, double R2, double &D, double &iD)
{
    root_rsqrt<true>(R0 * R0 + R1 * R1 + R2 * R2, D, iD);
    iD = fma(iD, fma(-D, iD, 1.0), iD);
}

// Returns the retarded distance |R| in precision F (for masking).  IC = false
// leaves out the factor 1/c of A and B (out[1..3] = Phi beta, out[7..9] = n x E),
// for callers that sum over charges first and scale the sums once.
template <typename F, bool IC = true>
__device__ __forceinline__ F lw_terms(const Kin &k, F kq, int field_kind, F out[10])
{
    const F R0 = (F)k.R[0], R1 = (F)k.R[1], R2 = (F)k.R[2];
    F D, iD;
    dist_inv(R0, R1, R2, D, iD);
    const F n0 = R0 * iD, n1 = R1 * iD, n2 = R2 * iD;
    F b0, b1, b2, d0, d1, d2;
    if constexpr (sizeof(F) == 4) {
        b0 = k.bf[0]; b1 = k.bf[1]; b2 = k.bf[2];
        d0 = k.df[0]; d1 = k.df[1]; d2 = k.df[2];
    } else {
        b0 = k.v[0] * INV_C; b1 = k.v[1] * INV_C; b2 = k.v[2] * INV_C;
        d0 = k.a[0] * INV_C; d1 = k.a[1] * INV_C; d2 = k.a[2] * INV_C;
    }
    const F ic = (F)INV_C;
    const F nb = n0 * b0 + n1 * b1 + n2 * b2;
    const F kappa = (F)1 - nb;
    F omb;                                                  // 1 - beta^2
    if constexpr (sizeof(F) == 4) omb = k.omb;
    else omb = (F)1 - (b0 * b0 + b1 * b1 + b2 * b2);
    const F u0 = n0 - b0, u1 = n1 - b1, u2 = n2 - b2;
    const F nd = n0 * d0 + n1 * d1 + n2 * d2;
    const F ik = recip<F>(kappa);
    const F kqD = kq * iD;
    const F phi = kqD * ik;
    const F f = phi * ik * ik;                              // kq / (kappa^3 R)
    F cu, cd;                                               // E = f (u cu - beta_dot cd)
    if (field_kind == F_COULOMB) {
        cu = omb * iD;
        cd = (F)0;
    } else if (field_kind == F_RADIATION) {
        cu = nd * ic;
        cd = kappa * ic;
    } else {
        cu = omb * iD + nd * ic;
        cd = kappa * ic;
    }
    cu *= f;
    cd *= f;
    const F E0 = u0 * cu - d0 * cd;
    const F E1 = u1 * cu - d1 * cd;
    const F E2 = u2 * cu - d2 * cd;
    const F m0 = IC ? n0 * ic : n0, m1 = IC ? n1 * ic : n1, m2 = IC ? n2 * ic : n2;  // n / c
    const F pc = IC ? phi * ic : phi;
    out[0] = phi;
    out[1] = pc * b0;
    out[2] = pc * b1;
    out[3] = pc * b2;
    out[4] = E0;
    out[5] = E1;
    out[6] = E2;
    out[7] = m1 * E2 - m2 * E1;
    out[8] = m2 * E0 - m0 * E2;
    out[9] = m0 * E1 - m1 * E0;
    return D;
}

// Reverse of lw_terms<double>: given the cotangent ob of (Phi, A, E, B), the
// cotangents of R, v, a and of kq = q / (4 pi eps0).  EONLY: only E has a
// cotangent (ob[4..6]; the other entries are not read), as for objectives of
// |E|^2.  The reverses of Phi, A and B are then left out, which gives the
// values of the general form with zero cotangents there (it adds only zeros).
// FAST: 1/|R| and 1/kappa from the refined hardware reciprocal square root and
// reciprocal (within an ulp or two) instead of the correctly rounded square
// root and divisions, as the forward FP64 evaluator takes them.
template <bool EONLY = false, bool FAST = false>
__device__ __forceinline__ void lw_terms_vjp(const Kin &k, double kq, int field_kind, const double ob[10],
                                             double Rb[3], double vb[3], double ab[3], double &kqb, double n[3],
                                             double &kappa_out)
{
    const double ic = INV_C;
    double D, iD;
    if constexpr (FAST) {
        dist_inv(k.R[0], k.R[1], k.R[2], D, iD);
    } else {
        D = sqrt(k.R[0] * k.R[0] + k.R[1] * k.R[1] + k.R[2] * k.R[2]);
        iD = 1.0 / D;
    }
    double b[3], d[3], u[3];
    for (int i = 0; i < 3; ++i) {
        n[i] = k.R[i] * iD;
        b[i] = k.v[i] * ic;
        d[i] = k.a[i] * ic;
        u[i] = n[i] - b[i];
    }
    const double nb = n[0] * b[0] + n[1] * b[1] + n[2] * b[2];
    const double kappa = 1.0 - nb;
    const double bb = b[0] * b[0] + b[1] * b[1] + b[2] * b[2];
    const double nd = n[0] * d[0] + n[1] * d[1] + n[2] * d[2];
    const double ik = FAST ? recip<double>(kappa) : 1.0 / kappa;
    const double kqD = kq * iD;
    const double phi = kqD * ik;
    const double f = phi * ik * ik;
    const bool coul = field_kind != F_RADIATION, rad = field_kind != F_COULOMB;
    const double cu = (coul ? (1.0 - bb) * iD : 0.0) + (rad ? nd * ic : 0.0);
    const double cd = rad ? kappa * ic : 0.0;
    double W[3], E[3], m[3];
    for (int i = 0; i < 3; ++i) {
        W[i] = u[i] * cu - d[i] * cd;
        E[i] = f * W[i];
        m[i] = n[i] * ic;
    }
    const double pc = phi * ic;
    // ---- reverse ----
    const double Eb[3] = {ob[4], ob[5], ob[6]};
    double mb[3] = {0.0, 0.0, 0.0}, Et[3] = {Eb[0], Eb[1], Eb[2]};
    double Phib = 0.0, pcb = 0.0, bbar[3] = {0.0, 0.0, 0.0};
    if constexpr (!EONLY) {
        Phib = ob[0];
        const double Ab[3] = {ob[1], ob[2], ob[3]};
        const double Bb[3] = {ob[7], ob[8], ob[9]};
        // B = m x E
        mb[0] = E[1] * Bb[2] - E[2] * Bb[1];
        mb[1] = E[2] * Bb[0] - E[0] * Bb[2];
        mb[2] = E[0] * Bb[1] - E[1] * Bb[0];
        Et[0] = Eb[0] + (Bb[1] * m[2] - Bb[2] * m[1]);
        Et[1] = Eb[1] + (Bb[2] * m[0] - Bb[0] * m[2]);
        Et[2] = Eb[2] + (Bb[0] * m[1] - Bb[1] * m[0]);
        // A = pc b
        pcb = Ab[0] * b[0] + Ab[1] * b[1] + Ab[2] * b[2];
        for (int i = 0; i < 3; ++i) bbar[i] = pc * Ab[i];
    }
    // E = f W, W = u cu - d cd
    const double fb = Et[0] * W[0] + Et[1] * W[1] + Et[2] * W[2];
    double ub[3], dbar[3];
    double cub = 0.0, cdb = 0.0;
    for (int i = 0; i < 3; ++i) {
        const double Wb = f * Et[i];
        ub[i] = Wb * cu;
        cub += Wb * u[i];
        dbar[i] = -Wb * cd;
        cdb -= Wb * d[i];
    }
    // phi = kqD ik feeds Phi, pc and f
    const double phib = EONLY ? fb * ik * ik : Phib + pcb * ic + fb * ik * ik;
    const double ikb_f = fb * 2.0 * phi * ik;
    double ikb = ikb_f + phib * kqD;
    const double kqDb = phib * ik;
    // cu, cd
    const double bbb = coul ? -cub * iD : 0.0;
    double iDb = coul ? cub * (1.0 - bb) : 0.0;
    const double ndb = rad ? cub * ic : 0.0;
    double kappab = rad ? cdb * ic : 0.0;
    // m = n / c
    double nbar[3] = {0.0, 0.0, 0.0};
    if constexpr (!EONLY)
        for (int i = 0; i < 3; ++i) nbar[i] = mb[i] * ic;
    // kqD = kq iD
    iDb += kqDb * kq;
    kqb = kqDb * iD;
    // ik = 1 / kappa
    kappab -= ikb * ik * ik;
    // nd = n . d
    for (int i = 0; i < 3; ++i) {
        nbar[i] += ndb * d[i] + ub[i];
        dbar[i] += ndb * n[i];
        bbar[i] += -ub[i] + 2.0 * bbb * b[i];
    }
    // kappa = 1 - n . b
    const double nbb = -kappab;
    for (int i = 0; i < 3; ++i) {
        nbar[i] += nbb * b[i];
        bbar[i] += nbb * n[i];
        vb[i] = bbar[i] * ic;
        ab[i] = dbar[i] * ic;
    }
    // n = R iD with iD = 1/|R|
    iDb += nbar[0] * k.R[0] + nbar[1] * k.R[1] + nbar[2] * k.R[2];
    const double s = -iDb * iD * iD;
    for (int i = 0; i < 3; ++i) Rb[i] = nbar[i] * iD + s * n[i];
    kappa_out = kappa;
}

}  // namespace lw
