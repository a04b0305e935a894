// lw_dipole.hpp -- oscillator records and history access shared by the
// forward run (lw_dipole.hip) and its adjoint (lw_dipole_adjoint.hip).
#pragma once

#include <limits>

#include "lw_device.hpp"
#include "lw_internal.hpp"

namespace lw {

struct DipDev {
    double origin[3];
    double axis[3];
    double omega0;
    double q;
    double f;        // q^2 / m  (m = m1 m2 / (m1 + m2), Eq. (eff_mass))
    double gamma0;   // q^2 omega0^2 / (6 pi eps0 c^3 m)  (Sec. 2.3)
    double cfp;      // offset of the +q charge per unit moment: m2 / (m1 + m2) / q   (Eq. (r_1))
    double cfm;      // offset of the -q charge per unit moment: -m1 / (m1 + m2) / q  (Eq. (r_2))
    double vfac;     // charge speed per unit d_dot: max(m1, m2) / (m1 + m2) / q
    double d0;
    double mamp[3];  // origin motion: origin + mamp cos(mw t + mph) (Sec. 4.3); mw = 0 when fixed
    double mw, mph;
    double mspeed;   // largest origin speed, mw |mamp|
    double ehalf;    // 0.5 / f, the factor of the energy (run_energy)
    double rk[9];    // one RK4 step's increments of d and d_dot (rk4_step)
};

// Per-dipole constants of the instance, staged in LDS.
struct DipLds {
    double ox, oy, oz;
    double px, py, pz;
    double cfp, cfm;
    double d0;
    double mx, my, mz, mw, mph;   // origin motion (mw = 0: fixed origin)
};

// Structure-of-arrays copy of the source fields the pair loops read: field f of
// dipole j at soa[f * n + j] (n dipoles in the run), so that a wave's load of
// one field over consecutive sources is coalesced.  It follows the DipDev
// array in the same block (dip_soa).
enum { SF_OX, SF_OY, SF_OZ, SF_PX, SF_PY, SF_PZ, SF_CFP, SF_CFM, SF_D0, SF_Q, SF_MX, SF_MY, SF_MZ, SF_MW, SF_MPH,
       SF_COUNT };

__host__ __device__ inline size_t dip_dev_array_bytes(int n) { return (sizeof(DipDev) * (size_t)n + 255) & ~(size_t)255; }
__host__ __device__ inline double *dip_soa(DipDev *dev, int n) { return (double *)((char *)dev + dip_dev_array_bytes(n)); }

// Field f of dipole j (the 32-bit byte offset of j lets each load take the
// field's base as a scalar operand).
__device__ __forceinline__ double soa_get(const double *__restrict__ s, int64_t n, int f, uint32_t j)
{
    return *(const double *)((const char *)(s + f * n) + j * 8u);
}

__device__ __forceinline__ DipLds soa_lds(const double *__restrict__ s, int64_t n, uint32_t j)
{
    return DipLds{soa_get(s, n, SF_OX, j),  soa_get(s, n, SF_OY, j),  soa_get(s, n, SF_OZ, j),
                  soa_get(s, n, SF_PX, j),  soa_get(s, n, SF_PY, j),  soa_get(s, n, SF_PZ, j),
                  soa_get(s, n, SF_CFP, j), soa_get(s, n, SF_CFM, j), soa_get(s, n, SF_D0, j),
                  soa_get(s, n, SF_MX, j),  soa_get(s, n, SF_MY, j),  soa_get(s, n, SF_MZ, j),
                  soa_get(s, n, SF_MW, j),  soa_get(s, n, SF_MPH, j)};
}

// Origin of a dipole at time t (fixed, or moving as O + m cos(w t + phi); the
// phase stays far below the 2^30 limit of sincos_reduced over any run).
__device__ __forceinline__ void origin_at(const DipLds &S, double t, double R[3])
{
    R[0] = S.ox;
    R[1] = S.oy;
    R[2] = S.oz;
    if (S.mw != 0.0) {
        double sn, c;
        sincos_reduced(S.mw * t + S.mph, sn, c);
        R[0] += S.mx * c;
        R[1] += S.my * c;
        R[2] += S.mz * c;
    }
}

// Stored kinematics (d, d_dot, d_ddot) of source j at s steps after t = 0 (s
// real).  Static at d0 before t = 0 (Sec. 3.2); linear interpolation between
// stored steps (Sec. 3.1); beyond the newest step `nstep` a second-order
// Taylor step from it (reached only when c dt exceeds a separation).
struct Hist {
    const double *ring;   // [ring][n][3]
    int n;
    int mask;             // ring - 1
    double dt;
    double inv_dt;
};

__device__ __forceinline__ DipLds dip_lds(const DipDev &D)
{
    return DipLds{D.origin[0], D.origin[1], D.origin[2], D.axis[0], D.axis[1], D.axis[2], D.cfp, D.cfm, D.d0,
                  D.mamp[0], D.mamp[1], D.mamp[2], D.mw, D.mph};
}

enum { ERR_HISTORY = 1u, ERR_NOCONV = 2u, ERR_VELOCITY = 4u, ERR_NONFINITE = 8u, ERR_STATE = 16u };

// Instance of global dipole g (last instance whose first dipole is <= g).
__device__ __forceinline__ int instance_of(const int32_t *off, int n_inst, int g)
{
    int lo = 0, hi = n_inst;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (off[mid] <= g) lo = mid; else hi = mid;
    }
    return lo;
}


// Stored samples k and k + 1 of one source; k = -1 stands for the static
// pre-history (t' < 0), where the state is (d0, 0, 0).  Step indices are of
// type I: int64_t, or int in a kernel that has checked its run fits (32-bit
// integer arithmetic is single instructions; 64-bit is not).  Every floating
// value is the same for both.
template <typename I>
struct SegT {
    I k;
    double d0, v0, a0;    // sample k: d, d_dot, d_ddot
    double d1, v1, a1;    // sample k + 1
};
using Seg = SegT<int64_t>;

// Segment index meaning "none loaded".
template <typename I> __host__ __device__ constexpr I seg_none() { return std::numeric_limits<I>::min(); }

template <typename I>
__device__ __forceinline__ void seg_load(const Hist &H, int j, double d0, I nstep, I k, SegT<I> &g, uint32_t &err)
{
    // k = -1 reads ring slot `mask` (in bounds) and discards it
    const bool pre = k < 0;
    g.k = pre ? -1 : k;
    if (!pre && k + H.mask < nstep) err |= ERR_HISTORY;   // the slot was overwritten: history too short
    const double *p0 = H.ring + ((I)(g.k & H.mask) * H.n + j) * 3;
    const double *p1 = H.ring + ((I)((g.k + 1) & H.mask) * H.n + j) * 3;
    g.d0 = pre ? d0 : p0[0];
    g.v0 = pre ? 0.0 : p0[1];
    g.a0 = pre ? 0.0 : p0[2];
    g.d1 = pre ? d0 : p1[0];
    g.v1 = pre ? 0.0 : p1[1];
    g.a1 = pre ? 0.0 : p1[2];
}

// Retarded time of the charge at offset cf d(t') p_j of a fixed source j, in
// closed form on the interpolated history.  Within the segment [k, k + 1] of
// stored steps the moment is linear in tau (t' = t - tau), so the charge's
// offset is rho = a + b tau and c tau = |Delta - rho p_j| becomes
//   (c^2 - b^2) tau^2 + 2 b P tau - Q = 0,
// P = sD - a, Q = |Delta - a p_j|^2 = L2 - 2 a sD + a^2, whose positive root
// tau = Q / (b P + sqrt(b^2 P^2 + (c^2 - b^2) Q)) has no cancellation
// (|b| << c).  The root is unique (the charge is slower than light), so if it
// falls outside the loaded segment it lies in the segment its own s points to,
// which is loaded next.  Returns false when the root lies past the newest
// stored step (the caller then uses the Newton solve with the extrapolation)
// or the hops do not settle.  On success tau_out is the root, h the
// interpolated state there and g the segment it lies in.
template <typename I>
__device__ __forceinline__ bool retarded_seg(const Hist &H, int j, double d0, I nstep, double base, double L2,
                                             double sD, double cf, SegT<I> &g, double h[3], double &tau_out,
                                             uint32_t &err)
{
    constexpr double C2 = C_LIGHT * C_LIGHT;
    for (int hop = 0; hop < 4; ++hop) {
        double a = cf * d0, b = 0.0;
        if (g.k >= 0) {
            const double dd = g.d1 - g.d0;
            a = cf * fma(base - (double)g.k, dd, g.d0);
            b = -cf * dd * H.inv_dt;
        }
        const double P = sD - a;
        const double Q = fma(a, a - 2.0 * sD, L2);
        const double bP = b * P;
        double S, iS;
        root_rsqrt<true>(fma(bP, bP, (C2 - b * b) * Q), S, iS);
        const double tau = Q * recip<double>(bP + S);
        const double s = base - tau * H.inv_dt;
        // a root within rounding of a segment end belongs to either side
        const double eps = 1e-9;
        if (g.k < 0 ? s <= eps : (s >= (double)g.k - eps && s <= (double)g.k + 1.0 + eps)) {
            const double u = g.k < 0 ? 0.0 : s - (double)g.k;
            h[0] = fma(u, g.d1 - g.d0, g.d0);
            h[1] = fma(u, g.v1 - g.v0, g.v0);
            h[2] = fma(u, g.a1 - g.a0, g.a0);
            tau_out = tau;
            return true;
        }
        const I kn = s < 0.0 ? -1 : (I)floor(s);
        if (kn >= nstep) return false;
        seg_load(H, j, d0, nstep, kn, g, err);
    }
    return false;
}

// Larmor power per |d_ddot|^2 (Sec. 2.5): 1 / (6 pi eps0 c^3).
constexpr double K_LARMOR = 1.0 / (6.0 * PI * EPS0 * C_LIGHT * C_LIGHT * C_LIGHT);

// Energy of Eq. (dipoleE) from (d, d_dot): (omega0^2 d^2 + d_dot^2) / (2 f),
// f = q^2 / m, in one fixed order of operations wherever it is evaluated.
// ehalf = 0.5 / f is the dipole's constant (DipDev::ehalf), so that no
// division sits on a step's critical path.
__device__ __forceinline__ double run_energy(double w2, double ehalf, double d, double v)
{
    return fma(w2 * d, d, v * v) * ehalf;
}

// One classic RK4 step of Eq. (LO_equation), y' = (d_dot, f E_d(t) - gamma0 d_dot -
// omega0^2 d) with the drives Ec, Em, Ee at t, t + dt/2, t + dt, is linear in the state
// and the drives.  c holds the coefficients of its increments, of d (on d, d_dot,
// Ec, Em) and of d_dot (on d, d_dot, Ec, Em, Ee).  Increments, not the propagator: the
// leading 1 of the propagator would round away the low bits of the rest the same
// way at every step.  Everything but the terms of Em and Ee is known before the
// drives are, so two dependent operations follow the drives here, against about 20
// through the stages.
__device__ __forceinline__ void rk4_stages(double w2, double g, double f, double dt, double y0, double y1, double Ec,
                                           double Em, double Ee, double &dd, double &dv)
{
    const double k1d = y1, k1v = f * Ec - g * y1 - w2 * y0;
    const double y0b = y0 + 0.5 * dt * k1d, y1b = y1 + 0.5 * dt * k1v;
    const double k2d = y1b, k2v = f * Em - g * y1b - w2 * y0b;
    const double y0c = y0 + 0.5 * dt * k2d, y1c = y1 + 0.5 * dt * k2v;
    const double k3d = y1c, k3v = f * Em - g * y1c - w2 * y0c;
    const double y0d = y0 + dt * k3d, y1d = y1 + dt * k3v;
    const double k4d = y1d, k4v = f * Ee - g * y1d - w2 * y0d;
    dd = dt / 6.0 * (k1d + 2.0 * k2d + 2.0 * k3d + k4d);
    dv = dt / 6.0 * (k1v + 2.0 * k2v + 2.0 * k3v + k4v);
}

// The two leading coefficients, dt (1 + e) of d_dot in d and -omega^2 dt (1 + e) of d in
// d_dot, rounded once: through the stages they carry three or four roundings, and an
// error of theirs is a phase error that grows with every step.
__device__ __forceinline__ void rk4_coefs(double om, double g, double f, double dt, double c[9])
{
    double skip;
    const double w2 = om * om;
    rk4_stages(w2, g, f, dt, 1.0, 0.0, 0.0, 0.0, 0.0, c[0], c[4]);
    rk4_stages(w2, g, f, dt, 0.0, 1.0, 0.0, 0.0, 0.0, c[1], c[5]);
    rk4_stages(w2, g, f, dt, 0.0, 0.0, 1.0, 0.0, 0.0, c[2], c[6]);
    rk4_stages(w2, g, f, dt, 0.0, 0.0, 0.0, 1.0, 0.0, c[3], c[7]);
    rk4_stages(w2, g, f, dt, 0.0, 0.0, 0.0, 0.0, 1.0, skip, c[8]);
    const double e = dt * (-0.5 * g + dt * ((g * g - w2) / 6.0 + dt * (2.0 * g * w2 - g * g * g) / 24.0));
    const double p = w2 * dt, p_lo = fma(w2, dt, -p) + fma(om, om, -w2) * dt;
    c[1] = fma(dt, e, dt);
    c[4] = -(p + fma(p, e, p_lo));
}

__device__ __forceinline__ void rk4_step(const double c[9], double y0, double y1, double Ec, double Em, double Ee,
                                         double &dn, double &vn)
{
    const double pd = fma(c[2], Ec, fma(c[1], y1, c[0] * y0));
    const double pv = fma(c[6], Ec, fma(c[5], y1, c[4] * y0));
    dn = y0 + fma(c[3], Em, pd);
    vn = y1 + fma(c[8], Ee, fma(c[7], Em, pv));
}

// Charges close to their dipole's origin.  With lengths in units of the separation
// L of the target from the source's origin and mu = cos of the angle between them and
// the source's axis, a charge at offset x has the distance D = sqrt(1 + y), y = x (x -
// 2 mu), and the offset is a known function of the retarded step, x(u) = X0 + u (X1 + u
// X2): linear within a history segment (X2 = 0), quadratic past the newest sample.
// The retarded condition D = 1 + q, u = u0 - w q (w = L / (c dt); u0: the step at q = 0)
// is solved by expanding about q = 0, where everything but x is a constant of the
// pair: q0 = sqrt(1 + y) - 1 and 1 / D by their series in y (through y^5: below 2e-17
// at |y| <= 2^-9), the slope zeta = dq/dq = -w x' (x - mu) / D by its geometric series, and
// for a quadratic x (quad = 1; 0 gives a linear one the bits of QUAD = false) the
// second-order term p q0^2.
// So the root takes no square root and no division: 35 instructions, against 70
// with two refined v_rsq_f64 and a reciprocal for the closed form on a segment and
// the distance from it.  The range is |x| 2^10 + |zeta| 2^13 + |q - q0| 2^27 + |p q0^2|
// 2^40 <= 1, within which the terms left out stay below 2^-53 (an offset of 1e-12 m
// is inside from about 1 nm, a speed of 2e-6 c always); beyond it (r.out > 1, or not a
// number) the caller takes the general solvers.
struct SmallRoot {
    double u, x, q, iD;    // step, offset, distance 1 + q (units of L) and its reciprocal at the root
    double out;            // above 1: outside the range
};

// The series' coefficients, held in registers over the caller's loop (opaque to the
// compiler, which would rebuild each 64-bit constant by two scalar moves next to its
// use): VGPRs for a kernel of one wave per SIMD, where each scalar move is an issue
// slot of the wave's chain, scalar registers otherwise.
struct SmallK {
    double q1, q2, q3, q4;        // sqrt(1 + y) - 1 = y (1/2 + q1 y + ...)
    double i1, i2, i3, i4;        // 1 / sqrt(1 + y) - 1 = y (-1/2 + i1 y + ...)
    double lx, lz, ld, lp;        // reciprocal limits of |x|, |zeta| and |b|, |q - q0|, |p q0^2|
    double k0, k1, k2, k3;        // 1 / kappa^3 - 1 = z (k0 + k1 z + ...)
};
template <bool VGPR> __device__ __forceinline__ void hold(double &k)
{
    if constexpr (VGPR) asm volatile("" : "+v"(k));
    else asm volatile("" : "+s"(k));
}
template <bool VGPR> __device__ __forceinline__ SmallK small_k()
{
    SmallK c{-1.0 / 8.0, 1.0 / 16.0, -5.0 / 128.0, 7.0 / 256.0, 3.0 / 8.0, -5.0 / 16.0, 35.0 / 128.0, -63.0 / 256.0,
             0x1p10, 0x1p13, 0x1p27, 0x1p40, 3.0, 6.0, 10.0, 15.0};
    hold<VGPR>(c.q1); hold<VGPR>(c.q2); hold<VGPR>(c.q3); hold<VGPR>(c.q4);
    hold<VGPR>(c.i1); hold<VGPR>(c.i2); hold<VGPR>(c.i3); hold<VGPR>(c.i4);
    hold<VGPR>(c.lx); hold<VGPR>(c.lz); hold<VGPR>(c.ld); hold<VGPR>(c.lp);
    hold<VGPR>(c.k0); hold<VGPR>(c.k1); hold<VGPR>(c.k2); hold<VGPR>(c.k3);
    return c;
}

template <bool QUAD>
__device__ __forceinline__ void small_root(const SmallK &c, double mu, double w, double u0, double X0, double X1,
                                           double X2, double quad, SmallRoot &r)
{
    double x, xs;
    if constexpr (QUAD) {
        x = fma(u0, fma(u0, X2, X1), X0);
        xs = fma(u0 + u0, X2, X1);
    } else {
        x = fma(u0, X1, X0);
        xs = X1;
    }
    const double y = x * fma(-2.0, mu, x), y2 = y * y;
    const double q0 = y * fma(y2, fma(y2, c.q4, fma(y, c.q3, c.q2)), fma(y, c.q1, 0.5));
    const double i0 = fma(y, fma(y2, fma(y2, c.i4, fma(y, c.i3, c.i2)), fma(y, c.i1, -0.5)), 1.0);
    const double t = (x - mu) * i0;
    const double wx = -w * xs;
    const double zeta = wx * t;
    double dq = q0 * fma(zeta, fma(zeta, zeta, zeta), zeta);
    r.out = fma(fabs(x), c.lx, fabs(zeta) * c.lz);
    if constexpr (QUAD) {
        const double p2 = quad * fma(w * w * X2, t, 0.5 * (wx * wx) * fma(-t, t, 1.0)) * (q0 * q0);
        r.out = fma(fabs(p2), c.lp, r.out);
        dq = fma(p2, 1.0 + zeta, dq);
    }
    r.out = fma(fabs(dq), c.ld, r.out);
    const double q = q0 + dq;
    r.u = fma(-w, q, u0);
    r.x = QUAD ? fma(r.u, fma(r.u, X2, X1), X0) : fma(r.u, X1, X0);
    r.q = q;
    r.iD = fma(i0, fma(-(1.0 + q), i0, 1.0), i0);
}

// p_i . E of a charge at the root of small_root, per kq / L^2 (Eq. (E) on the source's
// axis, as drive_scalar): muI = p_i . Delta / L, b = v / c and e = a L / c^2 along the
// axis, |b| <= 2^-13 (1 / kappa^3 by its series through b^4).  Every term is formed as
// its difference from the field muI of the charge at rest at the origin, so only
// the last sum rounds relative to one charge's field.  DIFF leaves that sum out: muI
// cancels exactly between a dipole's two charges, and what is left rounds
// relative to the dipole's field, 1e3 to 1e6 times smaller (the mixed form).
template <bool DIFF>
__device__ __forceinline__ double small_field(const SmallK &c, double mu, double muI, double pij, const SmallRoot &r,
                                              double b, double e)
{
    const double j = -r.q * r.iD;                       // 1 / D - 1
    const double wn = (mu - r.x) * r.iD;                // n . p_j
    const double dp = fma(j, muI, -(r.x * pij) * r.iD); // p_i . n - muI
    const double pin = muI + dp;
    const double jj = fma(j, j, j + j);                 // 1 / D^2 - 1
    const double z = b * wn;
    const double k = z * fma(z, fma(z, fma(z, c.k3, c.k2), c.k1), c.k0);      // 1 / kappa^3 - 1
    const double q = fma(-pin, wn, pij);
    double B = fma(pin, jj, dp);
    B = fma(-b * (1.0 + jj), fma(b, fma(-b, pij, pin), pij), B);
    B = fma(-e * q, r.iD, B);
    B = fma(k, muI + B, B);
    return DIFF ? B : muI + B;
}

// Output row of the state after `rel` steps of the call, or -1 when the
// stride skips it (stride 1, the usual case, needs no 64-bit division, which
// has no hardware instruction and would sit on each step's critical path).
__device__ __forceinline__ int64_t out_row(int64_t rel, int64_t stride)
{
    if (stride == 1) return rel;
    return rel % stride == 0 ? rel / stride : -1;
}

// Writes row `row` of the outputs for dipole gi.
__device__ __forceinline__ void put_row(const RunOut &o, int64_t row, int gi, double d, double v, double E, double Ed,
                                        double wa, double wr)
{
    const int64_t k = row * o.n_dip + gi;
    o.d[k] = d;
    if (o.v) o.v[k] = v;
    if (o.E) o.E[k] = E;
    if (o.Ed) o.Ed[k] = Ed;
    if (o.wabs) o.wabs[k] = wa;
    if (o.wrad) o.wrad[k] = wr;
}

}  // namespace lw
