// lw_dipole.hip -- self-consistent Lorentz-oscillator runs on gfx950.
//
// Algorithm 1 of the paper.  Small instances run persistently over all time
// steps in one workgroup each (lo_instances_kernel); large ones take one
// launch per step with one workgroup per target dipole (lo_step_kernel).
// Each step:
//   1. every (target i, stage time, source dipole j != i, charge +/-) pair
//      solves its retarded time against j's stored history (in closed form on
//      the linear interpolation segment, Newton past the newest stored step or
//      for a moving source) and evaluates the Lienard-Wiechert field of Eq. (E)
//      at R_i projected on p_i: per charge in FP64, or in the mixed form per
//      source dipole (FP64 static monopole difference, FP32 remainder);
//   2. the pairs of one (target, stage) are summed in a fixed order by a lane
//      group and a shuffle tree (bitwise reproducible);
//   3. one lane per dipole takes the RK4 step of Eq. (LO_equation), writes
//      (d, d_dot, d_ddot) at t_{n+1} into the history ring and the outputs.
// The history ring holds the last `ring` steps of every dipole of the
// instance (in LDS when it fits); its depth covers the longest light travel
// time inside the instance, so step n+1 overwrites a slot no retarded time can
// reach any more.
#include <math.h>
#include <algorithm>
#include <cmath>

#include "lw_device.hpp"
#include "lw_dipole.hpp"
#include "lw_internal.hpp"

#include <type_traits>

namespace lw {

size_t dip_dev_bytes(int n) { return dip_dev_array_bytes(n) + sizeof(double) * SF_COUNT * (size_t)n; }

__global__ void dipole_prep_kernel(const lw_dipole *__restrict__ in, int n, double dt, DipDev *__restrict__ dev,
                                   double *__restrict__ soa)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const lw_dipole &D = in[i];
    DipDev o;
    for (int k = 0; k < 3; ++k) {
        o.origin[k] = D.origin[k];
        o.axis[k] = D.axis[k];
    }
    const double M = D.m1 + D.m2;
    const double m = D.m1 * D.m2 / M;
    o.omega0 = D.omega0;
    o.q = D.q;
    o.f = D.q * D.q / m;
    o.gamma0 = D.q * D.q * D.omega0 * D.omega0 / (6.0 * PI * EPS0 * C_LIGHT * C_LIGHT * C_LIGHT * m);
    o.cfp = D.m2 / M / D.q;
    o.cfm = -D.m1 / M / D.q;
    o.vfac = fmax(D.m1, D.m2) / M / D.q;
    o.d0 = D.d0;
    const double am = sqrt(D.motion_amp[0] * D.motion_amp[0] + D.motion_amp[1] * D.motion_amp[1] +
                           D.motion_amp[2] * D.motion_amp[2]);
    const bool moves = am > 0.0;                  // the host requires motion_omega != 0 then
    for (int k = 0; k < 3; ++k) o.mamp[k] = moves ? D.motion_amp[k] : 0.0;
    o.mw = moves ? D.motion_omega : 0.0;
    o.mph = moves ? D.motion_phase : 0.0;
    o.mspeed = moves ? fabs(D.motion_omega) * am : 0.0;
    o.ehalf = 0.5 / o.f;
    rk4_coefs(o.omega0, o.gamma0, o.f, dt, o.rk);
    dev[i] = o;
    const double f[SF_COUNT] = {o.origin[0], o.origin[1], o.origin[2], o.axis[0], o.axis[1], o.axis[2], o.cfp,
                                o.cfm,       o.d0,        o.q,         o.mamp[0], o.mamp[1], o.mamp[2], o.mw, o.mph};
    for (int k = 0; k < SF_COUNT; ++k) soa[(int64_t)k * n + i] = f[k];
}

hipError_t launch_dipole_prep(const lw_dipole *d_in, int n, double dt, DipDev *d_dev, hipStream_t s)
{
    hipLaunchKernelGGL(dipole_prep_kernel, dim3((n + 255) / 256), dim3(256), 0, s, d_in, n, dt, d_dev,
                       dip_soa(d_dev, n));
    return hipGetLastError();
}

// region: 0 before t = 0, 1 between stored samples, 2 past the newest sample.
template <typename I>
__device__ __forceinline__ void hist_at(const Hist &H, int j, double d0, I nstep, double s, double out[3],
                                        double &slope, int &region, uint32_t &err)
{
    if (s < 0.0) {
        out[0] = d0;
        out[1] = 0.0;
        out[2] = 0.0;
        slope = 0.0;
        region = 0;
        return;
    }
    const double fk = floor(s);
    const I k = (I)fk;
    if (k >= nstep) {
        const double *h = H.ring + ((I)(nstep & H.mask) * H.n + j) * 3;
        const double tt = (s - (double)nstep) * H.dt;
        out[0] = h[0] + h[1] * tt + 0.5 * h[2] * tt * tt;
        out[1] = h[1] + h[2] * tt;
        out[2] = h[2];
        slope = out[1];
        region = 2;
        return;
    }
    if (k + H.mask < nstep) err |= 1u;          // the slot was overwritten: history too short
    const double u = s - fk;
    const double *h0 = H.ring + ((I)(k & H.mask) * H.n + j) * 3;
    const double *h1 = H.ring + ((I)((k + 1) & H.mask) * H.n + j) * 3;
    out[0] = (1.0 - u) * h0[0] + u * h1[0];
    out[1] = (1.0 - u) * h0[1] + u * h1[1];
    out[2] = (1.0 - u) * h0[2] + u * h1[2];
    slope = (h1[0] - h0[0]) * H.inv_dt;           // d/dt' of the interpolated moment
    region = 1;
}

// Retarded time of the charge at offset cf d(t') p_j of source j, seen from a
// point at separation Delta (|Delta|^2 = L2, Delta . p_j = sD) from the
// source's origin at time base * dt, by Newton (where the closed form of
// retarded_seg does not apply: past the newest stored step): the root of
// c tau = |Delta - cf d(t - tau) p_j| in [0, tau_hi], from tau.  Newton uses the exact slope of the
// interpolated moment.  Within one interpolation segment (or one side of the
// history's ends) g is smooth with |g''| <= rho'^2 / D + |rho''| (rho = cf d),
// so once Newton's error bound from the current iterate is below tol/4 the new
// iterate is accepted and the history evaluated there once more.  h holds the
// stored (d, d_dot, d_ddot) at the returned root.
template <typename I>
__device__ __forceinline__ double retarded_hist(const Hist &H, int j, double d0, I nstep, double base, double L2,
                                                double sD, double cf, double tau, double tau_hi, int max_iter,
                                                double h[3], uint32_t &err)
{
    const double tol = 4.0 * 2.220446049250313e-16;
    Bracket b(0.0, tau_hi);
    bool ok = false;
    for (int it = 0; it < max_iter; ++it) {
        const double s = base - tau * H.inv_dt;
        double slope;
        int region;
        hist_at(H, j, d0, nstep, s, h, slope, region, err);
        const double rho = cf * h[0];                            // charge offset along p_j
        double D, iD;
        root_rsqrt<true>(fmax(L2 - 2.0 * rho * sD + rho * rho, 1e-300), D, iD);
        const double r1 = cf * slope;
        const double dD = r1 * (sD - rho) * iD;
        bool free_step;
        const double tn = halley_step(tau, D, dD, 0.0, b, free_step);
        ok = converged(tn, tau, tol, b);
        if (ok) break;                                           // keep h at the last evaluated tau
        const double st = tn - tau;
        const double r2 = (region == 2) ? cf * h[2] : 0.0;
        const double sn = base - tn * H.inv_dt;
        const bool same_seg = (region == 1) ? (floor(sn) == floor(s) && sn < (double)nstep)
                                            : (region == 2 ? sn >= (double)nstep : sn < 0.0);
        tau = tn;
        if (free_step && same_seg && (r1 * r1 + fabs(r2) * D) * (st * st) <= 0.5 * tol * tn * D * (C_LIGHT - fabs(r1))) {
            double sl;
            int rg;
            hist_at(H, j, d0, nstep, sn, h, sl, rg, err);
            ok = true;
            break;
        }
    }
    if (!ok) err |= 2u;
    return tau;
}

// Retarded time past the newest stored step (the Taylor extrapolation of the
// history from sample nstep, Sec. 2.3 with the dt reading of the extrapolating
// policy): there the charge's offset is quadratic in tau,
//   rho(tau) = cf (d + v u + a u^2 / 2),  u = (base - nstep) dt - tau,
// and c tau = |Delta - rho p_j| is solved by the closed form of retarded_seg
// on the tangent line of rho, taken twice (at tau = L/c, then at the first
// root).  The linearisation error is rho'' (tau1 - tau0)^2 / 2, with
// |tau1 - tau0| ~ |rho| / c.  The result is accepted under retarded_hist's
// a-posteriori bound on the last step; returns false (the caller then uses
// Newton) when the root lies inside the stored history or the bound fails.
template <typename I>
__device__ __forceinline__ bool retarded_ext(const Hist &H, int j, I nstep, double base, double L2, double L,
                                             double sD, double cf, double h[3], double &tau_out)
{
    constexpr double C2 = C_LIGHT * C_LIGHT;
    const double *hn = H.ring + ((I)(nstep & H.mask) * H.n + j) * 3;
    const double U = (base - (double)nstep) * H.dt;
    const double al = cf * hn[0], be = cf * hn[1], ga = 0.5 * cf * hn[2];
    double tau = L * INV_C, step = 0.0, r1 = 0.0;
    for (int pass = 0; pass < 2; ++pass) {
        const double u = U - tau;
        const double rho = al + u * (be + u * ga);
        r1 = -(be + 2.0 * ga * u);                      // d rho / d tau
        const double a = rho - r1 * tau;                // tangent line a + r1 tau
        const double P = sD - a;
        const double Q = fma(a, a - 2.0 * sD, L2);
        const double bP = r1 * P;
        double S, iS;
        root_rsqrt<true>(fma(bP, bP, (C2 - r1 * r1) * Q), S, iS);
        const double tn = Q * recip<double>(bP + S);
        step = tn - tau;
        tau = tn;
    }
    const double u = U - tau;
    if (!(u >= 0.0)) return false;                      // inside the stored history
    const double D = C_LIGHT * tau, r2 = 2.0 * ga;
    const double tol = 4.0 * 2.220446049250313e-16;
    if (!((r1 * r1 + fabs(r2) * D) * (step * step) <= 0.5 * tol * tau * D * (C_LIGHT - fabs(r1)))) return false;
    h[0] = hn[0] + hn[1] * u + 0.5 * hn[2] * u * u;
    h[1] = hn[1] + hn[2] * u;
    h[2] = hn[2];
    tau_out = tau;
    return true;
}

// Retarded time of the charge at offset cf d(t') p_j of a moving source j seen
// from X at time base * dt: the root of c tau = |X - R_j(t') - cf d(t') p_j|,
// t' = t - tau, with R_j(t') = O_j + m_j cos(w t' + phi).  The same iteration
// and stopping rule as retarded_hist, with the origin's velocity and
// acceleration in the slope and the bound on g''.  Returns tau; h holds the
// stored state at the root and Ro, Vo, Ao the origin's position, velocity and
// acceleration there.
__device__ double retarded_hist_moving(const Hist &H, int j, const DipLds &Sj, const double X[3], double cf,
                                       int64_t nstep, double base, double tau, double tau_hi, int max_iter,
                                       double h[3], double Ro[3], double Vo[3], double Ao[3], uint32_t &err)
{
    const double tol = 4.0 * 2.220446049250313e-16;
    const double O[3] = {Sj.ox, Sj.oy, Sj.oz};
    const double m[3] = {Sj.mx, Sj.my, Sj.mz};
    const double p[3] = {Sj.px, Sj.py, Sj.pz};
    const double am = sqrt(m[0] * m[0] + m[1] * m[1] + m[2] * m[2]);
    Bracket b(0.0, tau_hi);
    bool ok = false;
    auto origin = [&](double s) {
        double sn, c;
        sincos_reduced(Sj.mw * (s * H.dt) + Sj.mph, sn, c);
        for (int k = 0; k < 3; ++k) {
            Ro[k] = O[k] + m[k] * c;
            Vo[k] = -Sj.mw * m[k] * sn;
            Ao[k] = -Sj.mw * Sj.mw * m[k] * c;
        }
    };
    for (int it = 0; it < max_iter; ++it) {
        const double s = base - tau * H.inv_dt;
        double slope;
        int region;
        hist_at(H, j, Sj.d0, nstep, s, h, slope, region, err);
        origin(s);
        const double rho = cf * h[0];
        double Rv[3], vel[3];
        for (int k = 0; k < 3; ++k) {
            Rv[k] = X[k] - Ro[k] - rho * p[k];
            vel[k] = Vo[k] + cf * slope * p[k];                 // d/dt' of the charge position
        }
        double D, iD;
        root_rsqrt<true>(fmax(Rv[0] * Rv[0] + Rv[1] * Rv[1] + Rv[2] * Rv[2], 1e-300), D, iD);
        const double dD = (Rv[0] * vel[0] + Rv[1] * vel[1] + Rv[2] * vel[2]) * iD;
        bool free_step;
        const double tn = halley_step(tau, D, dD, 0.0, b, free_step);
        ok = converged(tn, tau, tol, b);
        if (ok) break;
        const double st = tn - tau;
        const double sn = base - tn * H.inv_dt;
        const bool same_seg = (region == 1) ? (floor(sn) == floor(s) && sn < (double)nstep)
                                            : (region == 2 ? sn >= (double)nstep : sn < 0.0);
        const double v2 = vel[0] * vel[0] + vel[1] * vel[1] + vel[2] * vel[2];
        const double acc = Sj.mw * Sj.mw * am + ((region == 2) ? fabs(cf * h[2]) : 0.0);
        tau = tn;
        if (free_step && same_seg && (v2 + acc * D) * (st * st) <= 0.5 * tol * tn * D * (C_LIGHT - sqrt(v2))) {
            double sl;
            int rg;
            hist_at(H, j, Sj.d0, nstep, sn, h, sl, rg, err);
            origin(sn);
            ok = true;
            break;
        }
    }
    if (!ok) err |= 2u;
    return tau;
}

// Interpolated state h at the retarded time of the charge (cf) of fixed source
// j seen at separation Delta (|Delta|^2 = L2, |Delta| = L, Delta . p_j = sD):
// the closed form on the segment cached in g; past the newest stored step the
// closed form on the extrapolation; else Newton.  g.k = seg_none<I>() marks an
// empty cache.
template <typename I>
__device__ __forceinline__ void charge_fixed(const Hist &H, int j, double d0, I nstep, double base, double L2,
                                             double L, double sD, double cf, int max_iter, SegT<I> &g, double h[3],
                                             uint32_t &err)
{
    if (g.k == seg_none<I>()) {
        const double s0 = base - L * INV_C * H.inv_dt;
        const I k0 = s0 < 0.0 ? -1 : (I)floor(s0);
        if (k0 < nstep) seg_load(H, j, d0, nstep, k0, g, err);
    }
    double tau;
    if (g.k != seg_none<I>() && retarded_seg(H, j, d0, nstep, base, L2, sD, cf, g, h, tau, err)) return;
    if (retarded_ext(H, j, nstep, base, L2, L, sD, cf, h, tau)) return;
    retarded_hist(H, j, d0, nstep, base, L2, sD, cf, L * INV_C, 2.0 * L * INV_C, max_iter, h, err);
}

// Retarded separation R = X - r(t'), velocity and acceleration of the charge
// (cf) of a moving source j seen from X at time base * dt (Sec. 4.3: the
// charges ride on the source's origin at the retarded time).
__device__ __forceinline__ void charge_moving(const Hist &H, const DipLds &Sj, int j, double cf, int64_t nstep,
                                              double base, const double X[3], int max_iter, double R[3],
                                              double v[3], double a[3], uint32_t &err)
{
    // start from the present separation of the origins; the bracket's upper
    // end covers the origin's whole swing
    const double dx = X[0] - Sj.ox, dy = X[1] - Sj.oy, dz = X[2] - Sj.oz;
    const double reach = sqrt(dx * dx + dy * dy + dz * dz) + sqrt(Sj.mx * Sj.mx + Sj.my * Sj.my + Sj.mz * Sj.mz);
    double h[3], Ro[3], Vo[3], Ao[3];
    retarded_hist_moving(H, j, Sj, X, cf, nstep, base, reach * INV_C, 2.0 * reach * INV_C, max_iter, h, Ro, Vo, Ao,
                         err);
    const double rho = cf * h[0];
    const double p[3] = {Sj.px, Sj.py, Sj.pz};
    for (int c = 0; c < 3; ++c) {
        R[c] = X[c] - Ro[c] - rho * p[c];
        v[c] = Vo[c] + cf * h[1] * p[c];
        a[c] = Ao[c] + cf * h[2] * p[c];
    }
}

// p_i . E of one charge from its retarded separation, velocity and
// acceleration (FP64 field, Eq. (E)).
__device__ __forceinline__ double charge_field(const DipLds &Si, const double R[3], const double v[3],
                                               const double a[3], double kq)
{
    Kin k;
    for (int c = 0; c < 3; ++c) {
        k.R[c] = R[c];
        k.v[c] = v[c];
        k.a[c] = a[c];
    }
    k.tp = 0.0;
    k.cph = 1.0;
    k.sph = 0.0;
    k.flags = 0u;
    double o[10];
    lw_terms<double>(k, kq, F_TOTAL, o);
    return o[4] * Si.px + o[5] * Si.py + o[6] * Si.pz;
}

// p_i . E at the origin of target i of the charge (cf, kq) of source j, at
// time (nstep + theta) dt, all in FP64.  Moving origins (Sec. 4.3): the field is
// taken at the target's origin at that time.  MOVING: origins may move; without
// it every origin is taken as fixed (the kernels for fixed origins carry none
// of the moving-origin code).
// Separation of a target at X from a fixed source j: |Delta|^2, |Delta| and its
// reciprocal, and the projections Delta . p_j, Delta . p_i and p_i . p_j that the
// scalar drive needs (constant over a run when both origins are fixed).
struct PairGeo {
    double L2, L, iL, sD, sI, pij;
};

__device__ __forceinline__ PairGeo pair_geo(const double X[3], const DipLds &Si, const DipLds &Sj)
{
    PairGeo P;
    const double dx = X[0] - Sj.ox, dy = X[1] - Sj.oy, dz = X[2] - Sj.oz;
    P.L2 = dx * dx + dy * dy + dz * dz;
    root_rsqrt<true>(P.L2, P.L, P.iL);
    P.iL = fma(P.iL, fma(-P.L, P.iL, 1.0), P.iL);
    P.sD = dx * Sj.px + dy * Sj.py + dz * Sj.pz;     // Delta . p_j
    P.sI = dx * Si.px + dy * Si.py + dz * Si.pz;     // Delta . p_i
    P.pij = Si.px * Sj.px + Si.py * Sj.py + Si.pz * Sj.pz;
    return P;
}

// p_i . E (Eq. (E), total field, FP64) at the origin of target i of the charge
// (cf, kq) of a fixed source j, from its stored state h at the retarded time.  Every
// term is formed as its difference from p_i . Delta / L^3, the field of the charge at
// rest at the source's origin, which is added last (as small_field).
// The charge moves along p_j, so beta and beta_dot are multiples of p_j and
// every vector product of Eq. (E) reduces to the scalars
//   w = R . p_j = sD - rho,  p_i . R = sI - rho pij,  pij = p_i . p_j,
// with R = Delta - rho p_j, rho = cf d:
//   p_i . E = f [(p_i . n - b pij) (1 - b^2) / |R| - e q / c],  n = R / |R|,
//   b = cf d_dot / c, e = cf d_ddot / c, kappa = 1 - b (n . p_j),
//   f = kq / (kappa^3 |R|), q = pij - (p_i . n)(n . p_j),
// where the radiation term's beta parts cancel exactly (q is p_i . the part
// of p_j across n).
__device__ __forceinline__ double drive_scalar(const PairGeo &P, double cf, double kq, const double h[3])
{
    const double x = cf * h[0] * P.iL, mu = P.sD * P.iL, muI = P.sI * P.iL;
    const double y = x * fma(-2.0, mu, x);
    double D, iD;
    root_rsqrt<true>(1.0 + y, D, iD);
    iD = fma(iD, fma(-D, iD, 1.0), iD);
    const double b = cf * h[1] * INV_C, e = cf * h[2] * (INV_C * INV_C) * P.L;
    const double j = -y * recip<double>(1.0 + D) * iD;   // 1 / D - 1
    const double wn = (mu - x) * iD;                     // n . p_j
    const double dp = fma(j, muI, -(x * P.pij) * iD);    // p_i . n - muI
    const double pin = muI + dp;
    const double jj = fma(j, j, j + j);
    const double z = b * wn, kappa = 1.0 - z, ik = recip<double>(kappa);
    const double k = z * fma(kappa, kappa, 1.0 + kappa) * (ik * ik * ik);   // 1 / kappa^3 - 1
    const double q = fma(-pin, wn, P.pij);
    double B = fma(pin, jj, dp);
    B = fma(-b * (1.0 + jj), fma(b, fma(-b, P.pij, pin), P.pij), B);
    B = fma(-e * q, iD, B);
    B = fma(k, muI + B, B);
    return kq * (P.iL * P.iL) * (muI + B);
}

// p_i . E of the charge (cf, kq) of the fixed source j at separation P, at
// time base * dt, from the stored history.
template <typename I>
__device__ __forceinline__ double fixed_drive(const Hist &H, const PairGeo &P, int j, double d0, double cf,
                                              double kq, I nstep, double base, int max_iter, uint32_t &err)
{
    SegT<I> g;
    g.k = seg_none<I>();
    double h[3];
    charge_fixed(H, j, d0, nstep, base, P.L2, P.L, P.sD, cf, max_iter, g, h, err);
    return drive_scalar(P, cf, kq, h);
}

// The drive (small_field times kl = kq / L^2) of the charge cf of a fixed source whose root
// lies in the segment of rows r0, r1, from the step u0 at one light time of L.
// Returns false, for the caller's general solvers, outside small_root's and
// small_field's range or when the root leaves the segment.
template <bool DIFF>
__device__ __forceinline__ bool small_charge(const SmallK &c, double mu, double muI, double w, double u0, double cf, double kl,
                                             const PairGeo &P, const double r0[3], const double r1[3], double &drive)
{
    const double ci = cf * P.iL;
    SmallRoot r;
    small_root<false>(c, mu, w, u0, ci * r0[0], ci * (r1[0] - r0[0]), 0.0, 0.0, r);
    const double b = cf * INV_C * fma(r.u, r1[1] - r0[1], r0[1]);
    const double e = cf * (INV_C * INV_C) * P.L * fma(r.u, r1[2] - r0[2], r0[2]);
    // a root within rounding of a segment end belongs to either side
    const bool ok = fma(fabs(b), c.lz, r.out) <= 1.0 && fabs(r.u - 0.5) <= 0.5 + 1e-9;
    drive = kl * small_field<DIFF>(c, mu, muI, P.pij, r, b, e);
    return ok;
}

// The segment of a fixed source that one light time of L before stage theta points to,
// if it is stored or before t = 0 (the static pre-history, rows d0, 0, 0): the start u0
// in it and its rows.
__device__ __forceinline__ bool stored_segment(const Hist &H, const PairGeo &P, int j, int64_t nstep, double theta,
                                               double w, double d0, double &u0, double r0[3], double r1[3],
                                               uint32_t &err)
{
    const double f = floor(theta - w);
    const int kf = (int)f;
    if (!(f < 0.0)) return false;
    if (nstep + kf >= 0 && -kf > H.mask) err |= ERR_HISTORY;
    const double *p0 = H.ring + ((int64_t)((nstep + kf) & H.mask) * H.n + j) * 3;
    const double *p1 = H.ring + ((int64_t)((nstep + kf + 1) & H.mask) * H.n + j) * 3;
    const bool pre = nstep + kf < 0;
    for (int c = 0; c < 3; ++c) {
        r0[c] = pre ? (c == 0 ? d0 : 0.0) : p0[c];
        r1[c] = pre ? (c == 0 ? d0 : 0.0) : p1[c];
    }
    u0 = theta - w - f;
    return true;
}

// Both charges of a fixed source at one stage time by small_charge.  False: the
// caller takes the general solvers.
template <bool DIFF>
__device__ __forceinline__ bool small_source(const SmallK &c, const Hist &H, const PairGeo &P, int j, double d0, double cfp, double cfm,
                                             double kq, int64_t nstep, double theta, double &e, uint32_t &err)
{
    const double w = P.L * (INV_C * H.inv_dt), mu = P.sD * P.iL, muI = P.sI * P.iL, kl = kq * (P.iL * P.iL);
    double u0, r0[3], r1[3], ep, em;
    if (!stored_segment(H, P, j, nstep, theta, w, d0, u0, r0, r1, err)) return false;
    const bool op = small_charge<DIFF>(c, mu, muI, w, u0, cfp, kl, P, r0, r1, ep);
    const bool om = small_charge<DIFF>(c, mu, muI, w, u0, cfm, -kl, P, r0, r1, em);
    e = ep + em;
    return op && om;
}

// The same for one charge (kq with its sign).  (The kernels for moving origins
// take the general solvers throughout: the series' registers cost them a wave
// per SIMD, 2,048 moving instances of 12 in FP64 47.3 us per step with them, 39.8
// without.)
__device__ __forceinline__ bool small_one(const SmallK &c, const Hist &H, const PairGeo &P, int j, double d0, double cf, double kq,
                                          int64_t nstep, double theta, double &e, uint32_t &err)
{
    const double w = P.L * (INV_C * H.inv_dt);
    double u0, r0[3], r1[3];
    if (!stored_segment(H, P, j, nstep, theta, w, d0, u0, r0, r1, err)) return false;
    return small_charge<false>(c, P.sD * P.iL, P.sI * P.iL, w, u0, cf, kq * (P.iL * P.iL), P, r0, r1, e);
}

template <bool MOVING>
__device__ __forceinline__ double pair_drive(const SmallK &c, const Hist &H, const DipLds &Si, const DipLds &Sj, int j, double cf, double kq,
                             int64_t nstep, double theta, int max_iter, uint32_t &err)
{
    const double base = (double)nstep + theta;
    double X[3] = {Si.ox, Si.oy, Si.oz};
    if (MOVING) origin_at(Si, base * H.dt, X);
    if (!MOVING || Sj.mw == 0.0) {
        const PairGeo P = pair_geo(X, Si, Sj);
        if constexpr (!MOVING) {
            double e;
            if (small_one(c, H, P, j, Sj.d0, cf, kq, nstep, theta, e, err)) return e;
        }
        return fixed_drive(H, P, j, Sj.d0, cf, kq, nstep, base, max_iter, err);
    }
    if constexpr (MOVING) {
        double R[3], v[3], a[3];
        charge_moving(H, Sj, j, cf, nstep, base, X, max_iter, R, v, a, err);
        return charge_field(Si, R, v, a, kq);
    }
    return 0.0;
}

// Velocity and radiation part of one charge's field in the mixed form: with
// n = R/|R|, beta = v/c and kappa = 1 - n.beta, the field of Eq. (E) less its
// static monopole term kq R / |R|^3, projected on p_i, per unit kq, in lengths
// scaled by 1/Ls (ix = Ls / |R|, ga = acceleration Ls / c^2).  The charge
// moves along p_j (beta = be p_j, acceleration ga p_j), so with P = p_i . n,
// X = n . p_j, pij = p_i . p_j and q = pij - P X (p_i . the part of p_j across
// n) it is
//   ix^2 be kappa^-3 [P (X (1 + kappa + kappa^2) - be) - pij (1 - be^2)]
//     - ga q ix kappa^-3,
// where the radiation term's beta parts have cancelled exactly.  Its first
// order in beta, lead = ix^2 be (3 P X - pij) - ga q ix, carries the
// near-field coupling in the phase of the velocity: for close pairs the
// reactive coupling is 1e4 times the dissipative one, so FP32 rounding there
// moves the collective rates by 1e-3 gamma_0.  lead is FP64 (dynamic_lead);
// the rest, which is smaller by a factor of order beta (dynamic_corr_f32:
// (kappa^-3 - 1) = be X (1 + kappa + kappa^2) kappa^-3 taken out exactly), is
// FP32.
__device__ __forceinline__ double dynamic_lead(double P, double X, double ix, double be, double ga, double pij,
                                               double q)
{
    return be * ix * ix * (3.0 * P * X - pij) - ga * q * ix;
}
__device__ __forceinline__ float dynamic_corr_f32(float P, float X, float ix, float be, float ga, float pij, float q)
{
    const float kap = 1.0f - be * X;
    const float s3 = 1.0f + kap + kap * kap;
    const float ik = __builtin_amdgcn_rcpf(kap);
    const float ik3 = ik * ik * ik;
    const float A = P * X * s3 - P * be - pij + pij * be * be;
    return be * be * ix * ix * (X * s3 * ik3 * A - P * X * X * (kap + 2.0f) - P + pij * be) -
           ga * q * ix * be * X * s3 * ik3;
}

// Mixed form of the drive of one source dipole at a target (both charges: +q
// at cfp d p_j, -q at cfm d p_j), at time (nstep + theta) dt.  The retarded
// times are FP64 (the closed form, the two charges sharing one history
// segment).  The field is the sum of
//  - the static monopole difference kq [f(R+) - f(R-)], f(R) = R / |R|^3, the
//    dominant term in the near field, in FP64.  R+ and R- differ by
//    D = (rho- - rho+) p_j, taken exactly from the charges' offsets although
//    far below |R| (1e-4 |R| at 10 nm for a 1e-12 m displacement, down to
//    1e-13 |R| for the small induced moments of distant dipoles), by the
//    identities
//      f(a) - f(b) = D / |a|^3 + b (|b|^3 - |a|^3) / (|a|^3 |b|^3),
//      |b|^3 - |a|^3 = (|b| - |a|) (|a|^2 + |a| |b| + |b|^2),
//      |b| - |a| = -D . (a + b) / (|a| + |b|),
//    in which nothing cancels;
//  - each charge's velocity and radiation terms, first order in beta in FP64
//    (dynamic_lead) and the remainder in FP32 (dynamic_corr_f32).  Against
//    the static term they are of relative size omega |R| / c and its square
//    in the near field, and they have the same sign for both charges (their
//    q beta and q beta_dot agree), so the FP32 remainder's rounding stays at
//    its own size times 2^-24.
// Lengths are scaled by 1/|Delta| so that FP32 stays in range at nanometre
// separations.  A moving source's origin velocity is common to both charges,
// so its velocity terms would cancel: moving sources take the FP64 field of
// each charge.  kq is that of the +q charge.
// Separation of a target at X from a fixed source j for the mixed drive: |Delta|^2,
// |Delta| and its reciprocal, Delta . p_j, and the scaled projections u . p_j,
// p_i . u (u = Delta / |Delta|), p_i . p_j and the acceleration scale L / c^2.
struct MixedGeo {
    double L2, L, iL, sD, cup, ciu, pij, gsc;
};

__device__ __forceinline__ MixedGeo mixed_geo(const double X[3], const DipLds &Si, const DipLds &Sj)
{
    MixedGeo G;
    const double p[3] = {Sj.px, Sj.py, Sj.pz};
    const double dl[3] = {X[0] - Sj.ox, X[1] - Sj.oy, X[2] - Sj.oz};
    G.L2 = dl[0] * dl[0] + dl[1] * dl[1] + dl[2] * dl[2];
    G.sD = dl[0] * p[0] + dl[1] * p[1] + dl[2] * p[2];
    root_rsqrt<true>(G.L2, G.L, G.iL);
    G.cup = G.sD * G.iL;
    G.ciu = (dl[0] * Si.px + dl[1] * Si.py + dl[2] * Si.pz) * G.iL;
    G.pij = Si.px * p[0] + Si.py * p[1] + Si.pz * p[2];
    G.gsc = INV_C * INV_C * G.L;                    // acceleration -> beta_dot L / c
    return G;
}

// The mixed drive of a fixed source from its two charges' stored states hp (+q,
// offset cfp) and hm (-q, offset cfm) at their retarded times.
__device__ __forceinline__ double mixed_field(const MixedGeo &G, double cfp, double cfm, const double hp[3],
                                              const double hm[3], double kq)
{
    const double rp = cfp * hp[0] * G.iL, rm = cfm * hm[0] * G.iL;   // scaled offsets
    // a = u - rp p_j and b = u - rm p_j enter only through u . p_j, p_i . u,
    // p_i . p_j and their own lengths
    const double cup = G.cup, ciu = G.ciu, pij = G.pij;
    // static monopole difference (FP64)
    const double dsc = rm - rp;                     // D = dsc p_j (scaled)
    double ra, ia, rb, ib;
    root_rsqrt<true>(fma(rp, rp - 2.0 * cup, 1.0), ra, ia);
    root_rsqrt<true>(fma(rm, rm - 2.0 * cup, 1.0), rb, ib);
    const double ia3 = ia * ia * ia, ib3 = ib * ib * ib;
    const double dab = -dsc * (2.0 * cup - (rp + rm)) * recip<double>(ra + rb);   // |b| - |a|
    const double c3 = dab * (ra * ra + ra * rb + rb * rb) * ia3 * ib3;
    const double st = dsc * ia3 * pij + c3 * (ciu - rm * pij);
    // velocity and radiation terms of both charges: first order in beta in
    // FP64, the rest in FP32
    const double Pa = (ciu - rp * pij) * ia, Xa = (cup - rp) * ia, Pb = (ciu - rm * pij) * ib, Xb = (cup - rm) * ib;
    const double qa = pij - Pa * Xa, qb = pij - Pb * Xb;
    const double bea = cfp * hp[1] * INV_C, gaa = cfp * hp[2] * G.gsc;
    const double beb = cfm * hm[1] * INV_C, gab = cfm * hm[2] * G.gsc;
    const float fpij = (float)pij;
    const float corr = dynamic_corr_f32((float)Pa, (float)Xa, (float)ia, (float)bea, (float)gaa, fpij, (float)qa) -
                       dynamic_corr_f32((float)Pb, (float)Xb, (float)ib, (float)beb, (float)gab, fpij, (float)qb);
    const double rest = dynamic_lead(Pa, Xa, ia, bea, gaa, pij, qa) - dynamic_lead(Pb, Xb, ib, beb, gab, pij, qb) +
                        (double)corr;
    return kq * G.iL * G.iL * (st + rest);
}

template <bool MOVING>
__device__ __forceinline__ double dipole_drive_mixed(const SmallK &c, const Hist &H, const DipLds &Si, const DipLds &Sj, int j, double kq,
                                     int64_t nstep, double theta, int max_iter, uint32_t &err)
{
    const double base = (double)nstep + theta;
    double X[3] = {Si.ox, Si.oy, Si.oz};
    if (MOVING) origin_at(Si, base * H.dt, X);
    if constexpr (MOVING) {
        if (Sj.mw != 0.0) {
            double R[3], v[3], a[3];
            charge_moving(H, Sj, j, Sj.cfp, nstep, base, X, max_iter, R, v, a, err);
            double e = charge_field(Si, R, v, a, kq);
            charge_moving(H, Sj, j, Sj.cfm, nstep, base, X, max_iter, R, v, a, err);
            return e + charge_field(Si, R, v, a, -kq);
        }
    }
    if constexpr (!MOVING) {
        double e;
        if (small_source<true>(c, H, pair_geo(X, Si, Sj), j, Sj.d0, Sj.cfp, Sj.cfm, kq, nstep, theta, e, err)) return e;
    }
    const MixedGeo G = mixed_geo(X, Si, Sj);
    Seg g;
    g.k = seg_none<int64_t>();
    double hp[3], hm[3];
    charge_fixed(H, j, Sj.d0, nstep, base, G.L2, G.L, G.sD, Sj.cfp, max_iter, g, hp, err);
    charge_fixed(H, j, Sj.d0, nstep, base, G.L2, G.L, G.sD, Sj.cfm, max_iter, g, hm, err);
    return mixed_field(G, Sj.cfp, Sj.cfm, hp, hm, kq);
}

// p_i . E of both charges of source j in FP64 (Eq. (E), total field), one after
// the other in one lane: they share the separation of the origins, its
// projections and the cached history segment (the two charges' retarded times
// lie about 1e-4 of a step apart), so the lane loads the segment once.  The
// per-charge terms are those of pair_drive.
template <bool MOVING>
__device__ __forceinline__ double dipole_drive_fp64(const SmallK &c, const Hist &H, const DipLds &Si, const DipLds &Sj, int j, double kq,
                                    int64_t nstep, double theta, int max_iter, uint32_t &err)
{
    const double base = (double)nstep + theta;
    double X[3] = {Si.ox, Si.oy, Si.oz};
    if (MOVING) origin_at(Si, base * H.dt, X);
    if constexpr (MOVING) {
        if (Sj.mw != 0.0) {
            double R[3], v[3], a[3];
            charge_moving(H, Sj, j, Sj.cfp, nstep, base, X, max_iter, R, v, a, err);
            const double e = charge_field(Si, R, v, a, kq);
            charge_moving(H, Sj, j, Sj.cfm, nstep, base, X, max_iter, R, v, a, err);
            return e + charge_field(Si, R, v, a, -kq);
        }
    }
    const PairGeo P = pair_geo(X, Si, Sj);
    if constexpr (!MOVING) {
        double e;
        if (small_source<false>(c, H, P, j, Sj.d0, Sj.cfp, Sj.cfm, kq, nstep, theta, e, err)) return e;
    }
    Seg g;
    g.k = seg_none<int64_t>();
    double hp[3], hm[3];
    charge_fixed(H, j, Sj.d0, nstep, base, P.L2, P.L, P.sD, Sj.cfp, max_iter, g, hp, err);
    charge_fixed(H, j, Sj.d0, nstep, base, P.L2, P.L, P.sD, Sj.cfm, max_iter, g, hm, err);
    return drive_scalar(P, Sj.cfp, kq, hp) + drive_scalar(P, Sj.cfm, -kq, hm);
}

// The segments charge_fixed starts from at both stage times of a step (those
// of tau = L/c at base_h = n + 1/2 and base_f = n + 1), with the values
// seg_load gives each, loaded without a branch.  The two start points differ
// by half a step (rounding is monotonic, so by less than one), so the second
// segment is the first or the next one, and three ring rows hold both.  Rows
// are taken modulo the ring, so every load stays in bounds, also where a
// segment lies past the newest stored step (a row this launch may be writing):
// that segment is marked empty and its values are not used (charge_fixed goes
// on to the extrapolation, as it would have).
template <typename I>
__device__ __forceinline__ void seg_stages(const Hist &H, int j, double d0, I nstep, double base_h, double base_f,
                                           double L, SegT<I> &gh, SegT<I> &gf, uint32_t &err)
{
    const double sh = base_h - L * INV_C * H.inv_dt, sf = base_f - L * INV_C * H.inv_dt;
    const I kh = sh < 0.0 ? -1 : (I)floor(sh);
    const I kf = sf < 0.0 ? -1 : (I)floor(sf);
    const I k = kh < 0 ? -1 : kh;
    const double *p0 = H.ring + ((I)(k & H.mask) * H.n + j) * 3;
    const double *p1 = H.ring + ((I)((k + 1) & H.mask) * H.n + j) * 3;
    const double *p2 = H.ring + ((I)((k + 2) & H.mask) * H.n + j) * 3;
    const double r0[3] = {p0[0], p0[1], p0[2]}, r1[3] = {p1[0], p1[1], p1[2]}, r2[3] = {p2[0], p2[1], p2[2]};
    const bool preh = kh < 0, pref = kf < 0, next = kf != kh;
    gh.k = preh ? -1 : kh;
    gh.d0 = preh ? d0 : r0[0];
    gh.v0 = preh ? 0.0 : r0[1];
    gh.a0 = preh ? 0.0 : r0[2];
    gh.d1 = preh ? d0 : r1[0];
    gh.v1 = preh ? 0.0 : r1[1];
    gh.a1 = preh ? 0.0 : r1[2];
    gf.k = pref ? -1 : kf;
    gf.d0 = pref ? d0 : (next ? r1[0] : r0[0]);
    gf.v0 = pref ? 0.0 : (next ? r1[1] : r0[1]);
    gf.a0 = pref ? 0.0 : (next ? r1[2] : r0[2]);
    gf.d1 = pref ? d0 : (next ? r2[0] : r1[0]);
    gf.v1 = pref ? 0.0 : (next ? r2[1] : r1[1]);
    gf.a1 = pref ? 0.0 : (next ? r2[2] : r1[2]);
    if ((!preh && kh + H.mask < nstep) || (!pref && kf + H.mask < nstep)) err |= ERR_HISTORY;
    if (kh >= nstep) gh.k = seg_none<I>();
    if (kf >= nstep) gf.k = seg_none<I>();
}

// Both stage drives of a fixed source through the general solvers.
template <bool MIXED>
__device__ __forceinline__ void drive_stages_general(const Hist &H, const DipLds &Si, const DipLds &Sj, int j,
                                                     double kq, int64_t nstep, int max_iter, uint32_t &err,
                                                     double &e_half, double &e_full)
{
    const double X[3] = {Si.ox, Si.oy, Si.oz};
    const PairGeo P = pair_geo(X, Si, Sj);
    const double base_h = (double)nstep + 0.5, base_f = (double)nstep + 1.0;
    Seg gh, gf;
    seg_stages(H, j, Sj.d0, nstep, base_h, base_f, P.L, gh, gf, err);
    double hp[3], hm[3];
    charge_fixed(H, j, Sj.d0, nstep, base_h, P.L2, P.L, P.sD, Sj.cfp, max_iter, gh, hp, err);
    charge_fixed(H, j, Sj.d0, nstep, base_h, P.L2, P.L, P.sD, Sj.cfm, max_iter, gh, hm, err);
    if constexpr (MIXED) e_half = mixed_field(mixed_geo(X, Si, Sj), Sj.cfp, Sj.cfm, hp, hm, kq);
    else e_half = drive_scalar(P, Sj.cfp, kq, hp) + drive_scalar(P, Sj.cfm, -kq, hm);
    charge_fixed(H, j, Sj.d0, nstep, base_f, P.L2, P.L, P.sD, Sj.cfp, max_iter, gf, hp, err);
    charge_fixed(H, j, Sj.d0, nstep, base_f, P.L2, P.L, P.sD, Sj.cfm, max_iter, gf, hm, err);
    if constexpr (MIXED) e_full = mixed_field(mixed_geo(X, Si, Sj), Sj.cfp, Sj.cfm, hp, hm, kq);
    else e_full = drive_scalar(P, Sj.cfp, kq, hp) + drive_scalar(P, Sj.cfm, -kq, hm);
}

// Both stage times of a step (t_n + dt/2 and t_n + dt) for both charges of a
// fixed source.  The usual lane takes small_charge on three stored rows, which hold
// both stages' segments and are loaded together.  False: the segments are not all
// stored, or a root leaves its segment or small_root's range, and the source goes
// through the general solvers.  445 VALU instructions
// per source and step, 688 with the general solvers' closed forms.
template <bool DIFF>
__device__ __forceinline__ bool drive_stages(const SmallK &c, const Hist &H, const DipLds &Si, const DipLds &Sj, int j, double kq,
                                             int64_t nstep, uint32_t &err, double &e_half, double &e_full)
{
    const double X[3] = {Si.ox, Si.oy, Si.oz};
    const PairGeo P = pair_geo(X, Si, Sj);
    const double w = P.L * (INV_C * H.inv_dt);
    const double fh = floor(0.5 - w), ff = floor(1.0 - w);
    const int kh = (int)fh;
    bool ok = ff < 0.0;
    {
        const int64_t k = nstep + kh;
        const double *p0 = H.ring + ((int64_t)(k & H.mask) * H.n + j) * 3;
        const double *p1 = H.ring + ((int64_t)((k + 1) & H.mask) * H.n + j) * 3;
        const double *p2 = H.ring + ((int64_t)((k + 2) & H.mask) * H.n + j) * 3;
        double r0[3] = {p0[0], p0[1], p0[2]}, r1[3] = {p1[0], p1[1], p1[2]};
        const double r2[3] = {p2[0], p2[1], p2[2]};
        const bool next = ff != fh;                 // (by half a step: the same segment or the next)
        double s0[3], s1[3];
        for (int q = 0; q < 3; ++q) {
            s0[q] = next ? r1[q] : r0[q];
            s1[q] = next ? r2[q] : r1[q];
        }
        if (k < 0) {
            // the static pre-history (d0, 0, 0), where the whole wave or none of it is for
            // most of a run
            const bool pre = k + (next ? 1 : 0) < 0;
            for (int q = 0; q < 3; ++q) {
                const double z = q == 0 ? Sj.d0 : 0.0;
                r0[q] = r1[q] = z;
                if (pre) s0[q] = s1[q] = z;
            }
        }
        const double mu = P.sD * P.iL, muI = P.sI * P.iL;
        const double uh = 0.5 - w - fh, uf = 1.0 - w - ff, kl = kq * (P.iL * P.iL);
        double hp, hm, fp, fm;
        ok = small_charge<DIFF>(c, mu, muI, w, uh, Sj.cfp, kl, P, r0, r1, hp) && ok;
        ok = small_charge<DIFF>(c, mu, muI, w, uh, Sj.cfm, -kl, P, r0, r1, hm) && ok;
        ok = small_charge<DIFF>(c, mu, muI, w, uf, Sj.cfp, kl, P, s0, s1, fp) && ok;
        ok = small_charge<DIFF>(c, mu, muI, w, uf, Sj.cfm, -kl, P, s0, s1, fm) && ok;
        e_half = hp + hm;
        e_full = fp + fm;
    }
    if (nstep + kh >= 0 && -kh > H.mask) err |= ERR_HISTORY;
    return ok;
}

// Both stage drives at target i of its instance's M other dipoles (fixed origins), one
// source per lane of LANES and round, added to acc0, acc1.  The sources that
// drive_stages does not take go through the general solvers after the others, 64
// rounds at a time: in one loop the general solvers' registers would add to the usual
// path's.
template <int LANES, bool MIXED>
__device__ __forceinline__ void target_stages(const SmallK &c, const Hist &H, const DipLds &Si,
                                              const double *__restrict__ soa, int n_dip, int i0, int i, int M, int lane,
                                              int64_t nstep, int max_iter, uint32_t &err, double &acc0, double &acc1)
{
    int j;
    DipLds Sj;
    double qj;
    auto source = [&](int jj) {
        j = jj < i ? jj : jj + 1;
        Sj = soa_lds(soa, n_dip, (uint32_t)(i0 + j));
        qj = soa_get(soa, n_dip, SF_Q, (uint32_t)(i0 + j));
    };
    for (int base = lane; base < M; base += 64 * LANES) {
        const int end = min(M, base - lane + 64 * LANES);
        uint64_t left = 0u;
        int round = 0;
        for (int jj = base; jj < end; jj += LANES, ++round) {
            source(jj);
            double eh, ef;
            const bool ok = drive_stages<MIXED>(c, H, Si, Sj, j, qj * K_COUL, nstep, err, eh, ef);
            if (!ok) left |= (uint64_t)1 << round;
            acc0 += ok ? eh : 0.0;
            acc1 += ok ? ef : 0.0;
        }
        while (left) {
            const int r = __ffsll((unsigned long long)left) - 1;
            left &= left - 1u;
            source(base + r * LANES);
            double eh, ef;
            drive_stages_general<MIXED>(H, Si, Sj, j, qj * K_COUL, nstep, max_iter, err, eh, ef);
            acc0 += eh;
            acc1 += ef;
        }
    }
}

// Drive contribution of work unit w of source j: in FP64 one unit per charge
// (w = 0: +q, 1: -q), in the mixed form one unit per source dipole.
template <bool MOVING, bool MIXED>
__device__ __forceinline__ double unit_drive(const SmallK &c, const Hist &H, const DipLds &Si, const DipLds &Sj, int j, double qj,
                                             int w, int64_t nstep, double theta, int max_iter, uint32_t &err)
{
    if constexpr (MIXED) {
        return dipole_drive_mixed<MOVING>(c, H, Si, Sj, j, qj * K_COUL, nstep, theta, max_iter, err);
    } else {
        const double cf = w ? Sj.cfm : Sj.cfp;
        const double kq = (w ? -qj : qj) * K_COUL;
        return pair_drive<MOVING>(c, H, Si, Sj, j, cf, kq, nstep, theta, max_iter, err);
    }
}

template <bool MIXED> constexpr int units_per_source() { return MIXED ? 1 : 2; }

// The stepped kernel's work unit: one source dipole per lane in both forms (its
// targets have many sources, so fewer, fuller units pay; the persistent kernel
// keeps a lane per charge, which shortens the serial chain of small instances).
template <bool MOVING, bool MIXED>
__device__ __forceinline__ double source_drive(const SmallK &c, const Hist &H, const DipLds &Si, const DipLds &Sj, int j, double qj,
                                               int64_t nstep, double theta, int max_iter, uint32_t &err)
{
    if constexpr (MIXED) return dipole_drive_mixed<MOVING>(c, H, Si, Sj, j, qj * K_COUL, nstep, theta, max_iter, err);
    else return dipole_drive_fp64<MOVING>(c, H, Si, Sj, j, qj * K_COUL, nstep, theta, max_iter, err);
}

// Drive fields of all targets of the instance at stage times theta in
// `thetas[0..nth)` (in steps after nstep), written to Eout[th * n + i].
template <int BLOCK, bool MOVING, bool MIXED>
__device__ void drive_all(const SmallK &c, const Hist &H, const DipLds *S, const double *qv, int n, int64_t nstep,
                          const double *thetas, int nth, double *Eout, int max_iter, uint32_t &err)
{
    constexpr int U = units_per_source<MIXED>();
    const int M = U * (n - 1);                    // work units per (target, stage)
    const int G = nth * n;                        // (target, stage) groups
    // lanes per group Lg = 2^lg; the index arithmetic uses shifts (integer
    // division has no hardware instruction), and a group's stage is 0 or 1
    int lg = 0;
    while ((1 << lg) < M && lg < 6) ++lg;
    while (lg > 0 && (G << lg) > BLOCK) --lg;
    const int Lg = 1 << lg;
    const int per_pass = BLOCK >> lg;
    const int tid = threadIdx.x;
    const int sub = tid & (Lg - 1);
    for (int g0 = 0; g0 < G; g0 += per_pass) {
        const int g = g0 + (tid >> lg);
        double acc = 0.0;
        if (g < G && M > 0) {
            const int th = g >= n ? 1 : 0, i = g - th * n;
            for (int m = sub; m < M; m += Lg) {
                const int jj = m / U, w = m % U;
                const int j = jj < i ? jj : jj + 1;
                acc += unit_drive<MOVING, MIXED>(c, H, S[i], S[j], j, qv[j], w, nstep, thetas[th], max_iter, err);
            }
        }
        for (int off = 1; off < Lg; off <<= 1) acc += __shfl_xor(acc, off, 64);
        if (g < G && sub == 0) Eout[g] = acc;
    }
}

template <int BLOCK, bool MOVING, bool MIXED>
__global__ __launch_bounds__(BLOCK) void lo_instances_kernel(const DipDev *__restrict__ dev,
                                                             const int32_t *__restrict__ off,
                                                             const int32_t *__restrict__ inst_list, int ring,
                                                             int64_t steps, double dt,
                                                             double max_vel, int max_iter,
                                                             RunOut out,
                                                             double *__restrict__ state, int resume,
                                                             uint32_t *__restrict__ d_err)
{
    extern __shared__ double lds[];
    const int inst = inst_list[blockIdx.x];
    const int i0 = off[inst];
    const int n = off[inst + 1] - i0;
    const int tid = threadIdx.x;
    if (n <= 0) return;

    // LDS layout: constants, q, Ecur, Emid/Eend, absorbed and radiated energy,
    // oscillator constants (w0^2, gamma0, f, vfac, origin speed, 0.5 / f), (ring)
    DipLds *S = (DipLds *)lds;
    double *qv = (double *)(S + n);
    double *Ecur = qv + n;
    double *Enew = Ecur + n;                    // [2][n]: mid, end
    double *Wab = Enew + 2 * n;
    double *Wra = Wab + n;
    double *Kc = Wra + n;                       // [6][n]
    double *ringp = Kc + 6 * n;
    __shared__ uint32_t s_err;

    for (int j = tid; j < n; j += BLOCK) {
        const DipDev &D = dev[i0 + j];
        S[j] = dip_lds(D);
        qv[j] = D.q;
        Kc[j] = D.omega0 * D.omega0;
        Kc[n + j] = D.gamma0;
        Kc[2 * n + j] = D.f;
        Kc[3 * n + j] = D.vfac;
        Kc[4 * n + j] = D.mspeed;
        Kc[5 * n + j] = D.ehalf;
    }
    if (tid == 0) s_err = 0u;
    __syncthreads();

    const SmallK sk = small_k<true>();
    Hist H{ringp, n, ring - 1, dt, 1.0 / dt};
    uint32_t err = 0u;
    const int64_t ring3 = (int64_t)ring * n * 3;
    int64_t n0 = 0;                             // the run's first step

    if (resume) {
        // continue from the run state: history, E_d(t_n0) and the energy sums
        // (output row 0 is written from the state before this kernel runs)
        n0 = (int64_t)state[0];
        const double *sr = state + state_ring_off(i0, ring);
        for (int64_t k = tid; k < ring3; k += BLOCK) ringp[k] = sr[k];
        const int64_t oe = state_ecur_off(out.n_dip, ring), ow = state_w_off(out.n_dip, ring);
        for (int i = tid; i < n; i += BLOCK) {
            Ecur[i] = state[oe + i0 + i];
            Wab[i] = state[ow + 2 * (i0 + i)];
            Wra[i] = state[ow + 2 * (i0 + i) + 1];
        }
    } else {
        // t = 0: drive from the static pre-history, then sample 0 = (d0, 0, d_ddot(0))
        {
            const double th0[1] = {0.0};
            drive_all<BLOCK, MOVING, MIXED>(sk, H, S, qv, n, 0, th0, 1, Ecur, max_iter, err);
        }
        __syncthreads();
        for (int i = tid; i < n; i += BLOCK) {
            const DipDev &D = dev[i0 + i];
            double *h = ringp + (int64_t)i * 3;
            h[0] = D.d0;
            h[1] = 0.0;
            h[2] = D.f * Ecur[i] - D.omega0 * D.omega0 * D.d0;
            const int gi = i0 + i;
            Wab[i] = 0.0;
            Wra[i] = 0.0;
            put_row(out, 0, gi, D.d0, 0.0, run_energy(D.omega0 * D.omega0, D.ehalf, D.d0, 0.0), Ecur[i], 0.0, 0.0);
        }
    }
    __syncthreads();

    const double thetas[2] = {0.5, 1.0};
    for (int64_t nstep = n0; nstep < n0 + steps; ++nstep) {
        drive_all<BLOCK, MOVING, MIXED>(sk, H, S, qv, n, nstep, thetas, 2, Enew, max_iter, err);
        __syncthreads();
        for (int i = tid; i < n; i += BLOCK) {
            const double w2 = Kc[i], g = Kc[n + i], f = Kc[2 * n + i], vfac = Kc[3 * n + i], ms = Kc[4 * n + i];
            const double *h = ringp + ((int64_t)(nstep & (ring - 1)) * n + i) * 3;
            const double Em = Enew[i], Ee = Enew[n + i], Ec = Ecur[i];
            const double y0 = h[0], y1 = h[1];
            double dn, vn;
            rk4_step(dev[i0 + i].rk, y0, y1, Ec, Em, Ee, dn, vn);
            const double an = f * Ee - g * vn - w2 * dn;
            double *hn = ringp + ((int64_t)((nstep + 1) & (ring - 1)) * n + i) * 3;
            hn[0] = dn;
            hn[1] = vn;
            hn[2] = an;
            Ecur[i] = Ee;
            if (!(isfinite(dn) && isfinite(vn) && isfinite(an))) err |= ERR_NONFINITE;
            if (max_vel > 0.0 && ms + vfac * fabs(vn) > max_vel) err |= ERR_VELOCITY;
            // energy bookkeeping (Sec. 2.5), trapezoid rule over the step
            const double wa = Wab[i] + 0.5 * dt * (y1 * Ec + vn * Ee);
            const double wr = Wra[i] + 0.5 * dt * K_LARMOR * (h[2] * h[2] + an * an);
            Wab[i] = wa;
            Wra[i] = wr;
            const int64_t rel = nstep + 1 - n0;
            const int64_t row = out_row(rel, out.stride);
            if (row >= 0) put_row(out, row, i0 + i, dn, vn, run_energy(w2, Kc[5 * n + i], dn, vn), Ee, wa, wr);
        }
        if (err) atomicOr(&s_err, err);
        __syncthreads();
        if (s_err & (ERR_NONFINITE | ERR_VELOCITY | ERR_HISTORY)) break;
    }
    __syncthreads();
    if (state) {
        // save the run state: history, E_d and the energy sums
        double *sr = state + state_ring_off(i0, ring);
        for (int64_t k = tid; k < ring3; k += BLOCK) sr[k] = ringp[k];
        const int64_t oe = state_ecur_off(out.n_dip, ring), ow = state_w_off(out.n_dip, ring);
        for (int i = tid; i < n; i += BLOCK) {
            state[oe + i0 + i] = Ecur[i];
            state[ow + 2 * (i0 + i)] = Wab[i];
            state[ow + 2 * (i0 + i) + 1] = Wra[i];
        }
    }
    if (tid == 0 && s_err) atomicOr(d_err, s_err);
}

// ---------------------------------------------------------------------------
// Instances of at most SMALL_MAX_N fixed dipoles, one wave each.  A step of such
// an instance is a serial chain (drive, stage sums, RK4, then the next drive reads the
// new sample), so its time is that chain and the instructions its one wave
// issues.  Every lane holds one work unit for the whole run: target i, source j,
// charge w in groups of Lg lanes, stage t_n + dt/2 in lanes 0..31 and t_n + dt in
// lanes 32..63.
//  - The pair's geometry, the history segment its retarded time lies in relative to
//    the current step, and the start u0 there are constants of the unit; the
//    segment's first row is the row the lane loaded a step earlier, so one new row
//    is read per step.  Roots come from small_root, without a branch between
//    stored segments and the extrapolation past the newest sample (ext lanes: the
//    segment's rows coincide and cdt, hdt2 add the Taylor terms).  A root that leaves
//    its segment moves the lane's segment for good (twice per period at most, and
//    only for separations within 1e-4 of a step boundary).
//  - Steps that read before t = 0, and roots that small_root does not take, go
//    through the general solvers.
//  - Group sums by cross-lane moves (DPP, v_permlane32_swap), not LDS permutes; all
//    lanes of group i integrate dipole i (rk4_step), with its state, constants and energy
//    sums in registers, and share its stores: one LDS and one output store a step, each
//    lane its own value and pointer.
// 256 pairs x 4,000 steps, FP64: 2.56 ms (0.63 us per step: 171 VALU and 44 scalar
// instructions, half of the time their dependent chain), 4.81 ms with the closed form and
// two divergent paths, LDS permutes and the RK4 stages in sequence.
//   MIXED: small_field's DIFF form; in the general solvers the +q lane evaluates the
//   source's mixed drive from both charges' states.
// ---------------------------------------------------------------------------
constexpr int SMALL_MAX_N = 4;     // n * Lg <= 32 lanes a stage for n <= 4

// x from the lane at xor 1, 2 or 4 (sums over quads make 4 a mirror of 8 lanes)
template <int CTRL> __device__ __forceinline__ double dpp_move(double x)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}
constexpr int DPP_XOR1 = 0xB1, DPP_XOR2 = 0x4E, DPP_MIRROR8 = 0x141;

// x of lanes 0..31 and of lanes 32..63, each in both halves
__device__ __forceinline__ void both_halves(double x, double &low, double &high)
{
    low = high = x;
    lane_swap<32>(low, high);
}

template <bool MIXED>
__global__ __launch_bounds__(64) void lo_small_kernel(const DipDev *__restrict__ dev, const int32_t *__restrict__ off,
                                                      const int32_t *__restrict__ inst_list, int ring, int64_t steps,
                                                      double dt, double max_vel, int max_iter, RunOut out,
                                                      double *__restrict__ state, int resume,
                                                      uint32_t *__restrict__ d_err)
{
    constexpr int BLOCK = 64;
    extern __shared__ double lds[];
    const int inst = inst_list[blockIdx.x];
    const int i0 = off[inst];
    const int n = off[inst + 1] - i0;
    const int tid = threadIdx.x;
    if (n <= 0) return;
    if (n > SMALL_MAX_N) {                      // the host launches none; never silently skip one
        if (tid == 0) atomicOr(d_err, (uint32_t)ERR_STATE);
        return;
    }

    // LDS layout as lo_instances_kernel's (the t = 0 drive and the run state
    // use it); the step loop reads only the ring
    DipLds *S = (DipLds *)lds;
    double *qv = (double *)(S + n);
    double *Ecur = qv + n;
    double *Wab = Ecur + 3 * n;
    double *Wra = Wab + n;
    double *ringp = Wra + 7 * n;
    __shared__ uint32_t s_err;

    for (int j = tid; j < n; j += BLOCK) {
        const DipDev &D = dev[i0 + j];
        S[j] = dip_lds(D);
        qv[j] = D.q;
    }
    if (tid == 0) s_err = 0u;
    __syncthreads();

    // (mixed: in scalar registers, 241 VGPRs; with them in VGPRs it takes 268 and a SIMD holds one
    // wave: 2,048 pairs 1.37 us per step, 0.83 so)
    const SmallK sk = small_k<!MIXED>();
    Hist H{ringp, n, ring - 1, dt, 1.0 / dt};
    uint32_t err = 0u;
    int64_t n0 = 0;
    if (resume) {
        n0 = (int64_t)state[0];
        const double *sr = state + state_ring_off(i0, ring);
        const int64_t ring3 = (int64_t)ring * n * 3;
        for (int64_t k = tid; k < ring3; k += BLOCK) ringp[k] = sr[k];
        const int64_t oe = state_ecur_off(out.n_dip, ring), ow = state_w_off(out.n_dip, ring);
        for (int i = tid; i < n; i += BLOCK) {
            Ecur[i] = state[oe + i0 + i];
            Wab[i] = state[ow + 2 * (i0 + i)];
            Wra[i] = state[ow + 2 * (i0 + i) + 1];
        }
    } else {
        {
            const double th0[1] = {0.0};
            drive_all<BLOCK, false, MIXED>(sk, H, S, qv, n, 0, th0, 1, Ecur, max_iter, err);
        }
        __syncthreads();
        for (int i = tid; i < n; i += BLOCK) {
            const DipDev &D = dev[i0 + i];
            double *h = ringp + (int64_t)i * 3;
            h[0] = D.d0;
            h[1] = 0.0;
            h[2] = D.f * Ecur[i] - D.omega0 * D.omega0 * D.d0;
            Wab[i] = 0.0;
            Wra[i] = 0.0;
            put_row(out, 0, i0 + i, D.d0, 0.0, run_energy(D.omega0 * D.omega0, D.ehalf, D.d0, 0.0), Ecur[i], 0.0,
                    0.0);
        }
    }
    __syncthreads();

    // this lane's work unit
    const int M = 2 * (n - 1);
    int lg = 1;
    while ((1 << lg) < M) ++lg;
    const int th = tid >> 5, ui = (tid & 31) >> lg, sub = tid & ((1 << lg) - 1);
    const bool live = ui < n, active = live && sub < M;
    const bool plus = (sub & 1) == 0;           // the +q lane of its source's pair
    const int me = live ? ui : 0;
    int uj = 0;
    double ucf = 0.0, ukq = 0.0, ud0 = 0.0, utheta = 0.0;
    PairGeo P{1.0, 1.0, 1.0, 0.0, 0.0, 0.0};
    double mu = 0.0, muI = 0.0, kql2 = 0.0, w = 1.0, ci = 0.0, cb = 0.0, ce = 0.0;
    if (active) {
        const int jj = sub >> 1, wq = sub & 1;
        uj = jj < ui ? jj : jj + 1;
        const DipLds Si = S[ui], Sj = S[uj];
        ucf = wq ? Sj.cfm : Sj.cfp;
        ud0 = Sj.d0;
        utheta = th ? 1.0 : 0.5;
        ukq = (wq ? -qv[uj] : qv[uj]) * K_COUL;
        const double X[3] = {Si.ox, Si.oy, Si.oz};
        P = pair_geo(X, Si, Sj);
        mu = P.sD * P.iL;
        muI = P.sI * P.iL;
        kql2 = ukq * (P.iL * P.iL);
        w = P.L * (INV_C * H.inv_dt);
        ci = ucf * P.iL;
        cb = ucf * INV_C;
        ce = ucf * (INV_C * INV_C) * P.L;
    }
    // the segment, relative to the current step: rows kf and kf + 1, or the newest
    // row alone (kf = 0, extrapolation)
    int kf = active ? (int)floor(utheta - w) : -1;
    if (active && -kf > ring - 1) err |= ERR_HISTORY;     // (the ring covers every light time of the instance)
    double u0 = utheta - w - (double)kf, cdt = 0.0, hdt2 = 0.0, quad = 0.0, mid = 0.5, half = 0.5 + 1e-9;
    // group i's lanes: dipole i's state at the run's first step, constants and sums
    double y0 = 0.0, y1 = 0.0, y2 = 0.0, Ec = 0.0, wab = 0.0, wra = 0.0;
    double w2 = 0.0, gm = 0.0, fq = 0.0, vfac = 0.0, ms = 0.0, eh = 0.0, rk[9];
    for (int q = 0; q < 9; ++q) rk[q] = 0.0;
    if (live) {
        const DipDev &D = dev[i0 + me];
        w2 = D.omega0 * D.omega0;
        gm = D.gamma0;
        fq = D.f;
        vfac = D.vfac;
        ms = D.mspeed;
        eh = D.ehalf;
        for (int q = 0; q < 9; ++q) rk[q] = D.rk[q];
        const double *h = ringp + ((int64_t)(n0 & (ring - 1)) * n + me) * 3;
        y0 = h[0];
        y1 = h[1];
        y2 = h[2];
        Ec = Ecur[me];
        wab = Wab[me];
        wra = Wra[me];
    }
    const bool owner = live && th == 0 && sub == 0;
    // what this lane stores of its dipole: role 0 d, 1 d_dot, 2 the energy (and d_ddot
    // into the ring), 3 E_d; roles 0 and 1 the energy sums when they are asked for
    const int role = !live ? 4 : (th << lg) + sub;
    double *po = role == 0 ? out.d : role == 1 ? out.v : role == 2 ? out.E : role == 3 ? out.Ed : nullptr;
    double *pw = role == 0 ? out.wabs : role == 1 ? out.wrad : nullptr;
    const bool sums = out.wabs || out.wrad;
    const int64_t orow = out.n_dip + i0 + me;    // row 1's entry
    if (po) po += orow;
    if (pw) pw += orow;
    const int ring3 = ring * n * 3;
    const double hdt = 0.5 * dt, hdtl = 0.5 * dt * K_LARMOR;
    const double vlim = max_vel > 0.0 ? max_vel : __builtin_huge_val();
    const uint32_t stop_bits = ERR_NONFINITE | ERR_VELOCITY | ERR_HISTORY;

    // the steps, with 32-bit step indices when the run's last step fits
    auto run_steps = [&](auto index_type) {
      using I = decltype(index_type);
      double g0[3] = {0.0, 0.0, 0.0}, g1[3] = {0.0, 0.0, 0.0};   // the segment's rows (d, d_dot, d_ddot)
      bool rows = false;                           // g0, g1 and nx are this step's
      unsigned nx = 0;                             // ring index of the row the next step adds
      unsigned wx = (unsigned)((((I)n0 + 1) & (I)(ring - 1)) * n + me) * 3u + (role < 3 ? role : 0);
      I togo = (I)(out.stride < (int64_t)std::numeric_limits<I>::max() ? out.stride : (int64_t)std::numeric_limits<I>::max());
      const I stride = togo;
      auto row_index = [&](I k) { return (unsigned)((k & (I)(ring - 1)) * n + uj) * 3u; };
      // index of the row one step later than that at index x
      auto later = [&](unsigned x) {
          const unsigned y = x + 3u * (unsigned)n;
          return min(y, y - (unsigned)ring3);      // (unsigned: y below the ring's end stays)
      };
      auto load_rows = [&](I nstep) {
          const I k = nstep + kf;
          const unsigned a = row_index(k), b = row_index(kf < 0 ? k + 1 : k);
          const bool pre = k < 0;                  // static before t = 0
          for (int q = 0; q < 3; ++q) {
              g0[q] = pre ? (q == 0 ? ud0 : 0.0) : ringp[a + q];
              g1[q] = pre ? (q == 0 ? ud0 : 0.0) : ringp[b + q];
          }
          nx = later(b);
          cdt = kf < 0 ? 0.0 : dt;
          hdt2 = kf < 0 ? 0.0 : 0.5 * dt * dt;
          quad = kf < 0 ? 0.0 : 1.0;
          // roots of this segment: u in [0, 1], from 0 in the extrapolation, up to t = 0
          // in the pre-history (a root within rounding of an end belongs to either side)
          mid = pre ? (double)-k - 1000.0 : kf < 0 ? 0.5 : 1000.0;
          half = (pre || kf >= 0 ? 1000.0 : 0.5) + 1e-9;
      };
      for (I nstep = (I)n0; nstep < (I)(n0 + steps); ++nstep) {
        double acc = 0.0;
        bool done = false;
        for (int hop = 0; hop < 4; ++hop) {
            if (!rows) load_rows(nstep);
            rows = true;
            SmallRoot r;
            small_root<true>(sk, mu, w, u0, ci * g0[0], ci * fma(g0[1], cdt, g1[0] - g0[0]), ci * (g0[2] * hdt2), quad,
                             r);
            const double b = cb * fma(r.u, fma(g0[2], cdt, g1[1] - g0[1]), g0[1]);
            const double e = ce * fma(r.u, g1[2] - g0[2], g0[2]);
            acc = kql2 * small_field<MIXED>(sk, mu, muI, P.pij, r, b, e);
            const bool ok = fma(fabs(b), sk.lz, r.out) <= 1.0 && fabs(r.u - mid) <= half;
            if (!__any(active && !ok)) {
                done = true;
                break;
            }
            // not this segment's root (the lane moves for good), or out of range
            rows = false;
            if (__any(active && !(fma(fabs(b), sk.lz, r.out) <= 1.0))) break;
            const int move = !active || ok ? 0 : r.u < mid ? -1 : 1;
            if (__any(kf + move > 0 || -(kf + move) > ring - 1)) break;   // (no such segment: the general solvers)
            kf += move;
            u0 -= (double)move;
        }
        if (!__any(active && !done)) {
            if (!active) acc = 0.0;
        } else {
            // offsets or speeds beyond small_root's range
            rows = false;
            acc = 0.0;
            if constexpr (MIXED) {
                double h[3] = {0.0, 0.0, 0.0};
                if (active) {
                    SegT<I> g;
                    g.k = seg_none<I>();
                    charge_fixed(H, uj, ud0, nstep, (double)nstep + utheta, P.L2, P.L, P.sD, ucf, max_iter, g, h, err);
                }
                double ho[3];
                for (int q = 0; q < 3; ++q) ho[q] = dpp_move<DPP_XOR1>(h[q]);
                if (active && plus) {
                    const DipLds Si = S[ui], Sj = S[uj];
                    const double X[3] = {Si.ox, Si.oy, Si.oz};
                    acc = mixed_field(mixed_geo(X, Si, Sj), Sj.cfp, Sj.cfm, h, ho, ukq);   // (the +q charge's)
                }
            } else {
                if (active) acc = fixed_drive(H, P, uj, ud0, ucf, ukq, nstep, (double)nstep + utheta, max_iter, err);
            }
        }
        acc += dpp_move<DPP_XOR1>(acc);
        if (lg > 1) acc += dpp_move<DPP_XOR2>(acc);
        if (lg > 2) acc += dpp_move<DPP_MIRROR8>(acc);
        double Em, Ee, dn, vn;
        both_halves(acc, Em, Ee);
        rk4_step(rk, y0, y1, Ec, Em, Ee, dn, vn);
        const double an = fq * Ee - gm * vn - w2 * dn;
        const double dv = role == 0 ? dn : vn;
        if (role < 3) ringp[wx] = role == 2 ? an : dv;
        wx = later(wx);
        // the new samples are read by other lanes of this wave in the next step
        __syncthreads();
        if (rows) {
            if (__any(active && kf < 0 && nstep + kf < 0)) {
                rows = false;                      // (the pre-history ends: both rows anew)
            } else {
                // a stored segment's second row becomes its first
                const double a = ringp[nx], b = ringp[nx + 1], c = ringp[nx + 2];
                g0[0] = kf < 0 ? g1[0] : a;
                g0[1] = kf < 0 ? g1[1] : b;
                g0[2] = kf < 0 ? g1[2] : c;
                g1[0] = a;
                g1[1] = b;
                g1[2] = c;
                nx = later(nx);
            }
        }
        wab = wab + hdt * (y1 * Ec + vn * Ee);
        wra = wra + hdtl * (y2 * y2 + an * an);
        if (--togo == 0) {
            togo = stride;
            const double en = run_energy(w2, eh, dn, vn);
            if (po) {
                *po = role < 2 ? dv : role == 2 ? en : Ee;
                po += out.n_dip;
            }
            if (sums && pw) {
                *pw = role == 0 ? wab : wra;
                pw += out.n_dip;
            }
        }
        y0 = dn;
        y1 = vn;
        y2 = an;
        Ec = Ee;
        // d_ddot is not finite whenever d, d_dot or the drive is not
        const bool nf = !isfinite(an), fast = ms + vfac * fabs(vn) > vlim;
        if (__any(nf || fast || (err & stop_bits) != 0u)) {
            if (nf) err |= ERR_NONFINITE;
            if (fast) err |= ERR_VELOCITY;
            break;
        }
      }
    };
    if (n0 + steps < (int64_t)INT32_MAX) run_steps(int{});
    else run_steps(int64_t{});
    if (owner) {
        Ecur[me] = Ec;
        Wab[me] = wab;
        Wra[me] = wra;
    }
    if (err) atomicOr(&s_err, err);
    __syncthreads();
    if (state) {
        double *sr = state + state_ring_off(i0, ring);
        const int64_t ring3 = (int64_t)ring * n * 3;
        for (int64_t k = tid; k < ring3; k += BLOCK) sr[k] = ringp[k];
        const int64_t oe = state_ecur_off(out.n_dip, ring), ow = state_w_off(out.n_dip, ring);
        for (int i = tid; i < n; i += BLOCK) {
            state[oe + i0 + i] = Ecur[i];
            state[ow + 2 * (i0 + i)] = Wab[i];
            state[ow + 2 * (i0 + i) + 1] = Wra[i];
        }
    }
    if (tid == 0 && s_err) atomicOr(d_err, s_err);
}

// ---------------------------------------------------------------------------
// Instances of SMALL_MAX_N + 1 to GROUP_MAX_N fixed dipoles, a workgroup each: lo_small_kernel's
// step spread over waves.  A lane holds one (target i, source j, stage) for the whole
// run, both charges of the source: their two roots are independent chains that share
// the pair's geometry, and half the lanes of a charge per lane keep to two waves per
// SIMD at most.  The Lg = 8 (n <= 9) or 16 lanes of target i and a stage sum its drive by
// DPP; a wave holds both stages of 32 / Lg targets and integrates them, so only the new
// samples cross waves, behind one barrier a step: the ring holds twice the longest light
// time and three more samples, so the row a wave writes is not one that a wave still
// in its drives can read, and a stop is flagged per step parity, so that every wave
// leaves at the same step.
// Up to 9 dipoles a step is bound by that chain, beyond by the instructions of two waves
// per SIMD.  96 instances, FP64 (mixed), energy sums, us per step by lo_instances_kernel ->
// here: 8 dipoles 4.0 -> 0.94 (3.9 -> 0.99), 12 dipoles 3.4 -> 1.51 (3.7 -> 1.48); 2,048
// instances of 7 5.1 -> 3.1 (5.9 -> 3.0), 1,024 of 12 6.2 -> 6.0 (8.8 -> 5.8).  The series'
// constants sit in scalar registers and waves_per_eu(2) caps the rest at 256 VGPRs: above
// that a SIMD holds one wave (4.0 us for the 2,048 instances).  The mixed form is 12 short
// of that and spills 48 bytes a lane, which its times above include.
// ---------------------------------------------------------------------------
constexpr int GROUP8_MAX_N = 9, GROUP_MAX_N = 16;
constexpr int DPP_MIRROR16 = 0x140;
__host__ __device__ constexpr int group_lg(int n) { return n <= GROUP8_MAX_N ? 3 : 4; }
__host__ __device__ constexpr int group_threads(int n)
{
    return 64 * ((n + (32 >> group_lg(n)) - 1) >> (5 - group_lg(n)));
}

// One charge of a lane's source: its segment relative to the current step (rows kf and
// kf + 1, or the newest row alone), as in lo_small_kernel
struct GroupCharge {
    double ci, cb, ce;                           // offset, speed and acceleration factors
    double u0, cdt, hdt2, quad, mid, half;
    double g0[3], g1[3];
    int kf;
    unsigned nx;
};

template <bool MIXED, int LG>
__global__ __launch_bounds__(group_threads(LG == 3 ? GROUP8_MAX_N : GROUP_MAX_N))
__attribute__((amdgpu_waves_per_eu(2))) void lo_group_kernel(
    const DipDev *__restrict__ dev, const int32_t *__restrict__ off, const int32_t *__restrict__ inst_list, int ring,
    int64_t steps, double dt, double max_vel, int max_iter, RunOut out, double *__restrict__ state, int resume,
    uint32_t *__restrict__ d_err)
{
    extern __shared__ double lds[];
    const int inst = inst_list[blockIdx.x];
    const int i0 = off[inst];
    const int n = off[inst + 1] - i0;
    const int tid = threadIdx.x;
    if (n <= 0) return;
    constexpr int lg = LG;
    const int threads = 64 * ((n + (32 >> LG) - 1) >> (5 - LG));
    if (n - 1 > (1 << LG) || threads > (int)blockDim.x || threads < 128) {   // (the host launches none)
        if (tid == 0) atomicOr(d_err, (uint32_t)ERR_STATE);
        return;
    }
    if (tid >= threads) return;                  // waves that the launch's largest instance needs

    DipLds *S = (DipLds *)lds;                   // LDS layout as lo_instances_kernel's
    double *qv = (double *)(S + n);
    double *Ecur = qv + n;
    double *Wab = Ecur + 3 * n;
    double *Wra = Wab + n;
    double *ringp = Wra + 7 * n;
    __shared__ uint32_t s_err, s_stop[2];        // the run's error bits; a stop at an even or odd step

    for (int j = tid; j < n; j += threads) {
        const DipDev &D = dev[i0 + j];
        S[j] = dip_lds(D);
        qv[j] = D.q;
    }
    if (tid == 0) s_err = s_stop[0] = s_stop[1] = 0u;
    __syncthreads();

    const SmallK sk = small_k<false>();
    Hist H{ringp, n, ring - 1, dt, 1.0 / dt};
    uint32_t err = 0u;
    const int64_t ring_all = (int64_t)ring * n * 3;
    int64_t n0 = 0;
    if (resume) {
        n0 = (int64_t)state[0];
        const double *sr = state + state_ring_off(i0, ring);
        for (int64_t k = tid; k < ring_all; k += threads) ringp[k] = sr[k];
        const int64_t oe = state_ecur_off(out.n_dip, ring), ow = state_w_off(out.n_dip, ring);
        for (int i = tid; i < n; i += threads) {
            Ecur[i] = state[oe + i0 + i];
            Wab[i] = state[ow + 2 * (i0 + i)];
            Wra[i] = state[ow + 2 * (i0 + i) + 1];
        }
    } else {
        if (tid < 128) {
            const double th0[1] = {0.0};
            drive_all<128, false, MIXED>(sk, H, S, qv, n, 0, th0, 1, Ecur, max_iter, err);
        }
        __syncthreads();
        for (int i = tid; i < n; i += threads) {
            const DipDev &D = dev[i0 + i];
            double *h = ringp + (int64_t)i * 3;
            h[0] = D.d0;
            h[1] = 0.0;
            h[2] = D.f * Ecur[i] - D.omega0 * D.omega0 * D.d0;
            Wab[i] = 0.0;
            Wra[i] = 0.0;
            put_row(out, 0, i0 + i, D.d0, 0.0, run_energy(D.omega0 * D.omega0, D.ehalf, D.d0, 0.0), Ecur[i], 0.0,
                    0.0);
        }
    }
    __syncthreads();

    // this lane's target, source and stage
    const int th = (tid >> 5) & 1, sub = tid & ((1 << lg) - 1);
    const int ui = ((tid >> 6) << (5 - lg)) + ((tid & 31) >> lg);
    const bool live = ui < n, active = live && sub < n - 1;
    const int me = live ? ui : 0;
    int uj = 0;
    double ud0 = 0.0, utheta = 0.0, kq = 0.0, kql2 = 0.0, mu = 0.0, muI = 0.0, w = 1.0;
    PairGeo P{1.0, 1.0, 1.0, 0.0, 0.0, 0.0};
    GroupCharge C[2];
    if (active) {
        uj = sub < ui ? sub : sub + 1;
        const DipLds Si = S[ui], Sj = S[uj];
        ud0 = Sj.d0;
        utheta = th ? 1.0 : 0.5;
        kq = qv[uj] * K_COUL;
        const double X[3] = {Si.ox, Si.oy, Si.oz};
        P = pair_geo(X, Si, Sj);
        mu = P.sD * P.iL;
        muI = P.sI * P.iL;
        kql2 = kq * (P.iL * P.iL);
        w = P.L * (INV_C * H.inv_dt);
    }
    const int kf0 = active ? (int)floor(utheta - w) : -1;
    if (active && -kf0 > ring - 1) err |= ERR_HISTORY;    // (the ring covers every light time of the instance)
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const double cf = !active ? 0.0 : c ? S[uj].cfm : S[uj].cfp;
        C[c].ci = cf * P.iL;
        C[c].cb = cf * INV_C;
        C[c].ce = cf * (INV_C * INV_C) * P.L;
        C[c].kf = kf0;
        C[c].u0 = utheta - w - (double)kf0;
        C[c].nx = 0;
    }
    // group i's lanes: dipole i's state at the run's first step, constants and sums
    double y0 = 0.0, y1 = 0.0, y2 = 0.0, Ec = 0.0, wab = 0.0, wra = 0.0;
    double w2 = 0.0, gm = 0.0, fq = 0.0, vfac = 0.0, ms = 0.0, eh = 0.0, rk[9];
    for (int q = 0; q < 9; ++q) rk[q] = 0.0;
    if (live) {
        const DipDev &D = dev[i0 + me];
        w2 = D.omega0 * D.omega0;
        gm = D.gamma0;
        fq = D.f;
        vfac = D.vfac;
        ms = D.mspeed;
        eh = D.ehalf;
        for (int q = 0; q < 9; ++q) rk[q] = D.rk[q];
        const double *h = ringp + ((int64_t)(n0 & (ring - 1)) * n + me) * 3;
        y0 = h[0];
        y1 = h[1];
        y2 = h[2];
        Ec = Ecur[me];
        wab = Wab[me];
        wra = Wra[me];
    }
    // what this lane stores of its dipole: role 0 d, 1 d_dot, 2 the energy (and d_ddot
    // into the ring), 3 E_d; roles 0 and 1 the energy sums when they are asked for
    const int role = !live ? 4 : (th << lg) + sub;
    double *po = role == 0 ? out.d : role == 1 ? out.v : role == 2 ? out.E : role == 3 ? out.Ed : nullptr;
    double *pw = role == 0 ? out.wabs : role == 1 ? out.wrad : nullptr;
    const bool sums = out.wabs || out.wrad;
    const int64_t orow = out.n_dip + i0 + me;    // row 1's entry
    if (po) po += orow;
    if (pw) pw += orow;
    const unsigned ring3 = (unsigned)ring_all;
    const double hdt = 0.5 * dt, hdtl = 0.5 * dt * K_LARMOR;
    const double vlim = max_vel > 0.0 ? max_vel : __builtin_huge_val();
    const uint32_t stop_bits = ERR_NONFINITE | ERR_VELOCITY | ERR_HISTORY;

    bool rows = false, pre_any = false;          // the charges' rows are this step's; some lie before t = 0
    unsigned wx = (unsigned)(((n0 + 1) & (ring - 1)) * n + me) * 3u + (role < 3 ? role : 0);
    int64_t togo = out.stride;
    // index of the row one step later than that at index x
    auto later = [&](unsigned x) {
        const unsigned y = x + 3u * (unsigned)n;
        return min(y, y - ring3);                // (unsigned: y below the ring's end stays)
    };
    auto load_rows = [&](GroupCharge &c, int64_t nstep) {
        const int64_t k = nstep + c.kf;
        const unsigned a = (unsigned)((k & (ring - 1)) * n + uj) * 3u;
        const unsigned b = c.kf < 0 ? later(a) : a;
        const bool pre = k < 0;                  // static before t = 0
        for (int q = 0; q < 3; ++q) {
            c.g0[q] = pre ? (q == 0 ? ud0 : 0.0) : ringp[a + q];
            c.g1[q] = pre ? (q == 0 ? ud0 : 0.0) : ringp[b + q];
        }
        c.nx = later(b);
        c.cdt = c.kf < 0 ? 0.0 : dt;
        c.hdt2 = c.kf < 0 ? 0.0 : 0.5 * dt * dt;
        c.quad = c.kf < 0 ? 0.0 : 1.0;
        // roots of this segment: u in [0, 1], from 0 in the extrapolation, up to t = 0
        // in the pre-history (a root within rounding of an end belongs to either side)
        c.mid = pre ? (double)-k - 1000.0 : c.kf < 0 ? 0.5 : 1000.0;
        c.half = (pre || c.kf >= 0 ? 1000.0 : 0.5) + 1e-9;
        return active && pre;
    };
    for (int64_t nstep = n0; nstep < n0 + steps; ++nstep) {
        double acc = 0.0;
        bool done = false;
        for (int hop = 0; hop < 4; ++hop) {
            if (!rows) {
                const bool p0 = load_rows(C[0], nstep), p1 = load_rows(C[1], nstep);
                pre_any = __any(p0 || p1);
            }
            rows = true;
            double f[2], u[2];
            bool ok[2], in[2];
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const GroupCharge &q = C[c];
                SmallRoot r;
                small_root<true>(sk, mu, w, q.u0, q.ci * q.g0[0], q.ci * fma(q.g0[1], q.cdt, q.g1[0] - q.g0[0]),
                                 q.ci * (q.g0[2] * q.hdt2), q.quad, r);
                const double b = q.cb * fma(r.u, fma(q.g0[2], q.cdt, q.g1[1] - q.g0[1]), q.g0[1]);
                const double e = q.ce * fma(r.u, q.g1[2] - q.g0[2], q.g0[2]);
                f[c] = small_field<MIXED>(sk, mu, muI, P.pij, r, b, e);
                u[c] = r.u;
                in[c] = fma(fabs(b), sk.lz, r.out) <= 1.0;
                ok[c] = in[c] && fabs(r.u - q.mid) <= q.half;
            }
            acc = kql2 * f[0] - kql2 * f[1];
            if (!__any(active && !(ok[0] && ok[1]))) {
                done = true;
                break;
            }
            // not this segment's root (the lane moves for good), or out of range
            rows = false;
            if (__any(active && !(in[0] && in[1]))) break;
            int move[2];
            bool off_ring = false;
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                move[c] = !active || ok[c] ? 0 : u[c] < C[c].mid ? -1 : 1;
                off_ring = off_ring || C[c].kf + move[c] > 0 || -(C[c].kf + move[c]) > ring - 1;
            }
            if (__any(off_ring)) break;          // (no such segment: the general solvers)
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                C[c].kf += move[c];
                C[c].u0 -= (double)move[c];
            }
        }
        if (!done) {
            // offsets or speeds beyond small_root's range
            rows = false;
            acc = 0.0;
            if (active) {
                if constexpr (MIXED) {
                    const DipLds Si = S[ui], Sj = S[uj];
                    const double X[3] = {Si.ox, Si.oy, Si.oz}, base = (double)nstep + utheta;
                    Seg g;
                    g.k = seg_none<int64_t>();
                    double hp[3], hm[3];
                    charge_fixed(H, uj, ud0, nstep, base, P.L2, P.L, P.sD, Sj.cfp, max_iter, g, hp, err);
                    charge_fixed(H, uj, ud0, nstep, base, P.L2, P.L, P.sD, Sj.cfm, max_iter, g, hm, err);
                    acc = mixed_field(mixed_geo(X, Si, Sj), Sj.cfp, Sj.cfm, hp, hm, kq);
                } else {
                    const double base = (double)nstep + utheta;
                    acc = fixed_drive(H, P, uj, ud0, S[uj].cfp, kq, nstep, base, max_iter, err) +
                          fixed_drive(H, P, uj, ud0, S[uj].cfm, -kq, nstep, base, max_iter, err);
                }
            }
        }
        if (!active) acc = 0.0;
        acc += dpp_move<DPP_XOR1>(acc);
        acc += dpp_move<DPP_XOR2>(acc);
        acc += dpp_move<DPP_MIRROR8>(acc);
        if constexpr (LG > 3) acc += dpp_move<DPP_MIRROR16>(acc);
        double Em, Ee, dn, vn;
        both_halves(acc, Em, Ee);
        rk4_step(rk, y0, y1, Ec, Em, Ee, dn, vn);
        const double an = fq * Ee - gm * vn - w2 * dn;
        const double dv = role == 0 ? dn : vn;
        // d_ddot is not finite whenever d, d_dot or the drive is not
        if (!isfinite(an)) err |= ERR_NONFINITE;
        if (ms + vfac * fabs(vn) > vlim) err |= ERR_VELOCITY;
        if (role < 3) ringp[wx] = role == 2 ? an : dv;
        if (err & stop_bits) s_stop[nstep & 1] = 1u;
        wx = later(wx);
        __syncthreads();
        if (rows) {
            if (pre_any) {
                rows = false;                    // (the pre-history may end: both rows anew)
            } else {
                // a stored segment's second row becomes its first
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    GroupCharge &q = C[c];
                    for (int k = 0; k < 3; ++k) {
                        const double x = ringp[q.nx + k];
                        q.g0[k] = q.kf < 0 ? q.g1[k] : x;
                        q.g1[k] = x;
                    }
                    q.nx = later(q.nx);
                }
            }
        }
        const bool stop = s_stop[nstep & 1] != 0u;
        wab = wab + hdt * (y1 * Ec + vn * Ee);
        wra = wra + hdtl * (y2 * y2 + an * an);
        if (--togo == 0) {
            togo = out.stride;
            const double en = run_energy(w2, eh, dn, vn);
            if (po) {
                *po = role < 2 ? dv : role == 2 ? en : Ee;
                po += out.n_dip;
            }
            if (sums && pw) {
                *pw = role == 0 ? wab : wra;
                pw += out.n_dip;
            }
        }
        y0 = dn;
        y1 = vn;
        y2 = an;
        Ec = Ee;
        if (stop) break;
    }
    if (live && th == 0 && sub == 0) {
        Ecur[me] = Ec;
        Wab[me] = wab;
        Wra[me] = wra;
    }
    if (err) atomicOr(&s_err, err);
    __syncthreads();
    if (state) {
        double *sr = state + state_ring_off(i0, ring);
        for (int64_t k = tid; k < ring_all; k += threads) sr[k] = ringp[k];
        const int64_t oe = state_ecur_off(out.n_dip, ring), ow = state_w_off(out.n_dip, ring);
        for (int i = tid; i < n; i += threads) {
            state[oe + i0 + i] = Ecur[i];
            state[ow + 2 * (i0 + i)] = Wab[i];
            state[ow + 2 * (i0 + i) + 1] = Wra[i];
        }
    }
    if (tid == 0 && s_err) atomicOr(d_err, s_err);
}

// ---------------------------------------------------------------------------
// Large instances: one workgroup per target dipole, one launch per step.
// The step index comes from a device counter (advanced by step_advance_kernel)
// so that a captured sequence of steps can be replayed.  Block b advances dipole
// tgt[b]; its sources are the other dipoles of the same instance, whose history
// ring sits at ring + ring_base[b] ([ring][n][3]).  Writing step n+1 of dipole
// i touches the slot of step n+1-ring, which no retarded time of this step can
// reach, so all blocks of a launch may run in any order.
// ---------------------------------------------------------------------------


// Register budgets of the launches by targets: FEW targets (at most two workgroups per CU), SOME
// (up to four) with at most 128 other dipoles each or, SOME_LARGE, with more, and MANY.
enum StepPlan { MANY, FEW, SOME, SOME_LARGE };

template <int BLOCK, bool MOVING, bool MIXED, int PLAN>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(PLAN == FEW && !MOVING ? 2 : 3))) void lo_step_kernel(const DipDev *__restrict__ dev, const int32_t *__restrict__ tgt,
                                                        const int32_t *__restrict__ tgt_lo,
                                                        const int32_t *__restrict__ tgt_n,
                                                        const int64_t *__restrict__ ring_base, double *__restrict__ ring,
                                                        double *__restrict__ Ecur, double *__restrict__ W,
                                                        const int64_t *__restrict__ step_ctr, int kstep,
                                                        int ring_depth, double dt, double max_vel, int max_iter,
                                                        int init, RunOut out,
                                                        const double *__restrict__ soa, uint32_t *__restrict__ d_err)
{
    __shared__ double red[2][BLOCK / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int gi = tgt[blockIdx.x];
    const int i0 = tgt_lo[blockIdx.x];
    const int n = tgt_n[blockIdx.x];
    const int i = gi - i0;
    const int64_t nstep = init ? 0 : *step_ctr + kstep;
    double *rp = ring + ring_base[blockIdx.x];
    Hist H{rp, n, ring_depth - 1, dt, 1.0 / dt};
    uint32_t err = 0u;
    const DipLds Si = dip_lds(dev[gi]);
    const int M = n - 1;                             // source dipoles per stage
    const int nth = init ? 1 : 2;
    // Lane layout.  A launch with many targets is throughput-bound: a lane
    // takes one source for both stage times (the fewest instructions per drive).
    // A launch with few targets (all plans but MANY: at most one workgroup per SIMD) is a
    // latency chain, and the shortest chain that fits the block wins: in FP64
    // one charge per lane (4 drives' worth of lanes per source), else one source
    // per (stage, lane); in the mixed form one source per (stage, lane).  Sources that
    // do not fit so take both stages in a lane (900 dipoles, mixed: 38.9 us per step
    // with a lane per stage).
    const int layout = PLAN == MANY ? 0 : (!MIXED && 2 * nth * M <= BLOCK) ? 2 : (nth * M <= BLOCK) ? 1 : 0;
    const int units = layout == 2 ? 2 * nth * M : (layout == 1 ? nth * M : M);
    // the target's own state (only this workgroup writes it, and only at its
    // end): when the last lane has no pair work it reads the state into LDS
    // while the others solve, so the tail does not wait on those loads; held
    // in LDS, the values add no register pressure to the pair loop
    __shared__ double own[6];
    const bool early = !init && units < BLOCK;
    if (early && tid == BLOCK - 1) {
        const double *h = rp + ((int64_t)(nstep & (ring_depth - 1)) * n + i) * 3;
        own[0] = h[0];
        own[1] = h[1];
        own[2] = h[2];
        own[3] = Ecur[gi];
        own[4] = W[2 * gi];
        own[5] = W[2 * gi + 1];
    }
    // (with many targets the constants sit in scalar registers and three waves share a
    // SIMD: 10 instances of 160 14.9 us per step, 16.8 at two waves; with few the scalar
    // moves would lengthen the chain, 4.4 against 4.05 us at 32 dipoles.  Two waves hold two
    // workgroups per CU, so that from 513 targets on some would wait for a second turn: 40
    // instances of 16 5.9 us per step at two waves, 4.5 at three, 4 of 200 12.0 and 10.4)
    const SmallK c = small_k<PLAN == FEW || PLAN == SOME>();
    double acc0 = 0.0, acc1 = 0.0;                   // stage t_n + dt/2 (or t = 0), stage t_n + dt
    if (layout == 0) {
        // a lane takes one source for both stage times.  A launch of few targets lasts as long
        // as its slowest workgroup, and at each step some workgroup has a source that
        // drive_stages does not take.  So such a source goes on in place, on the values it has (3
        // instances of 200 9.1 us per step, 9.5 in a pass of its own), and where a lane has one
        // source and a CU at most two workgroups, all take the general solvers at once (1 of 200
        // 6.1 us per step, 6.9 with drive_stages first; 1 of 300, two rounds, 9.6 and 8.3)
        if (MOVING || init) {
            for (int jj = tid; jj < M; jj += BLOCK) {
                const int j = jj < i ? jj : jj + 1;
                const DipLds Sj = soa_lds(soa, out.n_dip, (uint32_t)(i0 + j));
                const double qj = soa_get(soa, out.n_dip, SF_Q, (uint32_t)(i0 + j));
                acc0 += source_drive<MOVING, MIXED>(c, H, Si, Sj, j, qj, nstep, init ? 0.0 : 0.5, max_iter, err);
                if (!init) acc1 += source_drive<MOVING, MIXED>(c, H, Si, Sj, j, qj, nstep, 1.0, max_iter, err);
            }
        } else if constexpr (PLAN == FEW || PLAN == SOME_LARGE) {
            for (int jj = tid; jj < M; jj += BLOCK) {
                const int j = jj < i ? jj : jj + 1;
                const DipLds Sj = soa_lds(soa, out.n_dip, (uint32_t)(i0 + j));
                const double kq = soa_get(soa, out.n_dip, SF_Q, (uint32_t)(i0 + j)) * K_COUL;
                double eh, ef;
                if ((PLAN == FEW && M <= BLOCK) || !drive_stages<MIXED>(c, H, Si, Sj, j, kq, nstep, err, eh, ef))
                    drive_stages_general<MIXED>(H, Si, Sj, j, kq, nstep, max_iter, err, eh, ef);
                acc0 += eh;
                acc1 += ef;
            }
        } else if constexpr (PLAN == MANY) {
            target_stages<BLOCK, MIXED>(c, H, Si, soa, out.n_dip, i0, i, M, tid, nstep, max_iter, err, acc0, acc1);
        }                                            // (SOME's targets all have layout 1 or 2)
    } else if (layout == 2) {
        // FP64, few targets: a lane per (stage, source, charge)
        for (int m = tid; m < 2 * nth * M; m += BLOCK) {
            const int th = m >= 2 * M ? 1 : 0, r = m - th * 2 * M;
            const int jj = r >> 1, w = r & 1;
            const int j = jj < i ? jj : jj + 1;
            const DipLds Sj = soa_lds(soa, out.n_dip, (uint32_t)(i0 + j));
            const double qj = soa_get(soa, out.n_dip, SF_Q, (uint32_t)(i0 + j));
            const double cf = w ? Sj.cfm : Sj.cfp, kq = (w ? -qj : qj) * K_COUL;
            const double theta = init ? 0.0 : (th ? 1.0 : 0.5);
            const double e = pair_drive<MOVING>(c, H, Si, Sj, j, cf, kq, nstep, theta, max_iter, err);
            if (th) acc1 += e; else acc0 += e;
        }
    } else {
        // a lane per (stage, source), for few targets
        for (int m = tid; m < nth * M; m += BLOCK) {
            const int th = m >= M ? 1 : 0, jj = m - th * M;    // (nth <= 2 stages)
            const int j = jj < i ? jj : jj + 1;
            const DipLds Sj = soa_lds(soa, out.n_dip, (uint32_t)(i0 + j));
            const double qj = soa_get(soa, out.n_dip, SF_Q, (uint32_t)(i0 + j));
            const double theta = init ? 0.0 : (th ? 1.0 : 0.5);
            const double e = source_drive<MOVING, MIXED>(c, H, Si, Sj, j, qj, nstep, theta, max_iter, err);
            if (th) acc1 += e; else acc0 += e;
        }
    }
    // lane 0 reads the target's constants here, and its state too without the
    // early read, so that the loads are in flight during the block sums (read
    // after the barrier they added one memory round trip to every workgroup)
    double st[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    double om = 0.0, gm = 0.0, fq = 0.0, dd0 = 0.0, eh = 0.0, ms = 0.0, vf = 0.0, rk[9];
    for (int q = 0; q < 9; ++q) rk[q] = 0.0;
    if (tid == 0) {
        const DipDev &D = dev[gi];
        for (int q = 0; q < 9; ++q) rk[q] = D.rk[q];
        om = D.omega0;
        gm = D.gamma0;
        fq = D.f;
        dd0 = D.d0;
        eh = D.ehalf;
        ms = D.mspeed;
        vf = D.vfac;
        if (!init && !early) {
            const double *h = rp + ((int64_t)(nstep & (ring_depth - 1)) * n + i) * 3;
            st[0] = h[0];
            st[1] = h[1];
            st[2] = h[2];
            st[3] = Ecur[gi];
            st[4] = W[2 * gi];
            st[5] = W[2 * gi + 1];
        }
    }
    // block sums in a fixed order: within each wave, then over the waves
    for (int o = 32; o > 0; o >>= 1) {
        acc0 += __shfl_xor(acc0, o, 64);
        acc1 += __shfl_xor(acc1, o, 64);
    }
    if (lane == 0) {
        red[0][wave] = acc0;
        red[1][wave] = acc1;
    }
    __syncthreads();
    if (tid == 0) {
        double s0 = red[0][0], s1 = red[1][0];
        for (int v = 1; v < BLOCK / 64; ++v) {
            s0 += red[0][v];
            s1 += red[1][v];
        }
        const double w2 = om * om, g = gm, f = fq;
        if (init) {
            // t = 0: drive from the static pre-history, sample 0 = (d0, 0, d_ddot(0))
            const double E0 = s0;
            double *h = rp + (int64_t)i * 3;
            h[0] = dd0;
            h[1] = 0.0;
            h[2] = f * E0 - w2 * dd0;
            Ecur[gi] = E0;
            W[2 * gi] = 0.0;
            W[2 * gi + 1] = 0.0;
            put_row(out, 0, gi, dd0, 0.0, run_energy(w2, eh, dd0, 0.0), E0, 0.0, 0.0);
        } else {
            const double Em = s0, Ee = s1;
            double y0, y1, a0, Ec, W0, W1;
            if (early) {
                y0 = own[0];
                y1 = own[1];
                a0 = own[2];
                Ec = own[3];
                W0 = own[4];
                W1 = own[5];
            } else {
                y0 = st[0];
                y1 = st[1];
                a0 = st[2];
                Ec = st[3];
                W0 = st[4];
                W1 = st[5];
            }
            double dn, vn;
            rk4_step(rk, y0, y1, Ec, Em, Ee, dn, vn);
            const double an = f * Ee - g * vn - w2 * dn;
            double *hn = rp + ((int64_t)((nstep + 1) & (ring_depth - 1)) * n + i) * 3;
            hn[0] = dn;
            hn[1] = vn;
            hn[2] = an;
            Ecur[gi] = Ee;
            if (!(isfinite(dn) && isfinite(vn) && isfinite(an))) err |= ERR_NONFINITE;
            if (max_vel > 0.0 && ms + vf * fabs(vn) > max_vel) err |= ERR_VELOCITY;
            // energy bookkeeping (Sec. 2.5), trapezoid rule over the step
            const double wa = W0 + 0.5 * dt * (y1 * Ec + vn * Ee);
            const double wr = W1 + 0.5 * dt * K_LARMOR * (a0 * a0 + an * an);
            W[2 * gi] = wa;
            W[2 * gi + 1] = wr;
            const int64_t rel = nstep + 1 - step_ctr[1];       // steps since the run's first
            const int64_t row = out_row(rel, out.stride);
            if (row >= 0) put_row(out, row, gi, dn, vn, run_energy(w2, eh, dn, vn), Ee, wa, wr);
        }
    }
    if (err) atomicOr(d_err, err);
}

// Launches with many targets of fixed dipoles: one wave per target, four to a
// workgroup.  Such a launch is bound by VALU issue as far as memory latency is hidden:
// a wave's start (its target's constants, three dependent loads) and end (the
// target's state, the lane sums, the step) are a chain of several microseconds, which
// one wave per target pays once for its ceil((n - 1) / 64) rounds, where a workgroup per
// target pays it in four waves for a quarter of the rounds each: 300 instances of 16, FP64,
// per step 10.5 us, 24.8 by workgroups.  Three waves per SIMD: four leave 128 VGPRs, 26
// short (11.3 us, and 20 instances of 96 12.7 for 11.0).  Large instances are bound by their
// row gathers as much as by VALU issue (lo_tile_kernel).
template <bool MIXED>
__global__ __launch_bounds__(256, 3) void lo_wave_kernel(const DipDev *__restrict__ dev, const int32_t *__restrict__ tgt,
                                                         const int32_t *__restrict__ tgt_lo,
                                                         const int32_t *__restrict__ tgt_n,
                                                         const int64_t *__restrict__ ring_base, int n_tgt,
                                                         double *__restrict__ ring, double *__restrict__ Ecur,
                                                         double *__restrict__ W, const int64_t *__restrict__ step_ctr,
                                                         int kstep, int ring_depth, double dt, double max_vel,
                                                         int max_iter, RunOut out, const double *__restrict__ soa,
                                                         uint32_t *__restrict__ d_err)
{
    const int lane = threadIdx.x & 63;
    const int b = __builtin_amdgcn_readfirstlane((int)blockIdx.x * 4 + (int)(threadIdx.x >> 6));
    if (b >= n_tgt) return;
    const int gi = tgt[b], i0 = tgt_lo[b], n = tgt_n[b], i = gi - i0;
    const int64_t nstep = *step_ctr + kstep;
    double *rp = ring + ring_base[b];
    const Hist H{rp, n, ring_depth - 1, dt, 1.0 / dt};
    const DipLds Si = dip_lds(dev[gi]);
    const SmallK c = small_k<false>();
    uint32_t err = 0u;
    double acc0 = 0.0, acc1 = 0.0;
    target_stages<64, MIXED>(c, H, Si, soa, out.n_dip, i0, i, n - 1, lane, nstep, max_iter, err, acc0, acc1);
    // the target's constants and state, in flight during the sums
    const DipDev &D = dev[gi];
    double rk[9];
    for (int q = 0; q < 9; ++q) rk[q] = D.rk[q];
    const double w2 = D.omega0 * D.omega0, g = D.gamma0, f = D.f, eh = D.ehalf, ms = D.mspeed, vf = D.vfac;
    const double *h = rp + ((int64_t)(nstep & (ring_depth - 1)) * n + i) * 3;
    const double y0 = h[0], y1 = h[1], a0 = h[2], Ec = Ecur[gi], W0 = W[2 * gi], W1 = W[2 * gi + 1];
    for (int o = 32; o > 0; o >>= 1) {
        acc0 += __shfl_xor(acc0, o, 64);
        acc1 += __shfl_xor(acc1, o, 64);
    }
    if (lane == 0) {
        double dn, vn;
        rk4_step(rk, y0, y1, Ec, acc0, acc1, dn, vn);
        const double an = f * acc1 - g * vn - w2 * dn;
        double *hn = rp + ((int64_t)((nstep + 1) & (ring_depth - 1)) * n + i) * 3;
        hn[0] = dn;
        hn[1] = vn;
        hn[2] = an;
        Ecur[gi] = acc1;
        if (!(isfinite(dn) && isfinite(vn) && isfinite(an))) err |= ERR_NONFINITE;
        if (max_vel > 0.0 && ms + vf * fabs(vn) > max_vel) err |= ERR_VELOCITY;
        // energy bookkeeping (Sec. 2.5), trapezoid rule over the step
        const double wa = W0 + 0.5 * dt * (y1 * Ec + vn * acc1);
        const double wr = W1 + 0.5 * dt * K_LARMOR * (a0 * a0 + an * an);
        W[2 * gi] = wa;
        W[2 * gi + 1] = wr;
        const int64_t row = out_row(nstep + 1 - step_ctr[1], out.stride);
        if (row >= 0) put_row(out, row, gi, dn, vn, run_energy(w2, eh, dn, vn), acc1, wa, wr);
    }
    if (err) atomicOr(d_err, err);
}

// ---------------------------------------------------------------------------
// Many fixed targets in instances large enough to share sources: lo_wave_kernel's drives
// with a lane per target.  That kernel is bound by its row gathers as much as by its
// arithmetic: 64 sources' rows lie in 64 cache lines per load, and the texture unit takes
// one line a cycle (557 line accesses against 445 VALU instructions per wave and round;
// unit 71 % busy, VALU 61 %).  Here a workgroup stages the sample window of TILE sources,
// every row any light time of the call can reach, in LDS by wide loads, once for up to
// 128 targets, and the lanes gather from LDS; the source is uniform, so its constants come
// by scalar loads, and the rows before t = 0 are staged as what they are.  A window's rows
// are padded to an odd count: 6 dwords a row put 64 lanes' rows on 32 banks.
// A unit is 128 targets x `chunk` sources of one instance; its waves are two target
// halves x two source phases (64 targets or fewer: four phases) and leave one partial sum
// per target and stage, which lo_finish_kernel adds in order and integrates.
// 64 clusters of 2 to 975 dipoles, FP64: 130 us per step there, 91 here and 4 in
// lo_finish_kernel (VALU-issue bound, 419 instructions per source and step; loads of the
// window one at a time: 102).
// ---------------------------------------------------------------------------
constexpr int TILE_TARGETS = 128;

// One source's both stage drives from its staged window (row r is step nstep - (R-1) + r).
template <bool DIFF>
__device__ __forceinline__ bool tile_drive(const SmallK &c, const double *win, int R, const DipLds &Si, const DipLds &Sj,
                                           double kq, double inv_dt, int64_t nstep, double &e_half, double &e_full)
{
    const double X[3] = {Si.ox, Si.oy, Si.oz};
    const PairGeo P = pair_geo(X, Si, Sj);
    const double w = P.L * (INV_C * inv_dt);
    const double fh = floor(0.5 - w), ff = floor(1.0 - w);
    const int kh = (int)fh, idx = R - 1 + kh;
    bool ok = ff < 0.0 && idx >= 0;
    const int next = ff != fh ? 1 : 0;              // (by half a step: the same segment or the next)
    const double *p = win + 3 * min(max(idx, 0), R - 2), *q = p + 3 * next;
    double r0[3] = {p[0], p[1], p[2]}, r1[3] = {p[3], p[4], p[5]};
    double s0[3] = {q[0], q[1], q[2]}, s1[3] = {q[3], q[4], q[5]};
    if (nstep < R) {
        // a segment that ends at t = 0 is static throughout
        if (nstep + kh == -1) {
            for (int k = 0; k < 3; ++k) r1[k] = r0[k];
        }
        if (nstep + kh + next == -1) {
            for (int k = 0; k < 3; ++k) s1[k] = s0[k];
        }
    }
    const double mu = P.sD * P.iL, muI = P.sI * P.iL;
    const double uh = 0.5 - w - fh, uf = 1.0 - w - ff, kl = kq * (P.iL * P.iL);
    double hp, hm, fp, fm;
    ok = small_charge<DIFF>(c, mu, muI, w, uh, Sj.cfp, kl, P, r0, r1, hp) && ok;
    ok = small_charge<DIFF>(c, mu, muI, w, uh, Sj.cfm, -kl, P, r0, r1, hm) && ok;
    ok = small_charge<DIFF>(c, mu, muI, w, uf, Sj.cfp, kl, P, s0, s1, fp) && ok;
    ok = small_charge<DIFF>(c, mu, muI, w, uf, Sj.cfm, -kl, P, s0, s1, fm) && ok;
    e_half = hp + hm;
    e_full = fp + fm;
    return ok;
}

template <bool MIXED>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void lo_tile_kernel(
    const DipDev *__restrict__ dev, const TileUnit *__restrict__ units, const int64_t *__restrict__ ring_base, int n_tgt,
    const double *__restrict__ ring, double *__restrict__ part, const int64_t *__restrict__ step_ctr, int kstep,
    int ring_depth, double dt, int R, int tile, int chunk, int max_iter, int n_dip, const double *__restrict__ soa,
    uint32_t *__restrict__ d_err)
{
    extern __shared__ double win[];                  // [tile][R][3], 8 doubles of padding
    const TileUnit U = units[blockIdx.x];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t nstep = *step_ctr + kstep;
    const double *rp = ring + ring_base[U.b0];
    const Hist H{rp, U.n, ring_depth - 1, dt, 1.0 / dt};
    const int halves = U.n - U.t0 > 64 ? 2 : 1;
    const int phase = wave / halves, phases = 4 / halves;
    const int i = U.t0 + (wave % halves) * 64 + lane;
    const bool live = i < U.n;
    const DipLds Si = soa_lds(soa, n_dip, (uint32_t)(U.i0 + (live ? i : U.t0)));
    const SmallK c = small_k<false>();
    uint32_t err = 0u;
    double acc0 = 0.0, acc1 = 0.0;
    uint64_t left = 0u;
    int round = 0;
    for (int s = U.s0; s < U.s1; s += tile) {
        const int here = min(tile, U.s1 - s);
        __syncthreads();
        // thread t: element t % (3 * here) of every row, rows t / (3 * here) and on
        const int cols = 3 * here, rows_at_once = 256 / cols;
        const int col = tid % cols, src = col / 3, q = col - 3 * src;
        if (tid < cols * rows_at_once) {
            const double pre = q == 0 ? dev[U.i0 + s + src].d0 : 0.0;
            double *dst = win + src * R * 3 + q;
            // in batches, so that a batch's loads are in flight together
            constexpr int BATCH = 8;
            for (int r = tid / cols; r < R; r += BATCH * rows_at_once) {
                double v[BATCH];
#pragma unroll
                for (int u = 0; u < BATCH; ++u) {
                    const int64_t k = nstep - (R - 1) + min(r + u * rows_at_once, R - 1);
                    v[u] = k < 0 ? pre : rp[((int64_t)(k & H.mask) * U.n + s) * 3 + col];
                }
#pragma unroll
                for (int u = 0; u < BATCH; ++u)
                    if (r + u * rows_at_once < R) dst[3 * (r + u * rows_at_once)] = v[u];
            }
        }
        __syncthreads();
        for (int m = phase; m < here; m += phases, ++round) {
            const int j = s + m;
            const DipDev &D = dev[U.i0 + j];
            const DipLds Sj = dip_lds(D);
            double eh, ef;
            const bool ok = tile_drive<MIXED>(c, win + m * R * 3, R, Si, Sj, D.q * K_COUL, H.inv_dt, nstep, eh, ef);
            if (!ok && live && j != i) left |= (uint64_t)1 << round;
            const bool add = ok && j != i;
            acc0 += add ? eh : 0.0;
            acc1 += add ? ef : 0.0;
        }
    }
    // the sources tile_drive does not take, by the general solvers: round r of this wave is
    // source (r / per_tile) * tile + phase + (r % per_tile) * phases
    const int per_tile = (tile - phase + phases - 1) / phases;
    while (left) {
        const int r = __ffsll((unsigned long long)left) - 1;
        left &= left - 1u;
        const int j = U.s0 + (r / per_tile) * tile + phase + (r % per_tile) * phases;
        double eh, ef;
        drive_stages_general<MIXED>(H, Si, dip_lds(dev[U.i0 + j]), j, dev[U.i0 + j].q * K_COUL, nstep, max_iter, err, eh,
                                    ef);
        acc0 += eh;
        acc1 += ef;
    }
    // the phases' sums, in order
    __syncthreads();
    win[tid] = acc0;
    win[256 + tid] = acc1;
    __syncthreads();
    if (phase == 0 && live) {
        for (int k = 1; k < phases; ++k) {
            acc0 += win[tid + 64 * halves * k];
            acc1 += win[256 + tid + 64 * halves * k];
        }
        double *out = part + (int64_t)(U.s0 / chunk) * 2 * n_tgt + U.b0 + i;
        out[0] = acc0;
        out[n_tgt] = acc1;
    }
    if (err) atomicOr(d_err, err);
}

// A target's state at the step's start.
struct TargetState {
    double y0, y1, a0, Ec, W0, W1;
};
__device__ __forceinline__ TargetState target_state(const Hist &H, int gi, int i, const double *Ecur, const double *W,
                                                    int64_t nstep)
{
    const double *h = H.ring + ((int64_t)(nstep & H.mask) * H.n + i) * 3;
    return {h[0], h[1], h[2], Ecur[gi], W[2 * gi], W[2 * gi + 1]};
}

// The end of a target's step: RK4 with the drives at t_n + dt/2 and t_n + dt, the new
// sample, the energy sums and the output row.
__device__ __forceinline__ void finish_target(const DipDev &D, const TargetState &S, int gi, int i, const Hist &H, double *ring, double *Ecur, double *W,
                                              int64_t nstep, int64_t n0, double Em, double Ee, double max_vel,
                                              const RunOut &out, uint32_t &err)
{
    const double w2 = D.omega0 * D.omega0;
    double dn, vn;
    rk4_step(D.rk, S.y0, S.y1, S.Ec, Em, Ee, dn, vn);
    const double an = D.f * Ee - D.gamma0 * vn - w2 * dn;
    double *hn = ring + ((int64_t)((nstep + 1) & H.mask) * H.n + i) * 3;
    hn[0] = dn;
    hn[1] = vn;
    hn[2] = an;
    Ecur[gi] = Ee;
    if (!(isfinite(dn) && isfinite(vn) && isfinite(an))) err |= ERR_NONFINITE;
    if (max_vel > 0.0 && D.mspeed + D.vfac * fabs(vn) > max_vel) err |= ERR_VELOCITY;
    // energy bookkeeping (Sec. 2.5), trapezoid rule over the step
    const double wa = S.W0 + 0.5 * H.dt * (S.y1 * S.Ec + vn * Ee);
    const double wr = S.W1 + 0.5 * H.dt * K_LARMOR * (S.a0 * S.a0 + an * an);
    W[2 * gi] = wa;
    W[2 * gi + 1] = wr;
    const int64_t row = out_row(nstep + 1 - n0, out.stride);
    if (row >= 0) put_row(out, row, gi, dn, vn, run_energy(w2, D.ehalf, dn, vn), Ee, wa, wr);
}

// 64 targets a workgroup; its four waves sum the partials of a target in four runs.
__global__ __launch_bounds__(256) void lo_finish_kernel(const DipDev *__restrict__ dev, const int32_t *__restrict__ tgt,
                                                        const int32_t *__restrict__ tgt_lo,
                                                        const int32_t *__restrict__ tgt_n,
                                                        const int64_t *__restrict__ ring_base, int n_tgt, double *ring,
                                                        double *Ecur, double *W, const int64_t *__restrict__ step_ctr,
                                                        int kstep, int ring_depth, double dt, double max_vel, int chunk,
                                                        RunOut out, const double *__restrict__ part,
                                                        uint32_t *__restrict__ d_err)
{
    __shared__ double sums[2][256];
    const int tid = threadIdx.x, b = blockIdx.x * 64 + (tid & 63), run = tid >> 6;
    const int bb = min(b, n_tgt - 1);
    const int gi = tgt[bb], i0 = tgt_lo[bb], n = tgt_n[bb];
    double Em = 0.0, Ee = 0.0;
    const int splits = (n + chunk - 1) / chunk;
#pragma unroll 4
    for (int s = run; s < splits; s += 4) {
        const double *p = part + (int64_t)s * 2 * n_tgt + bb;
        Em += p[0];
        Ee += p[n_tgt];
    }
    sums[0][tid] = Em;
    sums[1][tid] = Ee;
    const int64_t nstep = *step_ctr + kstep, n0 = step_ctr[1];
    const Hist H{ring + ring_base[bb], n, ring_depth - 1, dt, 1.0 / dt};
    const TargetState S = target_state(H, gi, gi - i0, Ecur, W, nstep);
    __syncthreads();
    if (run != 0 || b >= n_tgt) return;
    for (int r = 1; r < 4; ++r) {
        Em += sums[0][64 * r + tid];
        Ee += sums[1][64 * r + tid];
    }
    uint32_t err = 0u;
    finish_target(dev[gi], S, gi, gi - i0, H, ring + ring_base[b], Ecur, W, nstep, n0, Em, Ee, max_vel, out, err);
    if (err) atomicOr(d_err, err);
}

__global__ void step_advance_kernel(int64_t *step_ctr, int64_t delta)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) *step_ctr += delta;
}

// The run's first step: 0, or the step count of the run state it resumes.
__global__ void step_start_kernel(int64_t *step_ctr, const double *resume)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        const int64_t n0 = resume ? (int64_t)resume[0] : 0;
        step_ctr[0] = n0;
        step_ctr[1] = n0;
    }
}

// A resumed run: the header check and output row 0 of every dipole from the
// state (d, d_dot at the state's step, E_d and the energy sums).
__global__ void state_rows_kernel(const DipDev *__restrict__ dev, const int32_t *__restrict__ off, int n_inst,
                                  const double *__restrict__ state, int ring, RunOut out,
                                  uint32_t *__restrict__ d_err)
{
    const int gi = blockIdx.x * blockDim.x + threadIdx.x;
    if (gi == 0 && !(state[1] == (double)ring && state[2] == (double)out.n_dip)) atomicOr(d_err, ERR_STATE);
    if (gi >= out.n_dip) return;
    const int inst = instance_of(off, n_inst, gi);
    const int a0 = off[inst], n = off[inst + 1] - a0;
    const int64_t n0 = (int64_t)state[0];
    const double *h = state + state_ring_off(a0, ring) + ((int64_t)(n0 & (ring - 1)) * n + (gi - a0)) * 3;
    const DipDev &D = dev[gi];
    const int64_t ow = state_w_off(out.n_dip, ring);
    put_row(out, 0, gi, h[0], h[1], run_energy(D.omega0 * D.omega0, D.ehalf, h[0], h[1]),
            state[state_ecur_off(out.n_dip, ring) + gi], state[ow + 2 * gi], state[ow + 2 * gi + 1]);
}

__global__ void state_header_kernel(double *state, int ring, int n_dip, int64_t steps, int resume)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        const int64_t n0 = resume ? (int64_t)state[0] : 0;
        state[0] = (double)(n0 + steps);
        state[1] = (double)ring;
        state[2] = (double)n_dip;
        state[3] = 0.0;
    }
}

hipError_t launch_state_rows(const DipDev *d_dev, const int32_t *d_off, int n_inst, const double *d_state, int ring,
                             const RunOut &out, uint32_t *d_err, hipStream_t s)
{
    hipLaunchKernelGGL(state_rows_kernel, dim3((out.n_dip + 255) / 256), dim3(256), 0, s, d_dev, d_off, n_inst,
                       d_state, ring, out, d_err);
    return hipGetLastError();
}

hipError_t launch_state_header(double *d_state, int ring, int n_dip, int64_t steps, bool resume, hipStream_t s)
{
    hipLaunchKernelGGL(state_header_kernel, dim3(1), dim3(1), 0, s, d_state, ring, n_dip, steps, resume ? 1 : 0);
    return hipGetLastError();
}

static size_t tile_lds_bytes(int rows, int tile)
{
    return std::max(sizeof(double) * (3 * (size_t)rows * tile + 8), sizeof(double) * 512);
}

// Window rows and tile for light times of up to `steps` steps, or tile = 0 where no tile of
// at least 4 sources fits a third of a CU's LDS (light times beyond 550 steps).
void tile_shape(double steps, int *rows, int *tile)
{
    *tile = 0;
    *rows = 0;
    if (!(steps < 1e6)) return;
    *rows = ((int)std::ceil(steps) + 3) | 1;
    for (int t = 16; t >= 4; t /= 2)
        if (tile_lds_bytes(*rows, t) <= 53 * 1024) {
            *tile = t;
            return;
        }
}
int tile_targets() { return TILE_TARGETS; }

// Calls fn(std::integral_constant<bool, a>, std::integral_constant<bool, b>).
template <typename Fn> static void with_flags(bool a, bool b, Fn &&fn)
{
    if (a) {
        if (b) fn(std::true_type{}, std::true_type{});
        else fn(std::true_type{}, std::false_type{});
    } else {
        if (b) fn(std::false_type{}, std::true_type{});
        else fn(std::false_type{}, std::false_type{});
    }
}

hipError_t launch_dipole_steps(const DipDev *d_dev, const int32_t *d_tgt, const int32_t *d_tgt_lo, const int32_t *d_tgt_n,
                               const int64_t *d_ring_base, int n_tgt, double *d_ring, double *d_Ecur, double *d_W,
                               int64_t *d_step, int ring, int64_t steps, double dt, double max_vel, int max_iter,
                               const RunOut &out, bool moving, bool mixed, const double *d_resume, uint32_t *d_err,
                               int graph_chunk, const TilePlan &tiles, hipStream_t s, hipStream_t cap,
                               hipGraph_t *graph_out, hipGraphExec_t *exec_out)
{
    constexpr int B = 256;
    if (n_tgt <= 0) return hipSuccess;
    const dim3 grid((unsigned)n_tgt), block(B);
    // at most one workgroup per SIMD (256 CUs x 4): a latency-bound launch
    const StepPlan plan = n_tgt > 1024 ? MANY : n_tgt <= 512 ? FEW : 2 * (tiles.max_n - 1) <= B ? SOME : SOME_LARGE;
    const double *soa = dip_soa(const_cast<DipDev *>(d_dev), out.n_dip);
    auto step = [&](hipStream_t q, int k, int init) {
        if (tiles.n_units > 0 && !init) {
            hipLaunchKernelGGL(mixed ? lo_tile_kernel<true> : lo_tile_kernel<false>, dim3((unsigned)tiles.n_units), block,
                               tile_lds_bytes(tiles.rows, tiles.tile), q, d_dev, tiles.units, d_ring_base, n_tgt, d_ring,
                               tiles.part, d_step, k, ring, dt, tiles.rows, tiles.tile, tiles.chunk, max_iter, out.n_dip,
                               soa, d_err);
            hipLaunchKernelGGL(lo_finish_kernel, dim3((unsigned)((n_tgt + 63) / 64)), block, 0, q, d_dev, d_tgt,
                               d_tgt_lo, d_tgt_n, d_ring_base, n_tgt, d_ring, d_Ecur, d_W, d_step, k, ring, dt, max_vel,
                               tiles.chunk, out, tiles.part, d_err);
            return;
        }
        if (tiles.per_wave && !init) {
            const dim3 g4((unsigned)((n_tgt + 3) / 4));
            if (mixed)
                hipLaunchKernelGGL(lo_wave_kernel<true>, g4, block, 0, q, d_dev, d_tgt, d_tgt_lo, d_tgt_n, d_ring_base,
                                   n_tgt, d_ring, d_Ecur, d_W, d_step, k, ring, dt, max_vel, max_iter, out, soa, d_err);
            else
                hipLaunchKernelGGL(lo_wave_kernel<false>, g4, block, 0, q, d_dev, d_tgt, d_tgt_lo, d_tgt_n,
                                   d_ring_base, n_tgt, d_ring, d_Ecur, d_W, d_step, k, ring, dt, max_vel, max_iter, out,
                                   soa, d_err);
            return;
        }
        with_flags(moving, mixed, [&](auto mv, auto mx) {
            constexpr bool MV = decltype(mv)::value, MX = decltype(mx)::value;
            // (the kernels for moving origins have one budget)
            auto kernel = plan == MANY                 ? lo_step_kernel<B, MV, MX, MANY>
                          : plan == FEW || MV          ? lo_step_kernel<B, MV, MX, FEW>
                          : plan == SOME               ? lo_step_kernel<B, MV, MX, MV ? FEW : SOME>
                                                       : lo_step_kernel<B, MV, MX, MV ? FEW : SOME_LARGE>;
            hipLaunchKernelGGL(kernel, grid, block, 0, q, d_dev, d_tgt, d_tgt_lo, d_tgt_n, d_ring_base, d_ring, d_Ecur,
                               d_W, d_step, k, ring, dt, max_vel, max_iter, init, out, soa, d_err);
        });
    };
    hipLaunchKernelGGL(step_start_kernel, dim3(1), dim3(1), 0, s, d_step, d_resume);
    if (!d_resume) step(s, 0, 1);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || steps == 0) return e;
    // a chunk of steps is captured once into a graph and replayed: launch k of
    // a chunk advances step base + k, and the base (on the device) moves by the
    // chunk at its end, so every replay continues where the last ended
    auto enqueue = [&](hipStream_t q, int64_t count) {
        for (int64_t k = 0; k < count; ++k) step(q, (int)k, 0);
        hipLaunchKernelGGL(step_advance_kernel, dim3(1), dim3(1), 0, q, d_step, count);
    };
    const int64_t chunk = graph_chunk > 0 ? graph_chunk : 0;
    if (chunk == 0 || steps < chunk || !cap) {
        enqueue(s, steps);
        return hipGetLastError();
    }
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    e = hipStreamBeginCapture(cap, hipStreamCaptureModeThreadLocal);
    if (e == hipSuccess) {
        enqueue(cap, chunk);
        e = hipStreamEndCapture(cap, &graph);
    }
    if (e == hipSuccess) e = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
    const int64_t reps = steps / chunk;
    for (int64_t r = 0; r < reps && e == hipSuccess; ++r) e = hipGraphLaunch(exec, s);
    if (e == hipSuccess && steps > reps * chunk) {
        enqueue(s, steps - reps * chunk);
        e = hipGetLastError();
    }
    // handed to the caller, which releases them once the stream has passed them
    *graph_out = graph;
    *exec_out = exec;
    return e;
}

int ring_lds_bytes(int n, int ring)
{
    return (int)(sizeof(DipLds) * n + sizeof(double) * 12 * n + sizeof(double) * 3 * (size_t)ring * n);
}

template <int BLOCK>
static hipError_t launch_lo(bool moving, bool mixed, dim3 grid, size_t shmem, hipStream_t s, const DipDev *d_dev,
                            const int32_t *d_off, const int32_t *d_list, int ring, int64_t steps, double dt,
                            double max_vel, int max_iter, const RunOut &out, double *d_state, bool resume,
                            uint32_t *d_err)
{
    with_flags(moving, mixed, [&](auto mv, auto mx) {
        hipLaunchKernelGGL((lo_instances_kernel<BLOCK, decltype(mv)::value, decltype(mx)::value>), grid, dim3(BLOCK),
                           shmem, s, d_dev, d_off, d_list, ring, steps, dt, max_vel, max_iter, out, d_state,
                           resume ? 1 : 0, d_err);
    });
    return hipGetLastError();
}

int dipole_kind_max_n(int kind) { return kind == 0 ? SMALL_MAX_N : kind == 1 ? GROUP8_MAX_N : GROUP_MAX_N; }

hipError_t launch_dipole_instances(const DipDev *d_dev, const int32_t *d_off, const int32_t *d_list, int n_list,
                                   int min_n, int max_n, int ring, int64_t steps, double dt, double max_vel, int max_iter,
                                   const RunOut &out, bool moving, bool mixed, double *d_state, bool resume,
                                   uint32_t *d_err, hipStream_t s)
{
    if (n_list <= 0) return hipSuccess;
    const size_t shmem = (size_t)ring_lds_bytes(max_n, ring);
    const dim3 grid((unsigned)n_list);
    // more than the default 64 KB of dynamic LDS is asked for per kernel
    auto roomy = [&](auto kernel) {
        return shmem <= 64 * 1024 ? hipSuccess
                                  : hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                                        (int)shmem);
    };
    hipError_t e = hipSuccess;
    // Where instances of 10 and more (FP64: up to 13), or of 5 alone, are many, the SIMDs are full
    // whichever kernel holds them, and the general one issues less for them.  us per step, FP64
    // (mixed), by lo_group_kernel / lo_instances_kernel: 12 dipoles x 1,024 5.7 / 6.2 (5.6 / 5.6),
    // x 2,048 11.4 / 10.5 (11.1 / 9.6), x 8,192 45 / 39 (44 / 36); 15 x 4,096 22.7 / 25.2 (23.9 /
    // 19.1); 5 x 2,048 2.5 / 2.7 (2.6 / 2.0), x 4,096 4.9 / 4.7 (5.0 / 3.6); 6 x 8,192 9.2 / 10.8
    // (9.7 / 9.6).  (Its histories are at most 64 KB.)
    const bool crowded = shmem <= 64 * 1024 &&
                         ((max_n > GROUP8_MAX_N && max_n <= (mixed ? GROUP_MAX_N : 13) && n_list >= 1536) ||
                          (max_n == SMALL_MAX_N + 1 && n_list >= 3072));
    if (!moving && min_n > SMALL_MAX_N && max_n <= GROUP_MAX_N && !crowded) {
        const dim3 block((unsigned)group_threads(max_n));
        with_flags(mixed, group_lg(max_n) == 3, [&](auto mx, auto eight) {
            auto kernel = lo_group_kernel<decltype(mx)::value, decltype(eight)::value ? 3 : 4>;
            if ((e = roomy(kernel)) != hipSuccess) return;
            hipLaunchKernelGGL(kernel, grid, block, shmem, s, d_dev, d_off, d_list, ring, steps, dt, max_vel, max_iter,
                               out, d_state, resume ? 1 : 0, d_err);
        });
        return e != hipSuccess ? e : hipGetLastError();
    }
    if (!moving && max_n <= SMALL_MAX_N) {
        auto kernel = mixed ? lo_small_kernel<true> : lo_small_kernel<false>;
        if ((e = roomy(kernel)) != hipSuccess) return e;
        hipLaunchKernelGGL(kernel, grid, dim3(64), shmem, s, d_dev, d_off, d_list, ring, steps, dt, max_vel, max_iter,
                           out, d_state, resume ? 1 : 0, d_err);
        return hipGetLastError();
    }
    if (max_n <= 8)
        return launch_lo<64>(moving, mixed, grid, shmem, s, d_dev, d_off, d_list, ring, steps, dt, max_vel, max_iter,
                             out, d_state, resume, d_err);
    return launch_lo<256>(moving, mixed, grid, shmem, s, d_dev, d_off, d_list, ring, steps, dt, max_vel, max_iter, out,
                          d_state, resume, d_err);
}

}  // namespace lw
