// lw_adjoint.hip -- vector-Jacobian product of the grid fields with respect to
// the trajectory parameters of every charge (FP64).
//
// For one (point x, time t, charge) the outputs O = (Phi, A, E, B) depend on the
// retarded separation R = x - r(t'), velocity v(t') and acceleration a(t') and
// on q, with t' = t - tau and tau the root of c tau = |x - r(t - tau)| (Eq.
// (ret_t)).  For a parameter theta of the trajectory,
//   dR = -r_theta dtheta + v dtau,  dv = v_theta dtheta - a dtau,
//   da = a_theta dtheta - j dtau   (j = da/dt', the jerk),
// and differentiating the retarded-time equation (implicit function theorem)
//   dtau = -(n . r_theta) / (c kappa) dtheta,  c kappa = c - n . v.
// With Rb, vb, ab the cotangents of R, v, a (the reverse of the Lienard-Wiechert
// evaluator) and s = Rb.v - vb.a - ab.j, the cotangent of the trajectory
// position is rb = -Rb - s n / (c kappa), and the gradient of a parameter is
// rb . r_theta + vb . v_theta + ab . a_theta.  Sums over points and times are
// per-wave partials reduced in a fixed order (bitwise reproducible).
#include <math.h>

#include <algorithm>

#include "lw_device.hpp"
#include "lw_internal.hpp"

namespace lw {

// Parameters of a gradient row (q, c0, amp, omega, phase, accel, v), and the sums kept
// per charge: a family has at most three parameters besides q and c0, so eight sums
// hold any family's (amp, omega, phase; accel; or v from P_OWN on).
enum { NP = 11, NS = 8 };
enum { P_Q = 0, P_C0 = 1, P_OWN = 4, P_AMP = 4, P_OMEGA = 5, P_PHASE = 6, P_ACCEL = 4, P_V = 4 };
// Sum that parameter k of a charge of family `kind` is in, or -1.
__device__ __forceinline__ int sum_of(int kind, int k)
{
    if (k < 4) return k;
    if (kind == K_CIRCULAR || kind == K_LINEAR_OSC) return k < 7 ? k : -1;
    if (kind == K_ACCEL) return k == 7 ? P_ACCEL : -1;
    if (kind == K_UNIFORM_VELOCITY) return k >= 8 ? k - 4 : -1;
    return -1;
}
// Waves per workgroup of the VJP kernel (256 lanes): each writes its own partials.
constexpr int WAVES = 4;

// Gradient of one (point, time, charge) contribution of a uniformly moving or
// stationary charge, added into g[NS] (a = 0, so the jerk and the acceleration's
// cotangent drop out).  EONLY: only E has a cotangent (lw_terms_vjp<true>).
template <bool EONLY>
__device__ __forceinline__ void drift_grad(const SrcRec &S, const Kin &k, int field_kind, const double ob[10],
                                           double g[NS])
{
    double Rb[3], vb[3], ab[3], n[3], kqb, kappa;
    lw_terms_vjp<EONLY, true>(k, S.kq, field_kind, ob, Rb, vb, ab, kqb, n, kappa);
    double sres = 0.0;
    for (int i = 0; i < 3; ++i) sres += Rb[i] * k.v[i];
    const double fac = sres * recip<double>(C_LIGHT - (n[0] * k.v[0] + n[1] * k.v[1] + n[2] * k.v[2]));
    double rb[3];
    for (int i = 0; i < 3; ++i) rb[i] = -Rb[i] - fac * n[i];
    g[P_Q] += kqb * K_COUL;
    for (int i = 0; i < 3; ++i) g[P_C0 + i] += rb[i];
    if (S.kind == K_UNIFORM_VELOCITY)
        for (int i = 0; i < 3; ++i) g[P_V + i] += rb[i] * k.tp + vb[i];
}

// The scalar part of the field's reverse, shared by the families below: with the forward
// scalars of lw_terms (b, d: beta and beta_dot; nd = n.d, bb = |b|^2) and the
// contractions yu = Et.u, yd = Et.d of E's cotangent (B's included), phi's direct
// cotangent pb0 (Phi and A), it returns the multipliers
//   ub = cu_f Et (cotangent of u), dbar = -cd_f Et + ndb n,
//   bbar = -ub + 2 bbb b + nbb n (+ A's), nbar = ub + ndb d + nbb b (+ B's),
// and iDb, the cotangent of 1/|R| but for n's, and kqb.
struct FieldBar {
    double cu_f, cd_f, ndb, nbb, bbb, iDb, kqb;
};
struct FieldFwd {
    double iD, ik, phi, f, cu, cd;
};
__device__ __forceinline__ FieldFwd field_fwd(double kq, double iD, double kappa, double nd, double omb, int field_kind)
{
    FieldFwd F;
    const bool coul = field_kind != F_RADIATION, rad = field_kind != F_COULOMB;
    F.iD = iD;
    F.ik = recip<double>(kappa);
    F.phi = kq * iD * F.ik;
    F.f = F.phi * F.ik * F.ik;
    F.cu = (coul ? omb * iD : 0.0) + (rad ? nd * INV_C : 0.0);
    F.cd = rad ? kappa * INV_C : 0.0;
    return F;
}
__device__ __forceinline__ FieldBar field_bar(const FieldFwd &F, double kq, double omb, double yu, double yd, double pb0,
                                              int field_kind)
{
    FieldBar B;
    const bool coul = field_kind != F_RADIATION, rad = field_kind != F_COULOMB;
    const double fb = yu * F.cu - yd * F.cd;                // E = f (u cu - d cd)
    const double cub = F.f * yu, cdb = -F.f * yd;
    B.cu_f = F.f * F.cu;
    B.cd_f = F.f * F.cd;
    const double phib = pb0 + fb * F.ik * F.ik;
    const double ikb = fb * 2.0 * F.phi * F.ik + phib * (kq * F.iD);
    const double kqDb = phib * F.ik;
    B.bbb = coul ? -cub * F.iD : 0.0;
    B.ndb = rad ? cub * INV_C : 0.0;
    B.iDb = (coul ? cub * omb : 0.0) + kqDb * kq;
    B.kqb = kqDb * F.iD;
    B.nbb = ikb * F.ik * F.ik - (rad ? cdb * INV_C : 0.0);  // -(cotangent of kappa)
    return B;
}

// A circular orbit's contribution.  In the frame that turns with the charge, (radial,
// tangential, axis), beta = (0, beta, 0) and beta_dot = (-aw, 0, 0) are constants and the
// trajectory's derivatives are along single axes, so the reverse works on scalars:
// only the cotangents are turned into the frame (13 operations a vector), and the
// centre's gradient is kept in the orbit's fixed frame until the wave's sum.  w1, w2,
// w3: x - c0 along e1, e2, e3; ob in the same axes.  256^2 x 32 x 64 detector, E rows:
// 2.40 -> 1.32 ms per call together with the folded sums below (2.15 ms with the
// forward solves of this form alone).
template <bool EONLY>
__device__ __forceinline__ void circular_grad(const SrcRec &S, const Kin &k, double w1, double w2, double w3,
                                              const double ob[10], int field_kind, double mask_r2, bool fin,
                                              double g[NS])
{
    const double c = k.cph, s = k.sph, A = S.amp, om = S.omega, beta = A * S.koc, aw = beta * om;
    const double Xr = w1 * c + w2 * s - A, Xt = w2 * c - w1 * s;
    const double D2 = Xr * Xr + Xt * Xt + w3 * w3;
    if (!fin || !(D2 >= mask_r2) || D2 == 0.0) return;
    double D, iD;
    root_rsqrt<true>(D2, D, iD);
    iD = fma(iD, fma(-D, iD, 1.0), iD);
    const double nr = Xr * iD, nt = Xt * iD, n3 = w3 * iD;
    const double omb = fma(-beta, beta, 1.0);
    const FieldFwd F = field_fwd(S.kq, iD, 1.0 - beta * nt, -aw * nr, omb, field_kind);
    const double ut = nt - beta;
    // cotangents in the turning frame
    double yr = ob[4] * c + ob[5] * s, yt = ob[5] * c - ob[4] * s, y3 = ob[6];
    double pb0 = 0.0, mr = 0.0, mt = 0.0, m3 = 0.0, Ar = 0.0, At = 0.0;
    if constexpr (!EONLY) {
        Ar = ob[1] * c + ob[2] * s;
        At = ob[2] * c - ob[1] * s;
        const double Br = ob[7] * c + ob[8] * s, Bt = ob[8] * c - ob[7] * s, B3 = ob[9];
        // B = m x E, m = n / c; A = phi b / c
        const double Er = F.f * (nr * F.cu + aw * F.cd), Et = F.f * (ut * F.cu), E3 = F.f * (n3 * F.cu);
        mr = (Et * B3 - E3 * Bt) * INV_C;
        mt = (E3 * Br - Er * B3) * INV_C;
        m3 = (Er * Bt - Et * Br) * INV_C;
        const double xr = Bt * n3 - B3 * nt, xt = B3 * nr - Br * n3, x3 = Br * nt - Bt * nr;
        yr = yr + INV_C * xr;
        yt = yt + INV_C * xt;
        y3 = y3 + INV_C * x3;
        const double ba = At * beta;
        pb0 = ob[0] + ba * INV_C;
    }
    const double yu = yr * nr + yt * ut + y3 * n3;
    const FieldBar B = field_bar(F, S.kq, omb, yu, -aw * yr, pb0, field_kind);
    const double pc = EONLY ? 0.0 : F.phi * INV_C;
    // cotangents of n, beta, beta_dot
    double Nr = B.cu_f * yr - aw * B.ndb, Nt = B.cu_f * yt + B.nbb * beta, N3 = B.cu_f * y3;
    double br = B.nbb * nr - B.cu_f * yr, bt = B.nbb * nt + (2.0 * B.bbb * beta - B.cu_f * yt);
    if constexpr (!EONLY) {
        Nr = Nr + mr;
        Nt = Nt + mt;
        N3 = N3 + m3;
        const double ar = pc * Ar, at = pc * At;
        br = br + ar;
        bt = bt + at;
    }
    const double dr = B.ndb * nr - B.cd_f * yr, dt = B.ndb * nt - B.cd_f * yt;
    // R = D n
    const double sn = -(B.iDb * iD + (Nr * nr + Nt * nt + N3 * n3)) * iD;
    const double Rr = Nr * iD + sn * nr, Rt = Nt * iD + sn * nt, R3 = N3 * iD + sn * n3;
    // tau: s = Rb.v - vb.a - ab.j with v = A om t, a = -A om^2 r, j = -om^2 v
    const double fac = beta * (Rt + S.koc * br + S.koc * om * dt) * F.ik;
    const double Pr = -Rr - fac * nr, Pt = -Rt - fac * nt;
    g[P_Q] += B.kqb * K_COUL;
    g[P_C0] += Pr * c - Pt * s;
    g[P_C0 + 1] += Pr * s + Pt * c;
    g[P_C0 + 2] += -R3 - fac * n3;
    const double koc = S.koc;
    const double gphi = A * (Pt - koc * br - koc * om * dt);
    g[P_AMP] += Pr + koc * bt - koc * om * dr;
    g[P_PHASE] += gphi;
    g[P_OMEGA] += k.tp * gphi + A * INV_C * bt - 2.0 * A * koc * dr;
}

// A charge that moves along e1 (linear oscillation, acceleration from rest): beta =
// b e1 and beta_dot = d e1, so beta and beta_dot enter through their scalars and every
// vector is a combination of n, e1 and E's cotangent.  jc: the jerk over c along e1.
// Returns the cotangents of the charge's position, velocity / c and acceleration / c
// along e1 (for the family's own parameters); false where the pair is left out.
template <bool EONLY>
__device__ __forceinline__ bool axis_grad(const SrcRec &S, const double R[3], double b, double d, double jc,
                                          const double ob[10], int field_kind, double mask_r2, bool fin, double g[NS],
                                          double &r1, double &b1, double &d1)
{
    const double *e = S.e1;
    const double D2 = R[0] * R[0] + R[1] * R[1] + R[2] * R[2];
    if (!fin || !(D2 >= mask_r2) || D2 == 0.0) return false;
    double D, iD;
    root_rsqrt<true>(D2, D, iD);
    iD = fma(iD, fma(-D, iD, 1.0), iD);
    const double n[3] = {R[0] * iD, R[1] * iD, R[2] * iD};
    const double n1 = n[0] * e[0] + n[1] * e[1] + n[2] * e[2];
    const double omb = fma(-b, b, 1.0);
    const FieldFwd F = field_fwd(S.kq, iD, 1.0 - b * n1, d * n1, omb, field_kind);
    double y[3] = {ob[4], ob[5], ob[6]};
    double pb0 = 0.0, m[3] = {0.0, 0.0, 0.0}, A1 = 0.0;
    if constexpr (!EONLY) {
        const double *Bb = ob + 7;
        const double ge = b * F.cu + d * F.cd;              // E = f (n cu - ge e1)
        const double E[3] = {F.f * (n[0] * F.cu - ge * e[0]), F.f * (n[1] * F.cu - ge * e[1]),
                             F.f * (n[2] * F.cu - ge * e[2])};
        m[0] = (E[1] * Bb[2] - E[2] * Bb[1]) * INV_C;
        m[1] = (E[2] * Bb[0] - E[0] * Bb[2]) * INV_C;
        m[2] = (E[0] * Bb[1] - E[1] * Bb[0]) * INV_C;
        const double x0 = Bb[1] * n[2] - Bb[2] * n[1], x1 = Bb[2] * n[0] - Bb[0] * n[2], x2 = Bb[0] * n[1] - Bb[1] * n[0];
        y[0] = y[0] + INV_C * x0;
        y[1] = y[1] + INV_C * x1;
        y[2] = y[2] + INV_C * x2;
        A1 = ob[1] * e[0] + ob[2] * e[1] + ob[3] * e[2];
        const double ba = A1 * b;
        pb0 = ob[0] + ba * INV_C;
    }
    const double y1 = y[0] * e[0] + y[1] * e[1] + y[2] * e[2];
    const double yn = y[0] * n[0] + y[1] * n[1] + y[2] * n[2];
    const FieldBar B = field_bar(F, S.kq, omb, yn - b * y1, d * y1, pb0, field_kind);
    // nbar = cu_f y + ke e1 (+ m)
    const double ke = B.ndb * d + B.nbb * b;
    double Nn = B.cu_f * yn + ke * n1, N1 = B.cu_f * y1 + ke;
    b1 = B.nbb * n1 + (2.0 * B.bbb * b - B.cu_f * y1);
    if constexpr (!EONLY) {
        const double mn = m[0] * n[0] + m[1] * n[1] + m[2] * n[2], m1 = m[0] * e[0] + m[1] * e[1] + m[2] * e[2];
        Nn = Nn + mn;
        N1 = N1 + m1;
        const double at = F.phi * INV_C * A1;
        b1 = b1 + at;
    }
    d1 = B.ndb * n1 - B.cd_f * y1;
    const double sn = -(B.iDb * iD + Nn) * iD;
    const double R1 = N1 * iD + sn * n1;                    // cotangent of R along e1
    // tau: s / c = Rb1 b - vb1 d - ab1 j / c, over kappa
    const double fac = (R1 * b - INV_C * (b1 * d + d1 * jc)) * F.ik;
    const double kn = -sn - fac, ky = -B.cu_f * iD, k1 = -ke * iD;
    r1 = -R1 - fac * n1;
    g[P_Q] += B.kqb * K_COUL;
    for (int i = 0; i < 3; ++i) {
        double t = ky * y[i] + (kn * n[i] + k1 * e[i]);
        if constexpr (!EONLY) {
            const double mi = m[i] * iD;
            t = t - mi;
        }
        g[P_C0 + i] += t;
    }
    return true;
}

// The contributions of one charge of family KIND at point x over nt_here times
// (records Rc[ti * nch], cotangent rows cot[(ti * nrows + row) * npts + p]),
// added into g[NS]: per time the retarded kinematics (the FP64 correction
// solves, their fallback on a rebuilt geometry, so the geometry here needs no
// bracket) and their reverse.  The geometry is rebuilt per time: keeping it live
// across the times would take this kernel from 3 to 2 waves per SIMD.  EONLY:
// the cotangent holds the three E rows alone (outputs E), which are all it reads.
template <int KIND, bool EONLY, typename G>
__device__ __forceinline__ void charge_grad(const SrcRec *__restrict__ Rc, int nch, int nt_here, const double x[3],
                                            int64_t p, int64_t npts, int nrows, const int row[10], int field_kind,
                                            int max_iter, double tol_rel, double mask_r, const G *__restrict__ cot,
                                            double g[NS])
{
    const double e3[3] = {Rc->e1[1] * Rc->e2[2] - Rc->e1[2] * Rc->e2[1], Rc->e1[2] * Rc->e2[0] - Rc->e1[0] * Rc->e2[2],
                          Rc->e1[0] * Rc->e2[1] - Rc->e1[1] * Rc->e2[0]};
    for (int ti = 0; ti < nt_here; ++ti) {
        const SrcRec &S = Rc[(int64_t)ti * nch];
        double ob[10];
        bool fin = true;
#pragma unroll
        for (int j = 0; j < 10; ++j) {
            if (EONLY) {
                ob[j] = (j >= 4 && j < 7) ? (double)cot[((int64_t)ti * 3 + (j - 4)) * npts + p] : 0.0;
            } else {
                ob[j] = row[j] >= 0 ? (double)cot[((int64_t)ti * nrows + row[j]) * npts + p] : 0.0;
            }
            fin = fin && isfinite(ob[j]);
        }
        // the cotangent is tested after the solve, which does not depend on it,
        // so that its loads are in flight during the solve
        Geo geo;
        geo_prepare_k<KIND>(S, x, geo);
        Kin k;
        uint32_t flags = 0u;                  // (an unconverged solve is used as it is)
        retarded_kind<true, KIND>(S, geo, x, max_iter, tol_rel, k, flags);
        const double mask_r2 = mask_r * mask_r;
        if constexpr (KIND == K_CIRCULAR) {
            const double *w = geo.w;
            const double w1 = w[0] * S.e1[0] + w[1] * S.e1[1] + w[2] * S.e1[2];
            const double w2 = w[0] * S.e2[0] + w[1] * S.e2[1] + w[2] * S.e2[2];
            const double w3 = w[0] * e3[0] + w[1] * e3[1] + w[2] * e3[2];
            double oc[10];
            oc[0] = ob[0];
            for (int q = EONLY ? 4 : 1; q < (EONLY ? 7 : 10); q += 3) {
                oc[q] = ob[q] * S.e1[0] + ob[q + 1] * S.e1[1] + ob[q + 2] * S.e1[2];
                oc[q + 1] = ob[q] * S.e2[0] + ob[q + 1] * S.e2[1] + ob[q + 2] * S.e2[2];
                oc[q + 2] = ob[q] * e3[0] + ob[q + 1] * e3[1] + ob[q + 2] * e3[2];
            }
            circular_grad<EONLY>(S, k, w1, w2, w3, oc, field_kind, mask_r2, fin, g);
        } else if constexpr (KIND == K_LINEAR_OSC) {
            const double om = S.omega, A = S.amp, c = k.cph, sn = k.sph;
            const double b = -A * S.koc * sn, d = -A * S.koc * om * c;
            const double R[3] = {geo.w[0] - c * S.v[0], geo.w[1] - c * S.v[1], geo.w[2] - c * S.v[2]};
            double r1, b1, d1;
            if (!axis_grad<EONLY>(S, R, b, d, -om * om * b, ob, field_kind, mask_r2, fin, g, r1, b1, d1)) continue;
            const double vb = b1 * INV_C, ab = d1 * INV_C;
            const double gphi = -A * sn * r1 - A * om * c * vb + A * om * om * sn * ab;
            g[P_AMP] += r1 * c - om * sn * vb - om * om * c * ab;
            g[P_PHASE] += gphi;
            g[P_OMEGA] += k.tp * gphi - A * sn * vb - 2.0 * A * om * c * ab;
        } else if constexpr (KIND == K_ACCEL) {
            // (before the start of the motion b = d = 0)
            const bool on = k.tp >= 0.0;
            const double tp = on ? k.tp : 0.0, b = S.accel * tp * INV_C, d = k.tp > 0.0 ? S.accel * INV_C : 0.0;
            double r1, b1, d1;
            if (!axis_grad<EONLY>(S, k.R, b, d, 0.0, ob, field_kind, mask_r2, fin, g, r1, b1, d1)) continue;
            if (on) g[P_ACCEL] += 0.5 * tp * tp * r1 + (tp * b1 + d1) * INV_C;
        } else {
            const double D2 = k.R[0] * k.R[0] + k.R[1] * k.R[1] + k.R[2] * k.R[2];
            if (!fin || !(D2 >= mask_r2) || D2 == 0.0) continue;
            drift_grad<EONLY>(S, k, field_kind, ob, g);
        }
    }
    if constexpr (KIND == K_CIRCULAR) {
        // the centre's gradient from the orbit's frame
        const double a1 = g[P_C0], a2 = g[P_C0 + 1], a3 = g[P_C0 + 2];
        for (int i = 0; i < 3; ++i) g[P_C0 + i] = a1 * Rc->e1[i] + a2 * Rc->e2[i] + a3 * e3[i];
    }
}

// Lanes 0..31 get a's sum with lane + 32, lanes 32..63 b's with lane - 32.
__device__ __forceinline__ double fold32(double a, double b)
{
    lane_swap<32>(a, b);
    return a + b;
}
// Rows 0 and 2 of 16 lanes get a's sums of rows 0 + 1 and 2 + 3, rows 1 and 3 b's.
__device__ __forceinline__ double fold16(double a, double b)
{
    lane_swap<16>(a, b);
    return a + b;
}
// x of the lane that the DPP control names (rotations within a row of 16).
template <int CTRL> __device__ __forceinline__ double turn(double x)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}

template <typename G, bool EONLY>
__global__ __launch_bounds__(256) void fields_vjp_kernel(const SrcRec *__restrict__ recs, int nch,
                                                         const double *__restrict__ pts, int64_t npts, int nt,
                                                         int tchunk, int cchunk, int field_kind, int outputs,
                                                         int nrows, int max_iter, double tol_rel, double mask_r,
                                                         const G *__restrict__ cot, double *__restrict__ partial)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t p = (int64_t)blockIdx.x * 256 + tid;
    const bool live = p < npts;
    double x[3] = {0.0, 0.0, 0.0};
    if (live) {
        x[0] = pts[p];
        x[1] = pts[npts + p];
        x[2] = pts[2 * npts + p];
    }
    const int t0 = blockIdx.y * tchunk;
    const int t1 = min(t0 + tchunk, nt);
    const int64_t blk = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
    // cotangent row of each of the 10 outputs (-1: not requested, cotangent 0)
    int row[10];
    {
        int r = 0;
        row[0] = (outputs & OUT_PHI) ? r++ : -1;
        for (int q = 1; q < 4; ++q) row[q] = (outputs & OUT_A) ? r++ : -1;
        for (int q = 4; q < 7; ++q) row[q] = (outputs & OUT_E) ? r++ : -1;
        for (int q = 7; q < 10; ++q) row[q] = (outputs & OUT_B) ? r++ : -1;
    }
    const int c1 = min(nch, ((int)blockIdx.z + 1) * cchunk);
    for (int c = (int)blockIdx.z * cchunk; c < c1; ++c) {
        double g[NS];
#pragma unroll
        for (int j = 0; j < NS; ++j) g[j] = 0.0;
        if (live) {
            // every time's record of a charge carries the charge's family, so
            // the solver is chosen once per charge
            const SrcRec *Rc = recs + (int64_t)t0 * nch + c;
            switch (Rc->kind) {
            case K_CIRCULAR:
                charge_grad<K_CIRCULAR, EONLY>(Rc, nch, t1 - t0, x, p, npts, nrows, row, field_kind, max_iter, tol_rel,
                                        mask_r, cot + (int64_t)t0 * nrows * npts, g);
                break;
            case K_LINEAR_OSC:
                charge_grad<K_LINEAR_OSC, EONLY>(Rc, nch, t1 - t0, x, p, npts, nrows, row, field_kind, max_iter, tol_rel,
                                          mask_r, cot + (int64_t)t0 * nrows * npts, g);
                break;
            case K_ACCEL:
                charge_grad<K_ACCEL, EONLY>(Rc, nch, t1 - t0, x, p, npts, nrows, row, field_kind, max_iter, tol_rel,
                                     mask_r, cot + (int64_t)t0 * nrows * npts, g);
                break;
            case K_UNIFORM_VELOCITY:
                charge_grad<K_UNIFORM_VELOCITY, EONLY>(Rc, nch, t1 - t0, x, p, npts, nrows, row, field_kind, max_iter,
                                                tol_rel, mask_r, cot + (int64_t)t0 * nrows * npts, g);
                break;
            default:
                charge_grad<K_STATIONARY, EONLY>(Rc, nch, t1 - t0, x, p, npts, nrows, row, field_kind, max_iter, tol_rel,
                                          mask_r, cot + (int64_t)t0 * nrows * npts, g);
                break;
            }
        }
        // the wave's sums: two values fold into one register across the halves, two of
        // those across the rows of 16 (each half, row its own value), then turns within
        // the rows; 42 VALU instructions, where a shuffle tree for each of 11
        // parameters took 132 LDS permutes and 66 additions.  One partial per (wave,
        // charge), no barrier
        double t[4], u[2];
        for (int j = 0; j < 4; ++j) t[j] = fold32(g[2 * j], g[2 * j + 1]);
        for (int j = 0; j < 2; ++j) {
            u[j] = fold16(t[2 * j], t[2 * j + 1]);
            u[j] += turn<0x128>(u[j]);
            u[j] += turn<0x124>(u[j]);
            u[j] += turn<0x122>(u[j]);
            u[j] += turn<0x121>(u[j]);
        }
        // row r of u[j] holds sum 4 j + (0, 2, 1, 3)[r]
        const int r = lane >> 4, in = lane & 15, j0 = ((r & 1) << 1) | (r >> 1);
        if (in < 2) partial[((blk * WAVES + wave) * nch + c) * NS + 4 * in + j0] = in ? u[1] : u[0];
    }
}

// One workgroup per charge: 128 partials' eight sums at a time, then over the rows of
// lanes, all in a fixed order (bitwise reproducible), and the sums' places among the
// parameters.
__global__ __launch_bounds__(1024) void vjp_reduce_kernel(const SrcRec *__restrict__ recs,
                                                          const double *__restrict__ partial, int64_t nblk, int nch,
                                                          double *__restrict__ grad)
{
    __shared__ double red[1024];
    const int c = blockIdx.x, tid = threadIdx.x, sum = tid & 7;
    double s = 0.0;
    for (int64_t b = tid >> 3; b < nblk; b += 128) s += partial[(b * nch + c) * NS + sum];
    red[tid] = s;
    __syncthreads();
    for (int off = 512; off >= 8; off >>= 1) {
        if (tid < off) red[tid] += red[tid + off];
        __syncthreads();
    }
    if (tid < NP) {
        const int q = sum_of(recs[c].kind, tid);
        grad[(int64_t)c * NP + tid] = q < 0 ? 0.0 : red[q];
    }
}

int vjp_params() { return NP; }

// Times and charges per workgroup.  A charge's sums over the wave cost about as much as
// a fifth of one pair's work, so eight times share them where that leaves at least
// 2,048 workgroups (of 768 resident, so that the last ones do not leave the chip
// idle); fewer points take fewer times, then fewer charges a workgroup, down to one
// of each: 61 x 53 points x 9 times x 16 charges 72 us in 624 workgroups, 256 us in the
// 39 of four times and all charges each.
struct VjpShape {
    int64_t gx;
    int tchunk, cchunk;
};
static VjpShape vjp_shape(int64_t npts, int nt, int nch)
{
    constexpr int64_t want = 2048;
    VjpShape v;
    v.gx = (npts + 255) / 256;
    v.tchunk = 8;
    while (v.tchunk > 1 && v.gx * ((nt + v.tchunk - 1) / v.tchunk) * nch < want) v.tchunk >>= 1;
    const int64_t xy = v.gx * ((nt + v.tchunk - 1) / v.tchunk);
    const int64_t gz = std::min<int64_t>(nch, (want + xy - 1) / xy);
    v.cchunk = (int)((nch + gz - 1) / gz);
    // (grid.y and grid.z hold at most 65,535)
    while ((nt + v.tchunk - 1) / v.tchunk > 65535) v.tchunk <<= 1;
    while ((nch + v.cchunk - 1) / v.cchunk > 65535) ++v.cchunk;
    return v;
}

size_t vjp_partial_doubles(int64_t npts, int nt, int nch)
{
    const VjpShape v = vjp_shape(npts, nt, nch);
    return (size_t)(v.gx * ((nt + v.tchunk - 1) / v.tchunk) * WAVES) * (size_t)nch * NS;
}

template <typename G, bool EONLY>
static void vjp_launch(const VjpShape &v, const dim3 &grid, hipStream_t s, const SrcRec *d_recs, int nch,
                       const double *d_pts, int64_t npts, int nt, const lw_opts &o, double tol_rel, double mask_r,
                       const void *d_cot, double *d_partial)
{
    const int max_iter = o.max_iter > 0 ? o.max_iter : 100;
    hipLaunchKernelGGL((fields_vjp_kernel<G, EONLY>), grid, dim3(256), 0, s, d_recs, nch, d_pts, npts, nt, v.tchunk,
                       v.cchunk, o.field_kind, output_mask(o.outputs), output_rows(o.outputs), max_iter, tol_rel,
                       mask_r, (const G *)d_cot, d_partial);
}

hipError_t launch_fields_vjp(const SrcRec *d_recs, int nch, const double *d_pts, int64_t npts, int nt,
                             const lw_opts &o, double tol_rel, double mask_r, const void *d_cot, double *d_partial,
                             double *d_grad, hipStream_t s)
{
    const VjpShape v = vjp_shape(npts, nt, nch);
    const dim3 grid((unsigned)v.gx, (unsigned)((nt + v.tchunk - 1) / v.tchunk),
                    (unsigned)((nch + v.cchunk - 1) / v.cchunk));
    // a cotangent of E alone (objectives of |E|^2) takes the kernel that reads
    // and reverses only E
    const bool eonly = output_mask(o.outputs) == OUT_E;
    if (o.precision == LW_MIXED) {
        if (eonly) vjp_launch<float, true>(v, grid, s, d_recs, nch, d_pts, npts, nt, o, tol_rel, mask_r, d_cot, d_partial);
        else vjp_launch<float, false>(v, grid, s, d_recs, nch, d_pts, npts, nt, o, tol_rel, mask_r, d_cot, d_partial);
    } else {
        if (eonly) vjp_launch<double, true>(v, grid, s, d_recs, nch, d_pts, npts, nt, o, tol_rel, mask_r, d_cot, d_partial);
        else vjp_launch<double, false>(v, grid, s, d_recs, nch, d_pts, npts, nt, o, tol_rel, mask_r, d_cot, d_partial);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int64_t nblk = (int64_t)grid.x * grid.y * WAVES;      // partial rows, one per wave
    hipLaunchKernelGGL(vjp_reduce_kernel, dim3(nch), dim3(1024), 0, s, d_recs, d_partial, nblk, nch, d_grad);
    return hipGetLastError();
}

}  // namespace lw
