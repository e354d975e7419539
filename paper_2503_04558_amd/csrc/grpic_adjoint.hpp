// grpic_adjoint.hpp -- reverse-mode derivative of one GRPIC particle step
// (arXiv:2503.04558 Sec. 2.2-2.3, App. A): the vector-Jacobian product of
//   (xi, eta, u_r, u_th, u_ph, gathered D^i, B^i) -> (end point, u, deposit)
// needed by the adjoint of K push + deposit steps.
//
// Structure of one step (the forward replay records a tape of it):
//   gather D, B at x^n -> Boris kick at x^n -> geodesic predictor + ncorr
//   trapezoid correctors -> axis reflection -> Esirkepov deposit.
// The reverse sweep runs the same stages backwards, each differentiated by
// hand.  The geodesic right-hand side is Hamiltonian, dx/dt = H_u, du/dt =
// -H_x with H = alpha sqrt(eps + gamma^ij u_i u_j) - beta^r u_r, so its
// vector-Jacobian product with (g_x, g_u) is minus, for x, and plus, for u,
// its own directional derivative along (dx, du) = (-g_u, g_x): one tangent
// carried through the right-hand side's few terms.  (Contracting the r and
// theta derivatives of the 24 metric quantities it is written in took 7,100
// VALU instructions per particle-step for the whole reverse, 1e6 particles x
// 32 steps in 11.6 ms at one wave per SIMD.)
//
// Everything here is plain double arithmetic (host or device), apart from the
// reciprocal and square root below, which take the hardware's estimates on
// the GPU.
#pragma once

#include <math.h>
#include <stdint.h>

#include "grpic_device.hpp"

namespace grpic {
namespace adj {

// 1/x, and sqrt(x) with 1/sqrt(x).  Compiled for the GPU: the particle step's
// refined hardware estimates (a few ulp; the IEEE-rounded division and square
// root take twice the instructions and more registers).  Compiled for the
// host (the same per-particle sweep run on the CPU): the library's.
#if defined(__HIP_DEVICE_COMPILE__)
__device__ inline double inv_(double x) { return rcp(x); }
__device__ inline void sqrt_inv_(double x, double& sq, double& rsq) { sqrt_rsqrt(x, sq, rsq); }
#else
inline double inv_(double x) { return 1.0 / x; }
inline void sqrt_inv_(double x, double& sq, double& rsq) {
    sq = ::sqrt(x);
    rsq = 1.0 / sq;
}
#endif

// Between two stages of a step: neither the compiler nor its scheduler moves
// the next one's loads and arithmetic up across it (the register file is the
// sweep's limit).
__host__ __device__ inline void stage_end() {
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("" : : : "memory");
    __builtin_amdgcn_sched_barrier(0);
#endif
}

constexpr int kMaxCorr = 8;            // predictor-corrector passes the adjoint supports

// Grid and metric constants of a step.
struct Geo {
    double a, M, lnr0, dlnr, dth;
    int nr, nth, guard, pitch;
    double idlnr, idth;                        // 1/dlnr, 1/dth
    double a2, M2, M4a2;                       // a^2, 2 M, 4 M a^2: uniform, so not left to vector registers
    __host__ __device__ uint32_t index(int i, int j) const { return (uint32_t)((i + guard) * pitch + (j + guard)); }
};

// r, sin(theta), cos(theta) of a point: the only transcendental functions the
// metric needs.  SMALL (grids with 2 dlnr and 2 dth <= kSmallArg): all of a
// step's points are reached from its start cell's corner by the particle
// step's Taylor offsets.
struct Trig {
    double r, s, c;
};
struct Corner {
    Trig t;
    int ci, cj;
};
__host__ __device__ inline Trig trig_plain(const Geo& G, double xi, double eta) {
    Trig t;
    t.r = ::exp(G.lnr0 + xi * G.dlnr);
    sincos_theta(eta * G.dth, t.s, t.c);
    return t;
}
template <bool SMALL>
__host__ __device__ inline Corner corner_of(const Geo& G, double xi, double eta) {
    Corner k;
    k.ci = (int)::floor(xi);
    k.cj = (int)::floor(eta);
    k.t = SMALL ? trig_plain(G, (double)k.ci, (double)k.cj) : Trig{0.0, 0.0, 0.0};
    return k;
}
template <bool SMALL>
__host__ __device__ inline Trig trig_at(const Geo& G, const Corner& k, double xi, double eta) {
    if (!SMALL) return trig_plain(G, xi, eta);
    Trig t;
    if (k.t.s >= kPoleSin) {
        t.r = k.t.r * exp_small<false>((xi - (double)k.ci) * G.dlnr);
        double sy, cy;
        sincos_small<false>((eta - (double)k.cj) * G.dth, sy, cy);
        t.s = fma(k.t.s, cy, k.t.c * sy);
        t.c = fma(k.t.c, cy, -(k.t.s * sy));
    } else {
        return trig_plain(G, xi, eta);
    }
    return t;
}

// ---------------------------------------------------------------- RHS
// The terms of the geodesic right-hand side at a point (App. A substituted,
// as in the particle step): with rho^2 = r^2 + a^2 cos^2, T = 2 M r, Q =
// rho^2 + T, beta^r = T / Q, iR = rho^2 / Q = 1 - beta^r, y = u_ph / sin^2,
// W = a u_r + y, Z = a sin^2 u_r + u_ph, P = (r^2 + a^2) u_r + a u_ph,
// x = (u_th^2 + W u_ph + a u_r Z) / rho^2 = u^2 - (1 - beta^r) u_r^2:
//   u^0 = sqrt((eps + x + u_r^2 iR) / iR),  g = 1 / (rho^2 u^0),
//   dr/dt = g P - beta^r (1 + v) with v = u_r / u^0,  dtheta/dt = g u_th,
//   dphi/dt = g W,  du_r/dt = b0 h + r g x,
//   du_th/dt = b1 h - sin cos g (a^2 (x + u_r^2) - y^2),
// b0, b1 the r and theta derivatives of beta^r, h = (u^0 + u_r)(1 + v) / 2.
struct RhsTerms {
    double r, sc, s2, ra2, ir, is2, irho2, iQ, iR, beta, P, y, W, Z, x, E, R, u0, iu0, g, v, h, b0, b1;
};
__host__ __device__ inline RhsTerms rhs_terms(const Geo& G, double eps, const Trig& t, double ur, double ut, double up) {
    RhsTerms m;
    const double a = G.a, a2 = G.a2, r2 = t.r * t.r, T = G.M2 * t.r;
    m.r = t.r;
    m.s2 = t.s * t.s;
    m.sc = t.s * t.c;
    const double rho2 = r2 + a2 * (t.c * t.c), Q = rho2 + T;
    m.ra2 = r2 + a2;
    // 1/sin^2 on its own: near an axis the result hangs on how it is rounded
    m.ir = inv_(t.r);
    m.is2 = inv_(m.s2);
    m.irho2 = inv_(rho2);
    m.iQ = inv_(Q);
    m.beta = T * m.iQ;
    m.iR = rho2 * m.iQ;
    m.R = Q * m.irho2;
    m.P = m.ra2 * ur + a * up;
    m.y = m.is2 * up;
    m.W = a * ur + m.y;
    m.Z = a * m.s2 * ur + up;
    m.x = m.irho2 * (ut * ut + m.W * up + a * ur * m.Z);
    m.E = eps + m.x + ur * ur * m.iR;
    sqrt_inv_(m.E * m.R, m.u0, m.iu0);
    m.g = m.irho2 * m.iu0;
    m.v = ur * m.iu0;
    m.h = 0.5 * (m.u0 + ur) * (1.0 + m.v);
    const double iQ2 = m.iQ * m.iQ;
    m.b0 = G.M2 * (rho2 - 2.0 * r2) * iQ2;
    m.b1 = G.M4a2 * t.r * m.sc * iQ2;
    return m;
}

// Geodesic right-hand side (eq. particle-eom without the Lorentz force) in
// grid units: f = (dxi/dt, deta/dt, dphi/dt, du_r/dt, du_th/dt).
__host__ __device__ inline void rhs(const Geo& G, double eps, const Trig& t, double ur, double ut, double up,
                                    double f[5]) {
    const RhsTerms m = rhs_terms(G, eps, t, ur, ut, up);
    f[0] = (m.g * m.P - m.beta * (1.0 + m.v)) * m.ir * G.idlnr;
    f[1] = m.g * ut * G.idth;
    f[2] = m.g * m.W;
    f[3] = m.b0 * m.h + m.r * m.g * m.x;
    f[4] = m.b1 * m.h - m.sc * m.g * (G.a2 * (m.x + ur * ur) - m.y * m.y);
}

// Cotangent c of f at the point t, (ur, ut, up) -> cotangents of the point
// (added to yb[0..1] = xi, eta and ub[0..2] = u_r, u_th, u_ph): the
// directional derivative (d...; l... of a logarithm) of the terms above along
// (dr, dth) = -(c_3, c_4), (dur, dut, dup) = (c_0 / (r dlnr), c_1 / dth, c_2),
// and the factor 1 / r of f_0.
__host__ __device__ inline void rhs_vjp(const Geo& G, double eps, const Trig& t, double ur, double ut, double up,
                                        const double c[5], double yb[2], double ub[3]) {
    const RhsTerms m = rhs_terms(G, eps, t, ur, ut, up);
    const double a = G.a, a2 = G.a2;
    const double dr = -c[3], dth = -c[4], dur = c[0] * m.ir * G.idlnr, dut = c[1] * G.idth, dup = c[2];
    const double rdr2 = 2.0 * m.r * dr;
    const double ds2 = 2.0 * m.sc * dth, dsc = (1.0 - 2.0 * m.s2) * dth;
    const double drho2 = rdr2 - a2 * ds2, dT = G.M2 * dr;
    const double lrho = m.irho2 * drho2, lQ = m.iQ * (drho2 + dT);
    const double dbeta = m.iQ * dT - m.beta * lQ;
    const double dP = rdr2 * ur + m.ra2 * dur + a * dup;
    const double dy = m.is2 * (dup - m.y * ds2);
    const double dW = a * dur + dy;
    const double dZ = a * (ds2 * ur + m.s2 * dur) + dup;
    const double dx = m.irho2 * (2.0 * ut * dut + dW * up + m.W * dup + a * (dur * m.Z + ur * dZ)) - m.x * lrho;
    const double dE = dx + ur * m.iR * (2.0 * dur + ur * (lrho - lQ));
    const double du0 = 0.5 * m.iu0 * m.R * (dE + m.E * (lQ - lrho));
    const double lg = -(lrho + m.iu0 * du0);
    const double dv = m.iu0 * (dur - m.v * du0);
    const double dh = 0.5 * ((du0 + dur) * (1.0 + m.v) + (m.u0 + ur) * dv);
    const double iQ2 = m.iQ * m.iQ;
    const double db0 = G.M2 * iQ2 * (drho2 - 2.0 * rdr2) - 2.0 * m.b0 * lQ;
    const double db1 = G.M4a2 * iQ2 * (dr * m.sc + m.r * dsc) - 2.0 * m.b1 * lQ;
    ub[0] += m.g * (dP + m.P * lg) - dbeta * (1.0 + m.v) - m.beta * dv;
    ub[1] += m.g * (dut + ut * lg);
    ub[2] += m.g * (dW + m.W * lg);
    const double q = a2 * (m.x + ur * ur) - m.y * m.y, dq = a2 * (dx + 2.0 * ur * dur) - 2.0 * m.y * dy;
    const double dfur = db0 * m.h + m.b0 * dh + m.g * (dr * m.x + m.r * (dx + m.x * lg));
    const double dfut = db1 * m.h + m.b1 * dh - m.g * (dsc * q + m.sc * (dq + q * lg));
    const double fr = m.g * m.P - m.beta * (1.0 + m.v);
    yb[0] -= (dfur * m.r + dur * fr) * G.dlnr;
    yb[1] -= dfut * G.dth;
}

// ---------------------------------------------------------------- metric of the kick
enum { M_ALPHA, M_IALPHA, M_GRR, M_GRP, M_GTT, M_GPP, M_HRR, M_HRP, M_HTT, M_HPP, M_SQRTG, M_N };

__host__ __device__ inline void metric_at(const Geo& G, const Trig& t, double m[M_N]) {
    const double a = G.a, a2 = G.a2, r2 = t.r * t.r, s2 = t.s * t.s, T = G.M2 * t.r;
    const double rho2 = r2 + a2 * (t.c * t.c), Q = rho2 + T, ra2 = r2 + a2;
    const double irho2 = inv_(rho2), iQ = inv_(Q), is2 = inv_(s2);
    const double z = T * irho2, R = 1.0 + z;
    sqrt_inv_(R, m[M_IALPHA], m[M_ALPHA]);
    m[M_GRR] = R;
    m[M_GRP] = -a * s2 * R;
    m[M_GTT] = rho2;
    m[M_GPP] = s2 * (ra2 + a2 * s2 * z);
    m[M_HRR] = ra2 * irho2 - T * iQ;
    m[M_HRP] = a * irho2;
    m[M_HTT] = irho2;
    m[M_HPP] = irho2 * is2;
    m[M_SQRTG] = rho2 * t.s * m[M_IALPHA];
}

// Cotangents mb of the quantities m = metric_at(t) -> cotangents of r and theta.
__host__ __device__ inline void metric_vjp_at(const Geo& G, const Trig& t, const double m[M_N], const double mb[M_N],
                                              double& rb, double& thb) {
    const double a = G.a, a2 = G.a2, r2 = t.r * t.r, s2 = t.s * t.s, T = G.M2 * t.r;
    const double rho2 = m[M_GTT], irho2 = m[M_HTT], R = m[M_GRR], ra2 = r2 + a2;
    const double iQ = irho2 * m[M_ALPHA] * m[M_ALPHA], z = R - 1.0, al = m[M_ALPHA];
    const double is2rho2 = m[M_HPP];                                // 1/(sin^2 rho^2)
    const double is2 = is2rho2 * rho2;
    const double Rb = mb[M_GRR] - a * s2 * mb[M_GRP] +
                      0.5 * al * (mb[M_IALPHA] + rho2 * t.s * mb[M_SQRTG] - al * al * mb[M_ALPHA]);
    const double sb = rho2 * m[M_IALPHA] * mb[M_SQRTG];
    double s2b = (ra2 + 2.0 * a2 * s2 * z) * mb[M_GPP] - a * R * mb[M_GRP] - is2rho2 * is2 * mb[M_HPP];
    const double zb = a2 * s2 * s2 * mb[M_GPP] + Rb;
    const double ra2b = s2 * mb[M_GPP] + irho2 * mb[M_HRR];
    const double irho2b = ra2 * mb[M_HRR] + a * mb[M_HRP] + mb[M_HTT] + is2 * mb[M_HPP] + T * zb;
    const double Qb = T * iQ * iQ * mb[M_HRR];
    const double Tb = irho2 * zb - iQ * mb[M_HRR] + Qb;
    const double rho2b = mb[M_GTT] + t.s * m[M_IALPHA] * mb[M_SQRTG] - irho2 * irho2 * irho2b + Qb;
    s2b -= a2 * rho2b;
    rb += 2.0 * t.r * (ra2b + rho2b) + G.M2 * Tb;
    thb += (2.0 * t.s * s2b + sb) * t.c;
}

// ---------------------------------------------------------------- Boris
// o = sqrt(gamma) eps_ijk v^j w^k with v^j = gamma^jl a_l.
__host__ __device__ inline void cross(const double m[M_N], const double a[3], const double w[3], double o[3]) {
    const double v0 = m[M_HRR] * a[0] + m[M_HRP] * a[2], v1 = m[M_HTT] * a[1], v2 = m[M_HRP] * a[0] + m[M_HPP] * a[2];
    o[0] = m[M_SQRTG] * (v1 * w[2] - v2 * w[1]);
    o[1] = m[M_SQRTG] * (v2 * w[0] - v0 * w[2]);
    o[2] = m[M_SQRTG] * (v0 * w[1] - v1 * w[0]);
}

__host__ __device__ inline void cross_vjp(const double m[M_N], const double a[3], const double w[3],
                                          const double ob[3], double ab[3], double wb[3], double mb[M_N]) {
    const double sg = m[M_SQRTG];
    const double v0 = m[M_HRR] * a[0] + m[M_HRP] * a[2], v1 = m[M_HTT] * a[1], v2 = m[M_HRP] * a[0] + m[M_HPP] * a[2];
    mb[M_SQRTG] += ob[0] * (v1 * w[2] - v2 * w[1]) + ob[1] * (v2 * w[0] - v0 * w[2]) + ob[2] * (v0 * w[1] - v1 * w[0]);
    wb[0] += sg * (ob[1] * v2 - ob[2] * v1);
    wb[1] += sg * (ob[2] * v0 - ob[0] * v2);
    wb[2] += sg * (ob[0] * v1 - ob[1] * v0);
    const double v0b = sg * (ob[2] * w[1] - ob[1] * w[2]);
    const double v1b = sg * (ob[0] * w[2] - ob[2] * w[0]);
    const double v2b = sg * (ob[1] * w[0] - ob[0] * w[1]);
    ab[0] += v0b * m[M_HRR] + v2b * m[M_HRP];
    ab[1] += v1b * m[M_HTT];
    ab[2] += v0b * m[M_HRP] + v2b * m[M_HPP];
    mb[M_HRR] += v0b * a[0];
    mb[M_HRP] += v0b * a[2] + v2b * a[0];
    mb[M_HTT] += v1b * a[1];
    mb[M_HPP] += v2b * a[2];
}

struct BorisTape {
    double Dl[3], hk, um[3], S, iS, tf, t[3], tt, x1[3], ut[3], sf, s[3];
};

// Full-step generalised Boris kick (eqs. boris-plus-minus, u0bar, boris-scheme).
__host__ __device__ inline void boris(const double m[M_N], double qm, double dt, const double D[3], const double B[3],
                                      const double u[3], double up[3], BorisTape& T) {
    T.Dl[0] = m[M_GRR] * D[0] + m[M_GRP] * D[2];
    T.Dl[1] = m[M_GTT] * D[1];
    T.Dl[2] = m[M_GRP] * D[0] + m[M_GPP] * D[2];
    T.hk = qm * m[M_ALPHA] * dt * 0.5;
    for (int i = 0; i < 3; ++i) T.um[i] = u[i] + T.hk * T.Dl[i];
    const double uu = m[M_HRR] * T.um[0] * T.um[0] + 2.0 * m[M_HRP] * T.um[0] * T.um[2]
                    + m[M_HTT] * T.um[1] * T.um[1] + m[M_HPP] * T.um[2] * T.um[2];
    sqrt_inv_(1.0 + uu, T.S, T.iS);
    T.tf = 0.5 * qm * dt * T.iS * m[M_ALPHA];              // q/m dt / (2 S / alpha)
    for (int i = 0; i < 3; ++i) T.t[i] = T.tf * B[i];
    T.tt = m[M_GRR] * T.t[0] * T.t[0] + 2.0 * m[M_GRP] * T.t[0] * T.t[2]
         + m[M_GTT] * T.t[1] * T.t[1] + m[M_GPP] * T.t[2] * T.t[2];
    cross(m, T.um, T.t, T.x1);
    for (int i = 0; i < 3; ++i) T.ut[i] = T.um[i] + T.x1[i];
    T.sf = 2.0 * inv_(1.0 + T.tt);
    for (int i = 0; i < 3; ++i) T.s[i] = T.sf * T.t[i];
    double x2[3];
    cross(m, T.ut, T.s, x2);
    for (int i = 0; i < 3; ++i) up[i] = T.um[i] + x2[i] + T.hk * T.Dl[i];
}

// Cotangent of the kicked momentum -> cotangents of u, D, B and the metric.
__host__ __device__ inline void boris_vjp(const double m[M_N], double qm, double dt, const double D[3],
                                          const double B[3], const BorisTape& T, const double upb[3], double ub[3],
                                          double Db[3], double Bb[3], double mb[M_N]) {
    double umb[3], Dlb[3], utb[3] = {0, 0, 0}, sb[3] = {0, 0, 0}, x1b[3], tb[3] = {0, 0, 0};
    double hkb = 0.0;
    for (int i = 0; i < 3; ++i) {
        umb[i] = upb[i];
        hkb += upb[i] * T.Dl[i];
        Dlb[i] = upb[i] * T.hk;
    }
    // x2 = cross(ut, s), x2b = upb
    cross_vjp(m, T.ut, T.s, upb, utb, sb, mb);
    // s = sf t
    double sfb = 0.0;
    for (int i = 0; i < 3; ++i) { sfb += sb[i] * T.t[i]; tb[i] += sb[i] * T.sf; }
    const double ttb = -0.5 * sfb * T.sf * T.sf;
    // ut = um + x1
    for (int i = 0; i < 3; ++i) { umb[i] += utb[i]; x1b[i] = utb[i]; }
    cross_vjp(m, T.um, T.t, x1b, umb, tb, mb);
    // tt = t . g . t
    mb[M_GRR] += ttb * T.t[0] * T.t[0];
    mb[M_GRP] += ttb * 2.0 * T.t[0] * T.t[2];
    mb[M_GTT] += ttb * T.t[1] * T.t[1];
    mb[M_GPP] += ttb * T.t[2] * T.t[2];
    tb[0] += ttb * (2.0 * m[M_GRR] * T.t[0] + 2.0 * m[M_GRP] * T.t[2]);
    tb[1] += ttb * 2.0 * m[M_GTT] * T.t[1];
    tb[2] += ttb * (2.0 * m[M_GRP] * T.t[0] + 2.0 * m[M_GPP] * T.t[2]);
    // t = tf B
    double tfb = 0.0;
    for (int i = 0; i < 3; ++i) { tfb += tb[i] * B[i]; Bb[i] += tb[i] * T.tf; }
    // tf = qm dt / (2 u0b); u0b = S ialpha; S = sqrt(1 + uu)
    const double u0bb = -tfb * T.tf * T.iS * m[M_ALPHA];
    const double Sb = u0bb * m[M_IALPHA];
    mb[M_IALPHA] += u0bb * T.S;
    const double uub = 0.5 * Sb * T.iS;
    mb[M_HRR] += uub * T.um[0] * T.um[0];
    mb[M_HRP] += uub * 2.0 * T.um[0] * T.um[2];
    mb[M_HTT] += uub * T.um[1] * T.um[1];
    mb[M_HPP] += uub * T.um[2] * T.um[2];
    umb[0] += uub * (2.0 * m[M_HRR] * T.um[0] + 2.0 * m[M_HRP] * T.um[2]);
    umb[1] += uub * 2.0 * m[M_HTT] * T.um[1];
    umb[2] += uub * (2.0 * m[M_HRP] * T.um[0] + 2.0 * m[M_HPP] * T.um[2]);
    // um = u + hk Dl
    for (int i = 0; i < 3; ++i) {
        ub[i] += umb[i];
        hkb += umb[i] * T.Dl[i];
        Dlb[i] += umb[i] * T.hk;
    }
    mb[M_ALPHA] += hkb * qm * dt * 0.5;
    // Dl = g . D
    Db[0] += Dlb[0] * m[M_GRR] + Dlb[2] * m[M_GRP];
    Db[1] += Dlb[1] * m[M_GTT];
    Db[2] += Dlb[0] * m[M_GRP] + Dlb[2] * m[M_GPP];
    mb[M_GRR] += Dlb[0] * D[0];
    mb[M_GRP] += Dlb[0] * D[2] + Dlb[2] * D[0];
    mb[M_GTT] += Dlb[1] * D[1];
    mb[M_GPP] += Dlb[2] * D[2];
}

// ---------------------------------------------------------------- gather
// Bilinear interpolation in index space at (f, h) (already shifted by the
// stagger) and its reverse: field cotangents are handed to add(e, value).
template <class FieldT>
__host__ __device__ inline double gather(const Geo& G, const FieldT* F, double f, double h) {
    const double ff = ::floor(f), fh = ::floor(h);
    const double wf = f - ff, wh = h - fh;
    const FieldT* p = F + G.index((int)ff, (int)fh);
    const FieldT* q = p + G.pitch;
    return (1.0 - wf) * (1.0 - wh) * p[0] + wf * (1.0 - wh) * q[0] + (1.0 - wf) * wh * p[1] + wf * wh * q[1];
}

// The four field cotangents go to add(e, g): element e of the lower corner,
// then the values for e, e + pitch, e + 1, e + pitch + 1.
template <class FieldT, class Add>
__host__ __device__ inline void gather_vjp(const Geo& G, const FieldT* F, double f, double h, double gb,
                                           double& fb, double& hb, Add add) {
    const double ff = ::floor(f), fh = ::floor(h);
    const double wf = f - ff, wh = h - fh;
    const uint32_t e = G.index((int)ff, (int)fh);
    const FieldT *p = F + e, *q = p + G.pitch;
    const double F00 = p[0], F10 = q[0], F01 = p[1], F11 = q[1];
    fb += gb * ((1.0 - wh) * (F10 - F00) + wh * (F11 - F01));
    hb += gb * ((1.0 - wf) * (F01 - F00) + wf * (F11 - F10));
    const double g[4] = {gb * (1.0 - wf) * (1.0 - wh), gb * wf * (1.0 - wh), gb * (1.0 - wf) * wh, gb * wf * wh};
    add(e, g);
}

// ---------------------------------------------------------------- deposit
// d L / d(xi0, eta0, xi1, eta1, dphi) for L = lambda . (Esirkepov fluxes of
// the move) (eqs. esirkepov-decomp, j-phi-deposit with the local prefix sum).
// With F^r_ab = hf sum_{a' <= a} (wx1 - wx0)_a' (wy0 + wy1)_b, F^th likewise
// and G^ph_ab = cp (wx1 wy1 / 3 + wx0 wy0 / 3 + wx1 wy0 / 6 + wx0 wy1 / 6) the
// derivatives go to the four weight arrays first (the prefix sums become
// suffix sums), then through the weights' slopes to the end points.
// Weights of the window's vertices for an end point at d in [0, 2) from the
// first (the values of max(0, 1 - |d - a|)), and the contraction of dL/d(weights)
// with their slopes (at d = 0 and d = 1, where they jump, a weight of zero has
// slope 0 and a weight of 1 slope +1).
__host__ __device__ inline void window_weights(double d, double w[3]) {
    const double e = d - 1.0;
    w[0] = fmax(0.0, -e);
    w[1] = 1.0 - ::fabs(e);
    w[2] = fmax(0.0, e);
}
__host__ __device__ inline double window_slope(double d, const double g[3]) {
    const double hi = d < 1.0 ? g[1] : g[2], lo = d < 1.0 ? g[0] : g[1];
    return d == 0.0 ? g[0] : (d == 1.0 ? g[1] : hi - lo);
}

template <class LamT>
__host__ __device__ inline void deposit_vjp(const Geo& G, const LamT* lr, const LamT* lt, const LamT* lp, double qw,
                                            double dt, double xi0, double eta0, double xi1, double eta1, double dphi,
                                            double pb[5]) {
    const double fi = ::floor(fmin(xi0, xi1)), fj = ::floor(fmin(eta0, eta1));
    double wx0[3], wx1[3], wy0[3], wy1[3];
    window_weights(xi0 - fi, wx0);
    window_weights(xi1 - fi, wx1);
    window_weights(eta0 - fj, wy0);
    window_weights(eta1 - fj, wy1);
    const double qidt = qw / dt;
    const double hf = -0.5 * qidt, c3 = qidt * dphi * (1.0 / 3.0), c6 = qidt * dphi * (1.0 / 6.0);
    const double fx0 = wx1[0] - wx0[0], fx1 = fx0 + (wx1[1] - wx0[1]);
    const double fy0 = wy1[0] - wy0[0], fy1 = fy0 + (wy1[1] - wy0[1]);
    double gx0[3] = {0, 0, 0}, gx1[3] = {0, 0, 0}, gy0[3], gy1[3];  // dL/d(weights)
    double Ar0 = 0.0, Ar1 = 0.0;
    const uint32_t e0 = G.index((int)fi, (int)fj);
    for (int b = 0; b < 3; ++b) {
        const double l0 = (double)lr[e0 + b], l1 = (double)lr[e0 + G.pitch + b], sy = wy0[b] + wy1[b];
        Ar0 += l0 * sy;
        Ar1 += l1 * sy;
        gy0[b] = gy1[b] = hf * (fx0 * l0 + fx1 * l1);
    }
    gx1[0] = hf * (Ar0 + Ar1);
    gx1[1] = hf * Ar1;
    gx0[0] = -gx1[0];
    gx0[1] = -gx1[1];
    double At0 = 0.0, At1 = 0.0, L_dphi = 0.0;
    for (int a = 0; a < 3; ++a) {
        const uint32_t e = e0 + (uint32_t)(a * G.pitch);
        const double l0 = (double)lt[e], l1 = (double)lt[e + 1], sx = wx0[a] + wx1[a];
        At0 += l0 * sx;
        At1 += l1 * sx;
        const double both = hf * (fy0 * l0 + fy1 * l1);
        double m0 = 0.0, m1 = 0.0;
        for (int b = 0; b < 3; ++b) {
            const double l = (double)lp[e + b];
            m0 += l * wy0[b];
            m1 += l * wy1[b];
            gy0[b] += l * (c3 * wx0[a] + c6 * wx1[a]);
            gy1[b] += l * (c3 * wx1[a] + c6 * wx0[a]);
        }
        gx0[a] += both + c3 * m0 + c6 * m1;
        gx1[a] += both + c3 * m1 + c6 * m0;
        L_dphi += wx1[a] * (2.0 * m1 + m0) + wx0[a] * (2.0 * m0 + m1);
    }
    const double b0 = hf * (At0 + At1), b1 = hf * At1;
    gy1[0] += b0;
    gy1[1] += b1;
    gy0[0] -= b0;
    gy0[1] -= b1;
    pb[0] += window_slope(xi0 - fi, gx0);
    pb[1] += window_slope(eta0 - fj, gy0);
    pb[2] += window_slope(xi1 - fi, gx1);
    pb[3] += window_slope(eta1 - fj, gy1);
    pb[4] += qidt * (1.0 / 6.0) * L_dphi;
}

// ---------------------------------------------------------------- one step
enum { ST_ALIVE = 0, ST_OUT = 1, ST_BAD = 2 };

// Stagger (s_r, s_th) of D^r, D^th, D^ph, B^r, B^th, B^ph (Fig. Yee).
__host__ __device__ inline double stag_r(int c) { return (c == 0 || c == 4 || c == 5) ? 0.5 : 0.0; }
__host__ __device__ inline double stag_t(int c) { return (c == 1 || c == 3 || c == 5) ? 0.5 : 0.0; }

// Storage of the corrector points that f was evaluated at (xi, eta, u_r,
// u_th of each): an array, or the caller's (the GPU kernel's LDS).
template <int NC>                              // NC: bound on the corrector passes
struct PointArray {
    double p[NC][4];
    __host__ __device__ double& at(int it, int c) { return p[it][c]; }
};

template <class Points>
struct StepTape {
    double xi0, eta0;
    double D[3], B[3];
    double up[3];                              // momentum after the kick
    Points pts;
    double u1[2];                              // raw end momenta u_r, u_th
    double xi1, eta1, dphi;                    // end point after reflection
    Corner corner;                             // of the start cell
    int refl, status;
};

// Forward replay of one step from (xi0, eta0, u); fills the tape and returns
// the status.  The same formulas as the plain reference (Sec. 2.2-2.3).
template <bool SMALL, class Points, class FieldT>
__host__ __device__ inline int replay_step(const Geo& G, const FieldT* const F[6], double qm, bool massless,
                                           double dt, int ncorr, double xi0, double eta0, const double u[3],
                                           StepTape<Points>& T) {
    T.xi0 = xi0;
    T.eta0 = eta0;
    for (int c = 0; c < 3; ++c) {
        T.D[c] = gather(G, F[c], xi0 - stag_r(c), eta0 - stag_t(c));
        T.B[c] = gather(G, F[3 + c], xi0 - stag_r(3 + c), eta0 - stag_t(3 + c));
    }
    stage_end();
    T.corner = corner_of<SMALL>(G, xi0, eta0);
    const Trig t0 = trig_at<SMALL>(G, T.corner, xi0, eta0);
    for (int c = 0; c < 3; ++c) T.up[c] = u[c];
    if (!massless) {
        double m0[M_N];
        BorisTape bt;
        metric_at(G, t0, m0);
        boris(m0, qm, dt, T.D, T.B, u, T.up, bt);
    }
    stage_end();
    const double eps = massless ? 0.0 : 1.0;
    double f0[5], f1[5], y[5];
    rhs(G, eps, t0, T.up[0], T.up[1], T.up[2], f0);
    const double y0[5] = {xi0, eta0, 0.0, T.up[0], T.up[1]};
    for (int c = 0; c < 5; ++c) y[c] = y0[c] + dt * f0[c];
#pragma unroll 1
    for (int it = 0; it < ncorr; ++it) {
        stage_end();
        T.pts.at(it, 0) = y[0];
        T.pts.at(it, 1) = y[1];
        T.pts.at(it, 2) = y[3];
        T.pts.at(it, 3) = y[4];
        rhs(G, eps, trig_at<SMALL>(G, T.corner, y[0], y[1]), y[3], y[4], T.up[2], f1);
        for (int c = 0; c < 5; ++c) y[c] = y0[c] + 0.5 * dt * (f1[c] + f0[c]);
    }
    const bool finite = isfinite(y[0]) && isfinite(y[1]) && isfinite(y[2]) && isfinite(y[3]) && isfinite(y[4]) &&
                        isfinite(T.up[2]);
    if (!finite || ::fabs(y[0] - xi0) >= 1.0 || ::fabs(y[1] - eta0) >= 1.0) {
        T.status = ST_BAD;
        return T.status;
    }
    T.xi1 = y[0];
    T.eta1 = y[1];
    T.u1[0] = y[3];
    T.u1[1] = y[4];
    T.refl = 0;
    if (T.eta1 < 0.0) { T.eta1 = -T.eta1; T.refl = 1; }
    else if (T.eta1 > (double)G.nth) { T.eta1 = 2.0 * G.nth - T.eta1; T.refl = 2; }
    T.dphi = y[2];
    T.status = (T.xi1 < 0.0 || T.xi1 >= (double)G.nr) ? ST_OUT : ST_ALIVE;
    return T.status;
}

// Reverse of one step.  a[5] holds on entry the cotangent of the state after
// the step (xi, eta, u_r, u_th, u_ph; zero if the particle did not survive
// it) and on return the cotangent of the state before it.  start(u) reads the
// momentum before the step again (rather than the tape keeping it).  Field
// cotangents go to addF(component, lower-corner element, four values) as in
// gather_vjp.
template <bool SMALL, class Points, class FieldT, class LamT, class Start, class AddF>
__host__ __device__ inline void reverse_step(const Geo& G, const FieldT* const F[6], const LamT* const lam[3],
                                             double qm, bool massless, double qw, double dt, int ncorr,
                                             StepTape<Points>& T, double a[5], Start start, AddF addF) {
    if (T.status == ST_BAD) {
        for (int c = 0; c < 5; ++c) a[c] = 0.0;
        return;
    }
    if (T.status == ST_OUT) for (int c = 0; c < 5; ++c) a[c] = 0.0;
    // deposit: d/d(xi0, eta0, xi1, eta1, dphi)
    double pb[5] = {0, 0, 0, 0, 0};
    deposit_vjp(G, lam[0], lam[1], lam[2], qw, dt, T.xi0, T.eta0, T.xi1, T.eta1, T.dphi, pb);
    stage_end();
    // cotangent of the raw predictor-corrector output y = (xi, eta, phi, u_r, u_th) and u_ph
    double z[5];
    z[0] = a[0] + pb[2];
    double etab = a[1] + pb[3], utb = a[3];
    if (T.refl) { etab = -etab; utb = -utb; }
    z[1] = etab;
    z[2] = pb[4];
    z[3] = a[2];
    z[4] = utb;
    double upb[3] = {0.0, 0.0, a[4]};        // u_ph passes through the predictor-corrector
    // y_m = y0 + dt/2 (f(y_{m-1}) + f0), so the cotangents of y0 and f0 are
    // sum z_m (+ z_0) and dt/2 sum z_m (+ dt z_0)
    double sum[5] = {0, 0, 0, 0, 0}, y0b[5], f0b[5];
    const double eps = massless ? 0.0 : 1.0;
    const double h = 0.5 * dt;
#pragma unroll 1
    for (int m = ncorr; m >= 1; --m) {
        stage_end();
        double g[5], pyb[2] = {0.0, 0.0}, pub[3] = {0.0, 0.0, 0.0};
        for (int c = 0; c < 5; ++c) { sum[c] += z[c]; g[c] = h * z[c]; }
        const double px = T.pts.at(m - 1, 0), pe = T.pts.at(m - 1, 1);
        rhs_vjp(G, eps, trig_at<SMALL>(G, T.corner, px, pe), T.pts.at(m - 1, 2), T.pts.at(m - 1, 3), T.up[2], g, pyb, pub);
        z[0] = pyb[0];
        z[1] = pyb[1];
        z[2] = 0.0;                          // f does not depend on phi
        z[3] = pub[0];
        z[4] = pub[1];
        upb[2] += pub[2];
    }
    for (int c = 0; c < 5; ++c) { y0b[c] = sum[c] + z[c]; f0b[c] = h * sum[c] + dt * z[c]; }
    stage_end();
    // f0 = f(y0) at x^n; its metric adjoint goes into the position
    const Trig t0 = trig_at<SMALL>(G, T.corner, T.xi0, T.eta0);
    {
        double pyb[2] = {0.0, 0.0}, pub[3] = {0.0, 0.0, 0.0};
        rhs_vjp(G, eps, t0, T.up[0], T.up[1], T.up[2], f0b, pyb, pub);
        y0b[0] += pyb[0];
        y0b[1] += pyb[1];
        upb[0] += pub[0];
        upb[1] += pub[1];
        upb[2] += pub[2];
    }
    stage_end();
    upb[0] += y0b[3];
    upb[1] += y0b[4];
    double xib = y0b[0] + pb[0], etab0 = y0b[1] + pb[1];
    double ub[3] = {0.0, 0.0, 0.0}, Db[3] = {0.0, 0.0, 0.0}, Bb[3] = {0.0, 0.0, 0.0};
    if (massless) {
        for (int c = 0; c < 3; ++c) ub[c] = upb[c];
    } else {
        double m0[M_N], mb[M_N];
        double u[3];
        start(u);
        metric_at(G, t0, m0);
        for (int i = 0; i < M_N; ++i) mb[i] = 0.0;
        BorisTape bt;
        double up[3];
        boris(m0, qm, dt, T.D, T.B, u, up, bt);
        boris_vjp(m0, qm, dt, T.D, T.B, bt, upb, ub, Db, Bb, mb);
        double rb = 0.0, thb = 0.0;
        metric_vjp_at(G, t0, m0, mb, rb, thb);
        xib += rb * t0.r * G.dlnr;
        etab0 += thb * G.dth;
    }
    // gather: fields and the interpolation weights' dependence on position
    for (int c = 0; c < 6; ++c) {
        stage_end();
        const double gb = c < 3 ? Db[c] : Bb[c - 3];
        if (gb == 0.0) continue;
        double fb = 0.0, hb = 0.0;
        gather_vjp(G, F[c], T.xi0 - stag_r(c), T.eta0 - stag_t(c), gb, fb, hb,
                   [&](uint32_t e, const double g[4]) { addF(c, e, g); });
        xib += fb;
        etab0 += hb;
    }
    a[0] = xib;
    a[1] = etab0;
    a[2] = ub[0];
    a[3] = ub[1];
    a[4] = ub[2];
}

}  // namespace adj
}  // namespace grpic
