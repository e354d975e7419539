// fields.hip -- the field solver of Sec. 2.1 and App. B of arXiv:2503.04558:
// the integral form of the 3+1 Maxwell equations on the staggered Yee grid,
// advanced by a predictor and ncorr semi-implicit corrector passes.
//
// A pass evaluates the auxiliary fields E_i, H_i of eqs. auxE / auxH, their
// circulations (eqs. D-update, B-update; the axis rows of D^r by eq. Dr-axis)
// and the predictor or corrector value of every point; the metric
// coefficients are evaluated on the fly from tabulated r and sin, cos theta.
// Up to four passes run in one launch (field_march_kernel).
//
// Locations, array element (i, j) of each component (r_x = exp(lnr0 + x
// dlnr), theta_y = y dth): D^r, B^th, E_r, H_th at (i+1/2, j); D^th, B^r,
// E_th, H_r at (i, j+1/2); D^ph, E_ph at (i, j); B^ph, H_ph at (i+1/2, j+1/2).
// Areas and volumes are per unit phi (the deposit's flux-form currents are
// J^r A^D_r, J^th A^D_th, J^ph A^D_ph).
#include "grpic_device.hpp"
#include "grpic_fields.hpp"

#include <algorithm>

namespace grpic {
namespace {

__device__ __forceinline__ double rad(const FieldArgs& F, double x) { return exp(F.lnr0 + x * F.dlnr); }

// sqrt(det gamma) of the Kerr-Schild 3-metric (App. A, M reinstated).
__device__ __forceinline__ double sqrt_gamma(double a, double M, double r, double th) {
    const double s = sin(th), c = cos(th);
    const double rho2 = r * r + a * a * c * c;
    return rho2 * fabs(s) * sqrt(1.0 + 2.0 * M * r / rho2);
}

struct Coef {
    double aGrr, aGrp, aGtt, aGpp, sgB;                 // alpha gamma_ij, sqrt(gamma) beta^r
};

struct Quad {
    double x[10], w[10];
};

__device__ __forceinline__ double int_th(const FieldArgs& F, const Quad& Q, double r, double t0, double t1) {
    double s = 0.0;
    for (int k = 0; k < 10; ++k) s += Q.w[k] * sqrt_gamma(F.a, F.M, r, 0.5 * (t0 + t1) + 0.5 * (t1 - t0) * Q.x[k]);
    return 0.5 * (t1 - t0) * s;
}
__device__ __forceinline__ double int_r(const FieldArgs& F, const Quad& Q, double th, double r0, double r1) {
    double s = 0.0;
    for (int k = 0; k < 10; ++k) s += Q.w[k] * sqrt_gamma(F.a, F.M, 0.5 * (r0 + r1) + 0.5 * (r1 - r0) * Q.x[k], th);
    return 0.5 * (r1 - r0) * s;
}
__device__ __forceinline__ double int_rth(const FieldArgs& F, const Quad& Q, double r0, double r1, double t0,
                                          double t1) {
    double s = 0.0;
    for (int k = 0; k < 10; ++k) s += Q.w[k] * int_th(F, Q, 0.5 * (r0 + r1) + 0.5 * (r1 - r0) * Q.x[k], t0, t1);
    return 0.5 * (r1 - r0) * s;
}

__device__ __forceinline__ double inv_or_zero(double v) { return v != 0.0 ? 1.0 / v : 0.0; }

// Tables: inverse areas of the six components over the physical rows and
// columns (zero in the other rows -2, -1, nr + 1 that the table covers),
// radial edge lengths per row, radii and sin, cos at half-integer steps.
__global__ __launch_bounds__(256) void field_tables_kernel(FieldArgs F, Quad Q) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int ncol = F.nth + 1;
    if (t < field_nrad(F.nr)) F.rad[t] = rad(F, -2.0 + 0.5 * (double)t);
    if (t < field_nang(F.nth)) {
        F.sn[t] = sin(0.5 * (double)t * F.dth);
        F.sn[field_nang(F.nth) + t] = cos(0.5 * (double)t * F.dth);
    }
    if (t >= (int64_t)ncol * F.nrow) return;
    const int i = (int)(t / ncol) + kTableRowLo, j = (int)(t % ncol);
    const uint32_t e = F.at(i, j);
    const double th_j = j * F.dth, th_h = (j + 0.5) * F.dth;
    const double r_i = rad(F, i), r_h = rad(F, i + 0.5);
    auto clamp_th = [&](double y) { return fmin(fmax(y, 0.0), (double)F.nth) * F.dth; };
    double iADr = 0.0, iADt = 0.0, iADp = 0.0, iABr = 0.0, iABt = 0.0, iABp = 0.0;
    if (i >= 0 && i <= F.nr) {
        const double r_m = rad(F, i - 0.5), r_p = rad(F, i + 1.0);
        if (i < F.nr) iADr = inv_or_zero(int_th(F, Q, r_h, clamp_th(j - 0.5), clamp_th(j + 0.5)));
        if (j < F.nth) iADt = inv_or_zero(int_r(F, Q, th_h, r_m, r_h));
        if (j > 0 && j < F.nth) iADp = inv_or_zero(int_rth(F, Q, r_m, r_h, clamp_th(j - 0.5), clamp_th(j + 0.5)));
        if (j < F.nth) iABr = inv_or_zero(int_th(F, Q, r_i, th_j, (j + 1) * F.dth));
        if (i < F.nr && j > 0 && j < F.nth) iABt = inv_or_zero(int_r(F, Q, th_j, r_i, r_p));
        if (i < F.nr && j < F.nth) iABp = inv_or_zero(int_rth(F, Q, r_i, r_p, th_j, (j + 1) * F.dth));
    }
    double* T = F.tab;
    const size_t S = F.plane;
    T[kT_iADr * S + e] = iADr;
    T[kT_iADt * S + e] = iADt;
    T[kT_iADp * S + e] = iADp;
    T[kT_iABr * S + e] = iABr;
    T[kT_iABt * S + e] = iABt;
    T[kT_iABp * S + e] = iABp;
    if (j == 0) {                                       // radial edge lengths of row i
        F.drow[kDrPrimal * F.nrow + (i - kTableRowLo)] = rad(F, i + 1.0) - r_i;
        F.drow[kDrDual * F.nrow + (i - kTableRowLo)] = r_h - rad(F, i - 0.5);
    }
}

// ---------------------------------------------------------------- the passes
// A circulation pass reaches one row and one column to each side, so K passes
// need a halo of K.  K + 1 waves run K consecutive passes over a strip of 64
// columns and a segment of rows, marching up the rows: one wave loads them into
// LDS (the iterate, R and the areas) two rows ahead, wave w runs pass w, taking
// each row from its predecessor through LDS two rows behind it, and the last
// one writes it.  A lane is a column: neighbours in theta are lane shifts,
// neighbours in r the marching wave's own registers.  So an iterate, R and the
// areas go through memory once per K passes, and a point's coefficients are
// formed once per pass (a tile with a halo formed each four times over).
//
// Measured, predictor and 7 correctors on 2048 x 2048: 500 us in two launches
// of four passes, 0.96 and 0.87 GB of HBM traffic, where one launch per pass
// took 1560 us (0.82 to 1.12 GB each, 8 launches and 3 for the edges).  What
// bounds it now is the marching step's latency: the waves of a workgroup meet
// at a barrier each row, VALU issue fills half of the time and HBM runs at 3.7
// TB/s.  Three passes per launch: 870 us, two: 810 (without the second strip,
// which gave 685 for four); R and the areas re-read by each pass instead of
// kept in LDS: 1.58 GB per launch, 765 us.
constexpr int kMaxStages = 4;
constexpr int kRing = 8;                                // rows of R and the areas in LDS: 2 kMaxStages are in use

// The value of the lane below / above (lane - 1, lane + 1); zero where there is none.
__device__ __forceinline__ double lane_below(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x138, 0xF, 0xF, true);   // wave_shr:1
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x138, 0xF, 0xF, true);
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double lane_above(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x130, 0xF, 0xF, true);   // wave_shl:1
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x130, 0xF, 0xF, true);
    return __hiloint2double(hi, lo);
}

struct StageArgs {
    int strips, seg_rows;                               // strips of 64 columns, rows of a segment
    unsigned nwg, per_xcd;                              // strips x segments, and an XCD's share of them
    int last;                                           // the step's last launch: out is the state
    int store_R;                                        // a later launch needs R
    int guard_rows, pad_end;                            // guard rows that the last launch writes, end of their columns
    int damp_cells;
    double damp_max;
};

// The metric factors of one column: sin^2, a^2 cos^2, |sin|, and of one row.
struct ColK {
    double s2, ac2, s;
};
struct RowK {
    double r2, ra2, tMr;
};
__device__ __forceinline__ RowK row_at(const FieldArgs& F, double r) {
    return {r * r, fma(r, r, F.a * F.a), 2.0 * F.M * r};
}

// Coefficients at a row and column, with alpha = 1/sqrt(1 + z), z = 2 M r /
// rho^2: alpha gamma_rr = sqrt(1 + z), alpha gamma_rph = -a sin^2 sqrt(1 + z),
// alpha gamma_thth = rho^2 alpha, alpha gamma_phph = alpha Sigma sin^2 / rho^2
// with Sigma / rho^2 = r^2 + a^2 + z a^2 sin^2, and sqrt(gamma) beta^r =
// 2 M r |sin| alpha.  The hardware estimates of 1 / rho^2 and (1 + z)^(-1/2)
// (2^-23) take one third-order step each: d + d^2, and e/2 + 3 e^2 / 8 of the
// residual.  (From one estimate, of (rho^2 (rho^2 + 2 M r))^(-1/2), a step is
// 5 % faster and its error against 64-bit sums 5 to 10 % larger than that of
// two Newton steps; this one's is 0 to 15 % smaller.)
__device__ __forceinline__ Coef coef_point(const FieldArgs& F, const RowK& R, const ColK& C) {
    const double rho2 = R.r2 + C.ac2;
    const double i0 = __builtin_amdgcn_rcp(rho2);
    const double d = fma(-rho2, i0, 1.0);
    const double irho2 = fma(i0, fma(d, d, d), i0);
    const double opz = fma(R.tMr, irho2, 1.0);
    const double y0 = __builtin_amdgcn_rsq(opz);
    const double g = opz * y0;
    const double e = fma(-g, y0, 1.0), t = e * fma(0.375, e, 0.5);
    const double alpha = fma(y0, t, y0);
    Coef k;
    k.aGrr = fma(g, t, g);
    k.aGrp = (-F.a * C.s2) * k.aGrr;
    k.aGtt = alpha * rho2;
    k.aGpp = fma(R.tMr * irho2, F.a * F.a * C.s2, R.ra2) * (C.s2 * alpha);
    k.sgB = (R.tMr * C.s) * alpha;
    return k;
}

// What a marching pass carries from row to row: the products of row m - 1
// that the averages onto the next row take, the half-row auxiliary fields'
// own terms, the whole-row auxiliary fields of row m - 1 and the half-row
// ones of row m - 2.
struct MarchState {
    double p1, p2, q1, q2, b1, b2, t1, t2;
    double oDr, oBt, oBp;
    double Et, Ep, Hr, Hp, Ht;
};

// The step's last pass: row r of the new state, with the damping layer
// (values at radial position x >= nr - L scaled by 1 - d ((x - nr + L) /
// L)^2), the guard rows, and the columns beyond the axes, which the
// particles' gather reads within half a cell of an axis.  By axisymmetry (the
// extended chart's point (r, -theta, phi) is (r, theta, phi + pi), where only
// the theta basis vector is reversed) a component there is its value at the
// mirrored location, negated for D^th and B^th: integer columns -m <-> m and
// nth + m <-> nth - m, columns at j + 1/2 (D^th, B^r, B^ph) -m <-> m - 1 and
// nth - 1 + m <-> nth - m, m = 1 .. guard (nth > guard); each is stored by the
// lane of its mirror image (mirrors: this strip stores some).
// Rows between the edges, which are nearly all, take no loop: this wave's
// rows are what the others wait for.
__device__ __forceinline__ void store_state(const FieldArgs& F, const FieldPtrs& out, const StageArgs& S, int r, int j,
                                            int lane, bool owned, bool mirrors, bool last_strip, double v[6]) {
    const int L = S.damp_cells;
    if (L > 0 && r >= F.nr - L - 1) {                   // damping at x = r, r + 1/2
        const double x_in = (double)(F.nr - L);
        auto damp = [&](double x) {
            const double q = (x - x_in) / L;
            return x < x_in ? 1.0 : 1.0 - S.damp_max * q * q;
        };
        const double f_i = damp((double)r), f_h = damp(r + 0.5);
        for (int c = 0; c < 6; ++c) v[c] *= c == 0 || c > 3 ? f_h : f_i;
    }
    const int fm = F.nth - j;
    // row q of component c, and its mirrored columns
    auto put = [&](int c, int q) {
        const bool chalf = c == 1 || c == 3 || c == 5;
        if (owned && !(chalf && fm == 0)) *elem(out.c[c], F.at(q, j)) = v[c];   // (a mirrored column there)
    };
    auto mirror = [&](int c, int q) {
        const bool chalf = c == 1 || c == 3 || c == 5;
        const double mir = (c == 1 || c == 4) ? -v[c] : v[c];
        const int near = chalf ? -j - 1 : -j;
        if (owned && near < 0 && near >= -F.guard) *elem(out.c[c], F.at(q, near)) = mir;
        if (owned && fm >= 1 && fm <= F.guard) *elem(out.c[c], F.at(q, (chalf ? 2 * F.nth - 1 : 2 * F.nth) - j)) = mir;
    };
    if (r > 0 && r < F.nr - 1) {
        for (int c = 0; c < 6; ++c) put(c, r);
        if (mirrors)
            for (int c = 0; c < 6; ++c) mirror(c, r);
        return;
    }
    // (with no guard rows of its own this also stores row nr of the half-row components, one of them)
    for (int c = 0; c < 6; ++c) {
        const bool half = c == 0 || c > 3, chalf = c == 1 || c == 3 || c == 5;
        const int top = half ? F.nr - 1 : F.nr;
        if (r > top) continue;
        const int lo = r == 0 ? -S.guard_rows : r, hi = r == top ? F.nr + S.guard_rows : r;
        for (int q = lo; q <= hi; ++q) {
            put(c, q);
            if (mirrors) mirror(c, q);
        }
        // the guard rows' columns beyond the mirrored ones repeat the edge row's
        if (last_strip && lo < hi)
            for (int p = F.nth + F.guard + (chalf ? 0 : 1) + lane; p < S.pad_end; p += 64)
                for (int q = lo; q <= hi; ++q)
                    if (q != r) *elem(out.c[c], F.at(q, p)) = *elem(out.c[c], F.at(r, p));
    }
}

// K passes over one strip and segment.  FIRST: the launch's first pass is the
// predictor (in is the start state X^n, whose axis values of D^ph, B^th count
// as zero); it forms R = x0 + dt (w0 C - J) and the value x0 + dt (C - J),
// every other pass's value is R + dt w1 C.  Rows beyond the edges repeat the
// edge rows (zero gradient): a pass keeps the last row it was given, and at
// row 0 takes it for row -1 first.  The step's last launch writes the state.
//
// in must not alias out (neighbouring workgroups read their halo of it).
// Workgroup w runs on XCD w mod 8 (the dispatcher's round robin), so logical
// index (w mod 8) per + w / 8 gives each XCD neighbouring strips, whose halo
// columns then come through the same L2.
template <int K, bool FIRST, int H>
__global__ __launch_bounds__(64 * H * (K + 1)) __attribute__((amdgpu_waves_per_eu(3))) void field_march_kernel(
    FieldArgs F, FieldPtrs in, FieldPtrs R, FieldPtrs out, StageArgs S, const double* __restrict__ T,
    const double* __restrict__ rad, const double* __restrict__ drow) {
    __shared__ double xrs[H][K][2][6][64];   // rows handed to pass w
    __shared__ double ras[H][kRing][12][64]; // R (the predictor's x0 before it), then the inverse areas
    __shared__ double jrs[FIRST ? H : 1][2][3][64];   // the predictor's currents
    const unsigned wg = (blockIdx.x & 7u) * S.per_xcd + (blockIdx.x >> 3);
    if (wg >= S.nwg) return;                            // whole workgroup: before any barrier
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int h = wave / (K + 1), w = wave % (K + 1) - 1;
    auto& xr = xrs[h];
    auto& ra = ras[h];
    auto& jr = jrs[FIRST ? h : 0];
    const int pairs = (S.strips + H - 1) / H;
    const int strip = (int)(wg % (unsigned)pairs) * H + h;   // may be one past the last: an idle half
    const int a = (int)(wg / (unsigned)pairs) * S.seg_rows, b = min(a + S.seg_rows, F.nr + 1);
    const FieldStrips cut(K, F.nth);
    const int j = cut.first_column(strip) + lane, jc = min(j, F.nth);
    const bool axis = j == 0 || j >= F.nth;
    const int m0 = max(a - K, 0);                       // the first row read
    const int steps = b - m0 + 2 * K;                   // row b comes to the last pass in the last one

    if (w < 0) {                                        // the loading wave, two rows ahead
        const size_t P = F.plane;
        double q[2][21];
        auto load = [&](int t, double o[21]) {          // what step t hands on: row m0 + t, and R, areas, currents of the one before
            const int m = m0 + t;
            const uint32_t ei = F.at(min(m, F.nr), jc), eh = F.at(min(m, F.nr - 1), jc);
            const uint32_t e = F.at(min(max(m - 1, 0), F.nr), jc);
            for (int c = 0; c < 6; ++c) o[c] = *elem(in.c[c], c == 0 || c > 3 ? eh : ei);
            for (int c = 0; c < 6; ++c) o[6 + c] = *elem(FIRST ? in.c[c] : R.c[c], e);
            for (int c = 0; c < 6; ++c) o[12 + c] = *elem(T + c * P, e);
            if (FIRST)
                for (int c = 0; c < 3; ++c) o[18 + c] = F.J[c] ? *elem(F.J[c], e) : 0.0;
        };
        auto hand = [&](int t, const double o[21]) {
            const int m = m0 + t;
            for (int c = 0; c < 6; ++c) {
                const bool zero = FIRST && axis && (c == 2 || c == 4);
                xr[0][m & 1][c][lane] = zero ? 0.0 : o[c];
                ra[(m - 1) & (kRing - 1)][c][lane] = zero ? 0.0 : o[6 + c];
                ra[(m - 1) & (kRing - 1)][6 + c][lane] = o[12 + c];
            }
            if (FIRST)
                for (int c = 0; c < 3; ++c) jr[(m - 1) & 1][c][lane] = o[18 + c];
        };
        load(0, q[0]);
        load(1, q[1]);
        for (int t = 0; t < steps; t += 2) {
            hand(t, q[0]);
            load(t + 2, q[0]);
            __syncthreads();
            if (t + 1 < steps) {
                hand(t + 1, q[1]);
                load(t + 3, q[1]);
                __syncthreads();
            }
        }
        return;
    }

    const bool owned = cut.stores(strip, lane), mirrors = cut.mirrors(strip, F.guard);
    const bool beyond = j >= F.nth;
    ColK ci, ch;                                        // columns j and j + 1/2
    {
        const double* cs = F.sn + field_nang(F.nth);
        const int hi = 2 * jc, hh = min(2 * jc + 1, 2 * F.nth);
        const double si = F.sn[hi], cc = F.a * cs[hi], sh = F.sn[hh], chh = F.a * cs[hh];
        ci = {si * si, cc * cc, fabs(si)};
        ch = {sh * sh, chh * chh, fabs(sh)};
    }
    const int m_end = min(b + K - 1 - w, F.nr + 1);     // the last row this wave takes
    double X[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    MarchState s = {};
    for (int t = 0; t < steps; ++t) {
        const int m = m0 + t - 2 * w - 1;
        if (m >= m0 && m <= m_end) {
            {
                const double(*src)[64] = xr[w][m & 1];
                if (m <= F.nr)
                    for (int c = 1; c < 4; ++c) X[c] = src[c][lane];
                if (m < F.nr) {
                    X[0] = src[0][lane];
                    X[4] = src[4][lane];
                    X[5] = src[5][lane];
                }
            }
            if (m == 0) {                               // row -1, a copy of row 0
                const RowK ri = row_at(F, rad[2]), rh = row_at(F, rad[3]);
                const Coef kR = coef_point(F, rh, ci), kP = coef_point(F, ri, ci);
                const Coef kT = coef_point(F, ri, ch), kB = coef_point(F, rh, ch);
                s = {kP.aGrp * X[2], kP.sgB * X[2], kR.aGrp * X[0], kR.sgB * X[4], kB.sgB * X[5], kB.aGrp * X[5],
                     kT.aGrp * X[3], kT.sgB * X[1], kR.aGrr * X[0], kR.aGtt * X[4], kB.aGpp * X[5],
                     0.0, 0.0, 0.0, 0.0, 0.0};
            }
            const RowK ri = row_at(F, rad[2 * m + 4]), rh = row_at(F, rad[2 * m + 5]);
            const Coef kR = coef_point(F, rh, ci), kP = coef_point(F, ri, ci);
            const Coef kT = coef_point(F, ri, ch), kB = coef_point(F, rh, ch);
            const double np1 = kP.aGrp * X[2], np2 = kP.sgB * X[2];
            const double nq1 = kR.aGrp * X[0], nq2 = kR.sgB * X[4];
            const double nb1 = kB.sgB * X[5], nb2 = kB.aGrp * X[5];
            const double nt1 = kT.aGrp * X[3], nt2 = kT.sgB * X[1];
            // half-row auxiliary fields of row m - 1, whole-row ones of row m
            const double Er = s.oDr + 0.5 * (s.p1 + np1);
            const double Ht = s.oBt + 0.5 * (s.p2 + np2);
            double Hp = s.oBp + 0.5 * (s.t1 + nt1) - 0.5 * (s.t2 + nt2);
            const double Ep = kP.aGpp * X[2] + 0.5 * (nq1 + s.q1) + 0.5 * (nq2 + s.q2);
            double Et = kT.aGtt * X[1] - 0.5 * (nb1 + s.b1);
            double Hr = kT.aGrr * X[3] + 0.5 * (nb2 + s.b2);
            if (beyond) Hp = Et = Hr = 0.0;             // no such location beyond the far axis
            const int r = m - 1;                        // the row emitted
            if (r >= m0) {
                // circulations of row r
                const double dr = drow[kDrPrimal * F.nrow + (r - kTableRowLo)];
                const double drd = drow[kDrDual * F.nrow + (r - kTableRowLo)];
                const double Hpm = lane_below(Hp), Hrm = lane_below(s.Hr);
                const double Epp = lane_above(s.Ep), Erp = lane_above(Er);
                double Cv[6];
                Cv[0] = Hp - (j == 0 ? 0.0 : Hpm);
                Cv[1] = s.Hp - Hp;
                Cv[2] = (Ht - s.Ht) * F.dth + (Hrm - s.Hr) * drd;
                Cv[3] = -(Epp - s.Ep);
                Cv[4] = -(s.Ep - Ep);
                Cv[5] = -((Et - s.Et) * F.dth + (Er - Erp) * dr);
                double(*ring)[64] = ra[r & (kRing - 1)];
                double v[6];
                if (FIRST && w == 0) {
                    double Rv[6];
                    for (int c = 0; c < 6; ++c) {
                        const double x0 = ring[c][lane], A = ring[6 + c][lane];
                        const double C = Cv[c] * A, cur = c < 3 ? jr[r & 1][c][lane] * A : 0.0;
                        Rv[c] = x0 + F.dt * (F.w0 * C - cur);
                        v[c] = x0 + F.dt * (C - cur);
                    }
                    if (axis) Rv[2] = Rv[4] = 0.0;
                    if (K > 1)
                        for (int c = 0; c < 6; ++c) ring[c][lane] = Rv[c];
                    if (S.store_R && owned && r >= a && r < b) {
                        const uint32_t e = F.at(r, j);
                        for (int c = 0; c < 6; ++c) *elem(R.c[c], e) = Rv[c];
                    }
                } else {
                    for (int c = 0; c < 6; ++c) v[c] = ring[c][lane] + F.dt * F.w1 * (Cv[c] * ring[6 + c][lane]);
                }
                if (axis) v[2] = v[4] = 0.0;
                if (w < K - 1) {
                    for (int c = 0; c < 6; ++c) xr[w + 1][r & 1][c][lane] = v[c];
                } else if (r >= a && r < b) {
                    if (!S.last) {
                        const uint32_t e = F.at(r, jc);
                        if (owned)
                            for (int c = 0; c < 6; ++c) *elem(out.c[c], e) = v[c];
                    } else {
                        store_state(F, out, S, r, j, lane, owned, mirrors, strip == cut.count - 1, v);
                    }
                }
            }
            s = {np1, np2, nq1, nq2, nb1, nb2, nt1, nt2, kR.aGrr * X[0], kR.aGtt * X[4], kB.aGpp * X[5],
                 Et, Ep, Hr, Hp, Ht};
        }
        __syncthreads();
    }
}

// `runs` runs of `width` elements of the six arrays, a row apart, from e0.
__global__ __launch_bounds__(256) void field_copy_kernel(FieldArgs F, FieldPtrs dst, FieldPtrs src, uint32_t e0,
                                                         uint32_t runs, uint32_t width) {
    const uint32_t t = blockIdx.x * 256u + threadIdx.x, i = runs == 1u ? 0u : t / width;
    if (i >= runs || t - i * width >= width) return;
    const uint32_t e = e0 + i * (uint32_t)F.pitch + (t - i * width);
    for (int c = 0; c < 6; ++c) *elem(dst.c[c], e) = *elem(src.c[c], e);
}

// The guard rows, all columns, from the edge rows (zero gradient).
__global__ __launch_bounds__(256) void field_guard_rows_kernel(FieldArgs F, FieldPtrs X) {
    const uint32_t t = blockIdx.x * 256u + threadIdx.x, k = t / (uint32_t)F.pitch;
    const int j = (int)(t - k * (uint32_t)F.pitch) - F.guard;
    if (k > 2u * (uint32_t)F.guard) return;
    const int q = (int)k < F.guard ? (int)k - F.guard : F.nr + (int)k - F.guard;   // -guard .. -1, nr .. nr + guard
    for (int c = 0; c < 6; ++c) {
        const int edge = q < 0 ? 0 : c == 0 || c > 3 ? F.nr - 1 : F.nr;
        if (q != edge) *elem(X.c[c], F.at(q, j)) = *elem(X.c[c], F.at(edge, j));
    }
}

inline unsigned nb(int64_t n) { return (unsigned)((n + 255) / 256); }

}  // namespace

hipError_t launch_field_tables(const FieldArgs& F, const double* gx, const double* gw, hipStream_t stream) {
    Quad Q;
    for (int k = 0; k < 10; ++k) {
        Q.x[k] = gx[k];
        Q.w[k] = gw[k];
    }
    const int64_t n = std::max<int64_t>((int64_t)(F.nth + 1) * F.nrow,
                                        std::max(field_nrad(F.nr), field_nang(F.nth)));
    hipLaunchKernelGGL(field_tables_kernel, dim3(nb(n)), dim3(256), 0, stream, F, Q);
    return hipGetLastError();
}

template <int K, bool FIRST>
static void launch_march(const FieldArgs& F, FieldPtrs in, FieldPtrs R, FieldPtrs out, StageArgs S,
                         hipStream_t stream) {
    const FieldMarch L(K, F.nr, F.nth, F.plane);
    S.strips = L.strips;
    S.seg_rows = L.seg_rows;
    S.nwg = (unsigned)L.workgroups;
    S.per_xcd = (S.nwg + 7) / 8;
    const dim3 grid(8 * S.per_xcd);
    if (L.two)
        hipLaunchKernelGGL((field_march_kernel<K, FIRST, 2>), grid, dim3(128 * (K + 1)), 0, stream, F, in, R, out, S,
                           F.tab, F.rad, F.drow);
    else
        hipLaunchKernelGGL((field_march_kernel<K, FIRST, 1>), grid, dim3(64 * (K + 1)), 0, stream, F, in, R, out, S,
                           F.tab, F.rad, F.drow);
}

template <bool FIRST>
static void launch_passes(int K, const FieldArgs& F, FieldPtrs in, FieldPtrs R, FieldPtrs out, const StageArgs& S,
                          hipStream_t stream) {
    if (K == 1) launch_march<1, FIRST>(F, in, R, out, S, stream);
    else if (K == 2) launch_march<2, FIRST>(F, in, R, out, S, stream);
    else if (K == 3) launch_march<3, FIRST>(F, in, R, out, S, stream);
    else launch_march<4, FIRST>(F, in, R, out, S, stream);
}

constexpr int kFewGuardRows = 6;

// The step's 1 + ncorr passes in launches of up to kMaxStages.  Steps of one or
// two passes run in one launch that reads a copy of X (33 planes of traffic
// with the copy, 51 in two launches); others in at least two: the first reads X
// and leaves R, the last writes X, those between alternate between W1 and W2.
hipError_t launch_field_step(const FieldArgs& F, FieldPtrs X, FieldPtrs R, FieldPtrs W1, FieldPtrs W2, int ncorr,
                             int damp_cells, double damp_max, hipStream_t stream) {
    StageArgs S{};
    S.damp_cells = damp_cells;
    S.damp_max = damp_max;
    const int passes = ncorr + 1;
    // Guard rows: by the last launch's waves at the edge rows while they and their
    // padding are few, else by a launch of their own, as those waves store them one
    // after another.  256 x 256, no corrector: 6 guard rows 20.3 us in the waves and
    // 19.8 apart, 8 22 and 20, 100 90 and 21 (1000 x 1000: 6 61 and 63, 8 62 and 61);
    // 1000 x 1000 with 3000 columns of padding, one corrector, 292 and 76 us.
    const bool apart = F.guard > kFewGuardRows || F.pitch - F.nth - 2 * F.guard > 64;
    S.guard_rows = apart ? 0 : F.guard;
    S.pad_end = apart ? 0 : F.pitch - F.guard;
    auto finish = [&] {
        if (apart)
            hipLaunchKernelGGL(field_guard_rows_kernel, dim3(nb((int64_t)(2 * F.guard + 1) * F.pitch)), dim3(256), 0,
                               stream, F, X);
        return hipGetLastError();
    };
    if (passes <= 2) {
        // rows 0 .. nr, columns 0 .. nth are read: copied in one run while the padding is a sixteenth at most
        // (2048 x 2048: 265 us a step, 268 row by row; with 2048 columns of padding 486, 272 row by row)
        const bool one = F.pitch <= F.nth + 1 + 2 * F.guard + F.nth / 16;
        const uint32_t runs = one ? 1u : (uint32_t)F.nr + 1u;
        const uint32_t width = one ? F.at(F.nr, F.nth) - F.at(0, 0) + 1u : (uint32_t)F.nth + 1u;
        hipLaunchKernelGGL(field_copy_kernel, dim3(nb((int64_t)runs * width)), dim3(256), 0, stream, F, W2, X, F.at(0, 0),
                           runs, width);
        S.last = 1;
        launch_passes<true>(passes, F, W2, R, X, S, stream);
        return finish();
    }
    const int launches = std::max(2, (passes + kMaxStages - 1) / kMaxStages);
    FieldPtrs cur = X;
    for (int g = 0; g < launches; ++g) {
        const int K = passes / launches + (g < passes % launches ? 1 : 0);
        S.last = g == launches - 1;
        S.store_R = 1;
        const FieldPtrs nxt = S.last ? X : (g % 2 == 0 ? W1 : W2);
        if (g == 0) launch_passes<true>(K, F, cur, R, nxt, S, stream);
        else launch_passes<false>(K, F, cur, R, nxt, S, stream);
        cur = nxt;
    }
    return finish();
}

}  // namespace grpic
