// Deflection angle with the potential from a table in LDS.
//
// The pair rule of chi_quad.hpp evaluates V(r) about a hundred times per pair
// (root scan, Newton, 64 nodes), and V of the JAGER form costs two
// exponentials and the Tang-Toennies sums: some 300 operations.  Here V is
// tabulated once per workgroup as a piecewise polynomial in w = 1/r (the
// nodes' own variable: w = w_min (1 - t^2), no division), and an evaluation
// is an index, one LDS read of the interval's coefficients and a short
// polynomial.
//
// Intervals: CT_LR equal ones on [0, 1/r_sw] for the dispersion branch (w = 0
// is r = infinity, V = 0), CT_SR on [1/r_sw, CT_SPAN/r_sw] for the screened
// Coulomb branch, direct evaluation beyond.  Degree 5 through six Chebyshev
// nodes in FP64; FP32 polynomials are the same ones cut to degree 3.
//
// In the first intervals V ~ w^6 falls below the table's error, which is an
// absolute one there (1e-17 K for the argon set), and the angle sees it divided
// by E.  Pairs below an energy that this error sets (e_far: 0.15 K, 11 m/s, for
// argon; one pair in 10^5 of a gas at 273 K) therefore take V at w < w_far from
// the dispersion sum itself (ct_slow_lane, in FP64, and their refinement):
// damping and repulsion are below rounding there, and the sum has V's relative
// accuracy down to w = 0.  Their angles keep the direct rule's error (at 1 mm/s
// and 100 nm 1e-16; 2e-8 by the table alone).  From e_far on the table's error,
// some roundings of V's terms, shows where the integrand is peaked: 1.5e-14 RMS
// at 10-30 m/s and 6e-15 at 600-5000 m/s against 4e-15 and 2e-15 (argon, pairs
// that are not refined; in FP32 5e-7 against 9e-7).  Taking the sum at all
// energies would cost the refinement 3 % of a batch's time.  Set-up measures
// both errors against the direct evaluation on the host; parameters that the
// intervals do not resolve keep the direct kernels.
#pragma once

#include "chi_quad.hpp"

namespace dsmc {

constexpr int CT_LR = 1024, CT_SR = 256, CT_N = CT_LR + CT_SR;
constexpr int CT_C = 6;             // FP64 coefficients per interval
constexpr int CT_CF = 4;            // FP32 coefficients per interval
constexpr double CT_SPAN = 4.0;     // the short-range intervals end at CT_SPAN / r_sw
constexpr double CT_FAR = 0.125;    // w_far is at most CT_FAR / r_sw

// Interpolation on [-1/2, 1/2]: nodes x and the matrix m that takes the values
// at the nodes to the coefficients of 1, x, .., x^(CT_C - 1).  (About the
// middle: on [0, 1] the coefficients are 30 times larger than the polynomial
// and their rounding, 2e-15 of V, doubled the error of pairs near orbiting.)
struct CtRule {
    double x[CT_C];
    double m[CT_C][CT_C];
};

// Position y in units of intervals: w inv_lr up to w_sw, w inv_sr + k_sr from
// there (the smaller of the two lines, as inv_sr < inv_lr).
struct CtScale {
    double w_sw, w_end, inv_lr, inv_sr, k_sr;
    double w_far;   // no damping (x >= DAMP_OFF) below
};

CQ_HD CtScale ct_scale(const Pot& P)
{
    CtScale s;
    s.w_sw = 1.0 / P.r_sw;
    s.w_end = CT_SPAN * s.w_sw;
    s.inv_lr = CT_LR * P.r_sw;
    s.inv_sr = CT_SR / ((CT_SPAN - 1.0) * s.w_sw);
    s.k_sr = CT_LR - s.w_sw * s.inv_sr;
    const double wd = P.p.beta_tt / DAMP_OFF, wm = CT_FAR * s.w_sw;
    s.w_far = wd < wm ? wd : wm;
    return s;
}

// The two branches of the JAGER form on their own (r >= r_sw and below).
// Where 1 - e^-x S_n cancels (x well below n) the damping factors come from
// the series tail, as the FP32 form of tt_disp takes them: the direct form's
// rounding, 1e-13 of V near r_sw, would reach the table's slopes.
CQ_HD double ct_far(const Pot& P, double w)
{
    const dsmc_potential& p = P.p;
    const double r = 1.0 / w, x = p.beta_tt * r, w2 = w * w;
    const double rep = p.A * exp(p.a1 * r + p.a2 * r * r + p.am1 * w + p.am2 * w2);
    double disp = 0.0;
    if (x >= TAIL_X) {
        double unused;
        tt_disp<double, false>(p, r, w, disp, unused);
        return rep - disp;
    }
    double e = exp(-x), f = 0.0, ef[6];
#pragma unroll
    for (int k = 1; k <= 16; ++k) {
        e *= x * (1.0 / k);
        if (k >= 6 && (k & 1) == 0) ef[(k - 6) / 2] = e;   // e^-x x^k / k!, k = 6, 8, .., 16
    }
#pragma unroll
    for (int k = 17; k <= 52; ++k) {   // (8/18) .. (8/52): the rest is below 1e-20 of f_16
        e *= x * (1.0 / k);
        f += e;
    }
    double wp = w2 * w2;
    wp *= wp;
    wp *= wp;                          // w^16
    const double r2 = r * r, w_x = 1.0 / x;
#pragma unroll
    for (int n = 5; n >= 0; --n) {
        disp += f * p.C[n] * wp;       // f = f_(6 + 2 n)
        f += ef[n] * (1.0 + (6 + 2 * n) * w_x);
        wp *= r2;
    }
    return rep - disp;
}
CQ_HD double ct_near(const Pot& P, double w) { return P.p.A_sr * w * exp(-P.p.a_sr / w); }

// Coefficients of interval i in x = y - (i + 1/2).  The values are taken
// relative to their mean before the matrix: the coefficients' rounding is then
// that of V's variation over one interval.
CQ_HD void ct_build(const Pot& P, const CtScale& s, const CtRule& r, int i, double (&c)[CT_C])
{
    double f[CT_C], mean = 0.0;
    for (int j = 0; j < CT_C; ++j) {
        if (i < CT_LR) f[j] = ct_far(P, (i + (0.5 + r.x[j])) / s.inv_lr);
        else f[j] = ct_near(P, s.w_sw + (i - CT_LR + (0.5 + r.x[j])) / s.inv_sr);
        mean += f[j];
    }
    mean *= 1.0 / CT_C;
    for (int k = 0; k < CT_C; ++k) {
        double a = 0.0;
        for (int j = 0; j < CT_C; ++j) a += r.m[k][j] * (f[j] - mean);
        c[k] = k == 0 ? a + mean : a;
    }
}

// The same polynomial cut to degree 3: interpolated at the four Chebyshev
// nodes of the interval (Newton's divided differences).
CQ_HD void ct_build_f32(const double (&c)[CT_C], float (&o)[CT_CF])
{
    const double x[4] = {-0.46193976625564337, -0.19134171618254489, 0.19134171618254489,
                         0.46193976625564337};   // -cos((2 j + 1) pi / 8) / 2
    double f[4];
    for (int j = 0; j < 4; ++j)   // without the constant term, whose rounding would spread
        f[j] = x[j] * (c[1] + x[j] * (c[2] + x[j] * (c[3] + x[j] * (c[4] + x[j] * c[5]))));
    for (int d = 1; d < 4; ++d)
        for (int j = 3; j >= d; --j) f[j] = (f[j] - f[j - 1]) / (x[j] - x[j - d]);
    // p = f0 + (x - x0)(f1 + (x - x1)(f2 + (x - x2) f3))
    double a0 = f[2] - x[2] * f[3], a1 = f[3];
    double b0 = f[1] - x[1] * a0, b1 = a0 - x[1] * a1, b2 = a1;
    o[0] = (float)(c[0] + (f[0] - x[0] * b0));
    o[1] = (float)(b0 - x[0] * b1);
    o[2] = (float)(b1 - x[0] * b2);
    o[3] = (float)b2;
}

// Potential and its table (c64 [CT_N][CT_C], c32 [CT_N][CT_CF]).
struct TabPot {
    Pot P;
    CtScale s;
    const double* c64;
    const float* c32;
};

// Interval and position in it, measured from its middle (0 <= w <= w_end).
template <typename T> CQ_HD int ct_index(const CtScale& s, T w, T& x)
{
    const T a = w * T(s.inv_lr), b = w * T(s.inv_sr) + T(s.k_sr);
    const T y = (a < b ? a : b) - T(0.5), r = rint(y);
    const T f = r < T(CT_N - 1) ? r : T(CT_N - 1);   // (w = w_end: the last interval's end)
    x = y - f;
    return (int)f;
}

// V at w < w_far, -sum C_n w^n, with its first and second derivative in w: a
// polynomial p in s = w^2 and its derivatives by Horner's scheme, V = -s^3 p.
CQ_HD double ct_tail(const dsmc_potential& p, double w, double& dVw, double& d2Vw)
{
    const double s = w * w;
    double v = 0.0, d = 0.0, e = 0.0;
#pragma unroll
    for (int k = 5; k >= 0; --k) {
        e = fma(e, s, d);
        d = fma(d, s, v);
        v = fma(v, s, p.C[k]);
    }
    const double s2 = s * s, d1 = s2 * fma(s, d, 3.0 * v);   // -dV/ds
    dVw = -2.0 * w * d1;
    d2Vw = -2.0 * (d1 + 4.0 * s2 * fma(s, fma(s, e, 3.0 * d), 3.0 * v));
    return -(s2 * s) * v;
}

// Which part of the range a caller can meet.  Below the orbiting energy (LOW)
// every root lies on the dispersion branch and every sample short of w_end, so
// the evaluation beyond the table and the pieces of a range across the meeting
// point are left out; SLOW: also the dispersion sum at w < w_far.  (With all of
// it in every copy the kernels had 83 to 93 KB of code instead of 58 to 67, and
// the step of 7 million particles took 1 189 us instead of 1 162.)
enum CtRange { CT_ALL, CT_LOW, CT_SLOW };

// V and (DERIV) dV/dw in FP64.
template <bool DERIV, CtRange RG = CT_ALL>
CQ_HD double ct_V(const TabPot& t, double w, double& dVw)
{
    if (RG == CT_SLOW && w < t.s.w_far) {
        double unused;
        return ct_tail(t.P.p, w, dVw, unused);
    }
    if (RG == CT_ALL && !(w <= t.s.w_end)) {
        const double V = ct_near(t.P, w);
        if (DERIV) dVw = V * (1.0 / w + t.P.p.a_sr / (w * w));
        return V;
    }
    double x;
    const int i = ct_index<double>(t.s, w, x);
    const double* c = t.c64 + i * CT_C;
    const double c0 = c[0], c1 = c[1], c2 = c[2], c3 = c[3], c4 = c[4], c5 = c[5];
    if (DERIV)
        dVw = (i < CT_LR ? t.s.inv_lr : t.s.inv_sr) *
              (c1 + x * (2.0 * c2 + x * (3.0 * c3 + x * (4.0 * c4 + x * (5.0 * c5)))));
    return c0 + x * (c1 + x * (c2 + x * (c3 + x * (c4 + x * c5))));
}

// V and (DERIV) dV/dw in FP32.
template <bool DERIV, CtRange RG = CT_ALL>
CQ_HD float ct_V(const TabPot& t, float w, float& dVw)
{
    static_assert(RG == CT_ALL, "slow pairs and the refinement are FP64");
    if (!(w <= float(t.s.w_end))) {
        const float V = float(t.P.p.A_sr) * w * expf(-float(t.P.p.a_sr) / w);
        if (DERIV) dVw = V * (1.0f / w + float(t.P.p.a_sr) / (w * w));
        return V;
    }
    float x;
    const int i = ct_index<float>(t.s, w, x);
    const float* c = t.c32 + i * CT_CF;
    const float c0 = c[0], c1 = c[1], c2 = c[2], c3 = c[3];
    if (DERIV)
        dVw = (i < CT_LR ? float(t.s.inv_lr) : float(t.s.inv_sr)) *
              (c1 + x * (2.0f * c2 + x * (3.0f * c3)));
    return c0 + x * (c1 + x * (c2 + x * c3));
}

template <typename T, CtRange RG = CT_ALL> CQ_HD T ct_value(const TabPot& t, T w)
{
    T unused;
    return ct_V<false, RG>(t, w, unused);
}

// V, dV/dw and d2V/dw2 in FP64, below the orbiting energy.
template <CtRange RG>
CQ_HD double ct_V2(const TabPot& t, double w, double& dVw, double& d2Vw)
{
    if (RG == CT_SLOW && w < t.s.w_far) return ct_tail(t.P.p, w, dVw, d2Vw);
    double x;
    const int i = ct_index<double>(t.s, w, x);
    const double inv = i < CT_LR ? t.s.inv_lr : t.s.inv_sr;
    const double* c = t.c64 + i * CT_C;
    const double c0 = c[0], c1 = c[1], c2 = c[2], c3 = c[3], c4 = c[4], c5 = c[5];
    dVw = inv * (c1 + x * (2.0 * c2 + x * (3.0 * c3 + x * (4.0 * c4 + x * (5.0 * c5)))));
    d2Vw = inv * inv * (2.0 * c2 + x * (6.0 * c3 + x * (12.0 * c4 + x * (20.0 * c5))));
    return c0 + x * (c1 + x * (c2 + x * (c3 + x * (c4 + x * c5))));
}

CQ_HD double cq_rsqrt(double x)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return rsqrt(x);
#else
    return 1.0 / sqrt(x);
#endif
}
CQ_HD float cq_rsqrt(float x)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_rsqf(x);
#else
    return 1.0f / sqrtf(x);
#endif
}

// What the scan and Newton's iteration leave.
template <typename T> struct CtRoot {
    T w;         // 1 / r_min
    T q0;        // r_min D'(r_min)
    T w_int;     // half-width estimate of an interior peak (1e30: none)
    bool flag;   // the root is left to the refinement
    bool done;   // no integral: a dip may reach zero (flagged)
    bool fail;   // the root search failed
};

// Largest root of D = 1 - b^2 w^2 - V(w)/E (smallest w), as chi_lane finds
// it, in w = 1/r.
template <typename T, CtRange RG = CT_ALL>
CQ_HD CtRoot<T> ct_root(const TabPot& t, const QuadCfg& q, T b, T E, bool low)
{
    CtRoot<T> R;
    R.q0 = T(0);
    R.w_int = T(1e30);
    R.flag = R.done = R.fail = false;
    const T b2 = b * b, iE = T(1) / E;
    const T rz = T(t.P.r_zero);
    const T r_top = b > rz ? b : rz;
    T w1 = T(1) / r_top;
    // At r = b > r_zero D is -V/E > 0, which the rounding of 1/b or, at w near 0,
    // of the table would hide for distant pairs; b - b keeps an infinite b's NaN.
    const T V1 = ct_value<T, RG>(t, w1);
    T f1 = b > rz ? (b - b) + fabs(V1) * iE : T(1) - b2 * (w1 * w1) - V1 * iE;
    if (f1 <= T(0)) {
        R.w = w1;
        R.flag = low;
        return R;
    }
    // the samples go on until D <= 0 or, below the orbiting energy, until they
    // have passed a local minimum of D (NaN ends them too)
    const T step = T(1) / (low ? T(q.scan_ratio) : T(0.7));
    T w0 = w1, f0 = low ? T(0) : T(-1e30), w2 = w1, f2 = f1;
    int it = 0;
    for (; it < 4000; ++it) {
        w2 = w1 * step;
        f2 = T(1) - b2 * (w2 * w2) - ct_value<T, RG>(t, w2) * iE;
        if (!(f2 > T(0)) || (f1 < f0 && f1 < f2) || w2 > T(1e4)) break;
        w0 = w1;
        f0 = low ? f1 : f0;
        w1 = w2;
        f1 = f2;
    }
    T wa = w1, wb = w2, ws = (-f2 < f1) ? w2 : w1;
    bool have_min = false;
    T pk_rm = T(0), pk_dm = T(0), pk_d2 = T(0);
    if (!(f2 <= T(0))) {
        if (!(f2 > T(0) && f1 < f0 && f1 < f2)) {
            R.w = w1;
            R.flag = low;
            R.fail = true;
            return R;
        }
        // a local minimum of D was passed: parabola through the samples (in r)
        const T r0 = T(1) / w0, r1 = T(1) / w1, r2 = T(1) / w2;
        const T h0 = r0 - r1, h2 = r1 - r2;
        const T s0 = (f0 - f1) / h0, s2 = (f1 - f2) / h2;
        const T d2 = T(2) * (s0 - s2) / (h0 + h2);
        const T d1 = s2 + T(0.5) * d2 * h2;
        const T dm = f1 - T(0.5) * d1 * d1 / d2;
        if (!(dm > T(LaneTol<T>::DM_MARGIN)) || !(d2 > T(0))) {
            R.w = w1;
            R.flag = R.done = true;   // a dip may reach zero: refinement
            return R;
        }
        // a positive minimum: the root is the inner one, inside r_zero
        have_min = true;
        pk_rm = r1 - d1 / d2;
        pk_dm = dm;
        pk_d2 = d2;
        wa = w2;
        wb = T(1) / rz;
        ws = wb;
    }
    // safeguarded Newton in [wa, wb], D(wa) > 0 >= D(wb)
    T w = ws, fp = T(0);
    for (int it = 0; it < q.max_iter; ++it) {
        T dV = T(0);
        const T V = ct_V<true, RG>(t, w, dV);
        const T f = T(1) - b2 * (w * w) - V * iE;
        if (f > T(0)) wa = w; else wb = w;
        fp = -T(2) * b2 * w - dV * iE;
        T wn = w - f / fp;
        if (!(wn > wa && wn < wb)) wn = T(0.5) * (wa + wb);
        const T dw = wn - w;
        w = wn;
        if (fabs(dw) <= Consts<T>::rtol * w || wb - wa <= Consts<T>::rtol * w) break;
    }
    R.w = w;
    R.q0 = -w * fp;
    if (have_min) {
        const T rmin = T(1) / w;
        const T ts2 = T(1) - rmin / pk_rm;
        const T ts = ts2 > T(0) ? sqrt(ts2) : T(0);
        const T om = T(1) - ts2;
        const T rp = T(2) * rmin * ts / (om * om);
        R.w_int = sqrt(T(2) * pk_dm / (pk_d2 * rp * rp + T(1e-30)));
    }
    return R;
}

// 2 t / sqrt(F) at t in (0, 1), F as in chi_quad.hpp with the potential
// difference near r_min as the integral of dV/dw (2-point Gauss-Legendre).
template <CtRange RG>
CQ_HD double ct_node(const TabPot& t, double w, double beta2, double Vmin, double iE, double tt,
                     double& smax, int& nonpos)
{
    const double g1 = 0.5 - 0.28867513459481287, g2 = 0.5 + 0.28867513459481287;
    const double t2 = tt * tt;
    const double u = 1.0 - t2;
    double dV;
    if (t2 < 1e-3) {
        const double h = w * t2, wsw = t.s.w_sw;
        double da, db;
        if (RG == CT_ALL && w > wsw && w - h < wsw) {
            // the two branches meet inside the step: each side on its own,
            // plus their (set-up) difference
            const double h1 = w - wsw, h2 = wsw - (w - h);
            const double over = wsw * (1.0 + Consts<double>::rtol);
            double dc, dd;
            const double wa = w - g1 * h1, wb = w - g2 * h1;
            ct_V<true, RG>(t, wa > over ? wa : over, da);
            ct_V<true, RG>(t, wb > over ? wb : over, db);
            ct_V<true, RG>(t, wsw - g1 * h2, dc);
            ct_V<true, RG>(t, wsw - g2 * h2, dd);
            dV = 0.5 * (h1 * (da + db) + h2 * (dc + dd)) + t.P.v_jump;
        } else {
            ct_V<true, RG>(t, w - g1 * h, da);
            ct_V<true, RG>(t, w - g2 * h, db);
            dV = 0.5 * h * (da + db);
        }
    } else {
        dV = Vmin - ct_value<double, RG>(t, w * u);
    }
    const double F = beta2 * (t2 * (2.0 - t2)) + dV * iE;
    if (!(F > 0.0)) {
        nonpos += 1;
        return 0.0;
    }
    const double s1 = 2.0 * tt * cq_rsqrt(F);
    smax = s1 > smax ? s1 : smax;
    return s1;
}

// The flags of chi_lane below the orbiting energy; peaked: the integrand's
// F / t^2 fell below QN_FLAG at a node, or F was not positive.
template <typename T> CQ_HD bool ct_peaked(const CtRoot<T>& R, bool peaked)
{
    return R.q0 < T(LaneTol<T>::Q0_FLAG) || R.q0 > T(LaneTol<T>::Q0_HIGH) || peaked ||
           R.w_int < T(LaneTol<T>::W_FLAG);
}

// Node constants of the whole range, the same for every pair: u = 1 - t^2 and
// the weight times 2 t.
struct CtNode {
    double u, wt;
};
// In FP32, u as a sum of two floats, so the interval and the position in it
// come out to FP32 rounding of the position (rounding w itself would move V
// by 15 times as much).
struct CtNodeF {
    float uh, ul, t2, wt;
};

// What the lane rule leaves: chi, or a pair for the workgroup to finish.
template <typename T> struct CtLane {
    T chi;
    bool flag;      // needs the FP64 refinement
    double kink_w;  // 1 / r_min of a pair whose range crosses the branches' meeting point (0: none);
                    // flagged as well, it is refined
};

// chi(b, E) as chi_lane gives it (b in Angstrom, E / k_B in K), FP64.
CQ_HD CtLane<double> chi_tab_lane(const TabPot& t, const QuadCfg& q, const GLRule& gl,
                                  const CtNode* __restrict__ nd, double b, double E)
{
    const double pi = Consts<double>::pi;
    CtLane<double> o{pi, false, 0.0};
    if (E == 0.0) {           // a pair at rest: the limit
        if (!(b < 1e300)) o.chi = NAN;
        return o;
    }
    const bool low = E < t.P.e_scan;
    const CtRoot<double> R = ct_root<double>(t, q, b, E, low);
    o.flag = R.flag;
    if (R.done || R.fail) {
        o.chi = R.done ? 0.0 : NAN;
        return o;
    }
    if (R.w > t.s.w_sw) {     // (below: the node loops index the dispersion branch)
        o.flag = o.flag || low;   // below e_scan an iteration that did not converge
        o.kink_w = R.w;
        return o;
    }
    const double beta = b * R.w, beta2 = beta * beta, iE = 1.0 / E;
    const double Vmin = ct_value<double>(t, R.w);
    const double y0 = R.w * t.s.inv_lr;
    constexpr double QN = LaneTol<double>::QN_FLAG;
    double I = 0.0, zmin = 1e300, fmin_ = 1e300;
    const double g1 = 0.5 - 0.28867513459481287, g2 = 0.5 + 0.28867513459481287;
    int k = 0;
    for (; k < gl.n && gl.t[k] * gl.t[k] < 1e-3; ++k) {
        // near r_min: V(r_min) - V(r) as the integral of the derivative
        const double t2 = gl.t[k] * gl.t[k];
        double d[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const double y = fma(-(e ? g2 : g1) * t2, y0, y0) - 0.5, f = rint(y), x = y - f;
            const int i = (int)f < CT_LR - 1 ? (int)f : CT_LR - 1;
            const double* c = t.c64 + i * CT_C;
            const double xx = i == (int)f ? x : x + 1.0;
            d[e] = c[1] + xx * (2.0 * c[2] + xx * (3.0 * c[3] + xx * (4.0 * c[4] + xx * (5.0 * c[5]))));
        }
        const double F = beta2 * (t2 * (2.0 - t2)) + 0.5 * (y0 * t2) * (d[0] + d[1]) * iE;
        const double z = F - QN * t2 + QN;
        zmin = z < zmin ? z : zmin;
        fmin_ = F < fmin_ ? F : fmin_;
        I += nd[k].wt * (F > 0.0 ? cq_rsqrt(F) : 0.0);
    }
#pragma unroll 2
    for (; k < gl.n; ++k) {
        const double u = nd[k].u;
        const double y = fma(y0, u, -0.5), f = rint(y), x = y - f;
        const double* c = t.c64 + (int)f * CT_C;
        const double V = fma(x, fma(x, fma(x, fma(x, fma(x, c[5], c[4]), c[3]), c[2]), c[1]), c[0]);
        const double F = fma(beta2, fma(-u, u, 1.0), (Vmin - V) * iE);
        const double z = fma(QN, u, F);
        zmin = z < zmin ? z : zmin;
        fmin_ = F < fmin_ ? F : fmin_;
        I = fma(nd[k].wt, F > 0.0 ? cq_rsqrt(F) : 0.0, I);
    }
    if (low && ct_peaked<double>(R, zmin < QN || !(fmin_ > 0.0))) o.flag = true;
    o.chi = pi - 2.0 * beta * I;
    return o;
}

// chi(b, E) with FP32 nodes.  The FP32 root is polished by one FP64 Newton
// step, and V(r_min), beta and the position of r_min in the table are taken
// in FP64 there.
CQ_HD CtLane<float> chi_tab_lane(const TabPot& t, const QuadCfg& q, const GLRule& gl,
                                 const CtNodeF* __restrict__ nd, double bd, double Ed)
{
    const float pi = Consts<float>::pi;
    CtLane<float> o{pi, false, 0.0};
    const float b = float(bd), E = float(Ed);
    const bool low = E < float(t.P.e_scan);
    if (E == 0.0f) {          // at rest (no FP32 result), or below FP32's range (the limit)
        if (!(Ed > 1e-300 && b < 1e30f)) o.chi = NAN;
        o.flag = low;
        return o;
    }
    const CtRoot<float> R = ct_root<float>(t, q, b, E, low);
    o.flag = R.flag;
    if (R.done || R.fail) {
        o.chi = R.done ? 0.0f : NAN;
        return o;
    }
    const double w0 = double(R.w);
    double dV, V = ct_V<true>(t, w0, dV);
    const double iEd = 1.0 / Ed;
    double w = w0 - (1.0 - bd * bd * (w0 * w0) - V * iEd) / (-2.0 * bd * bd * w0 - dV * iEd);
    if (!(fabs(w - w0) <= 1e-5 * w0)) {
        w = w0;
        if (low) o.flag = true;
    }
    if (w > t.s.w_sw) {
        o.flag = o.flag || low;
        o.kink_w = w;
        return o;
    }
    V = ct_value<double>(t, w);
    const float beta = float(bd * w), iE = float(iEd), Vmin = float(V), beta2 = beta * beta;
    float I = 0.0f, zmin = 1e30f, fmin_ = 1e30f;
    constexpr float QN = LaneTol<float>::QN_FLAG;
    const double y = w * t.s.inv_lr;
    const float yh = float(y), yl = float(y - double(yh));
    const float g1 = 0.5f - 0.28867513459481287f, g2 = 0.5f + 0.28867513459481287f;
    int k = 0;
    for (; k < gl.n && nd[k].t2 < 1e-3f; ++k) {
        // near r_min: V(r_min) - V(r) as the integral of the derivative
        const float t2 = nd[k].t2;
        float d[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const float off = (e ? g2 : g1) * t2;
            float f = rintf(__builtin_fmaf(-off, yh, yh) - 0.5f);
            f = f < CT_LR - 1 ? f : CT_LR - 1;
            const float x = __builtin_fmaf(-off, yh, yh - f) + (yl - 0.5f);
            const float* c = t.c32 + (int)f * CT_CF;
            d[e] = c[1] + x * (2.0f * c[2] + x * (3.0f * c[3]));
        }
        const float F = beta2 * (t2 * (2.0f - t2)) + 0.5f * yh * t2 * (d[0] + d[1]) * iE;
        const float z = F - QN * t2;
        zmin = z < zmin ? z : zmin;
        fmin_ = F < fmin_ ? F : fmin_;
        I += nd[k].wt * (F > 0.0f ? cq_rsqrt(F) : 0.0f);
    }
#pragma unroll 4
    for (; k < gl.n; ++k) {
        const CtNodeF v = nd[k];
        const float f = rintf(__builtin_fmaf(yh, v.uh, -0.5f));
        const float x = __builtin_fmaf(yh, v.uh, -f) +
                        __builtin_fmaf(yh, v.ul, __builtin_fmaf(yl, v.uh, -0.5f));
        const float* c = t.c32 + (int)f * CT_CF;
        const float c0 = c[0], c1 = c[1], c2 = c[2], c3 = c[3];
        const float Vk = __builtin_fmaf(x, __builtin_fmaf(x, __builtin_fmaf(x, c3, c2), c1), c0);
        const float F = __builtin_fmaf(beta2, v.t2 * (2.0f - v.t2), (Vmin - Vk) * iE);
        const float z = __builtin_fmaf(-QN, v.t2, F);
        zmin = z < zmin ? z : zmin;
        fmin_ = F < fmin_ ? F : fmin_;
        I = __builtin_fmaf(v.wt, F > 0.0f ? cq_rsqrt(F) : 0.0f, I);
    }
    if (low && ct_peaked<float>(R, zmin < 0.0f || !(fmin_ > 0.0f))) o.flag = true;
    o.chi = pi - 2.0f * beta * I;
    return o;
}

// chi of a slow pair (0 < E < e_far) by the lane rule in FP64.
CQ_HD CtLane<double> ct_slow_lane(const TabPot& t, const QuadCfg& q, const GLRule& gl, double b,
                                  double E)
{
    CtLane<double> o{0.0, false, 0.0};
    const CtRoot<double> R = ct_root<double, CT_SLOW>(t, q, b, E, true);
    o.flag = R.flag || R.w > t.s.w_sw;
    if (R.done || R.fail) {
        o.chi = R.done ? 0.0 : NAN;
        return o;
    }
    const double beta = b * R.w, beta2 = beta * beta, iE = 1.0 / E;
    const double Vmin = ct_value<double, CT_SLOW>(t, R.w);
    double I = 0.0, smax = 0.0;
    int nonpos = 0;
#pragma unroll 1
    for (int k = 0; k < gl.n; ++k)
        I += gl.w[k] * ct_node<CT_SLOW>(t, R.w, beta2, Vmin, iE, gl.t[k], smax, nonpos);
    if (ct_peaked<double>(R, smax * smax * LaneTol<double>::QN_FLAG > 4.0 || nonpos > 0))
        o.flag = true;
    o.chi = Consts<double>::pi - 2.0 * beta * I;
    return o;
}

// Node m (0 <= m < 2 n) of a pair whose range crosses the branches' meeting
// point, a kink of the integrand: n nodes on either side of it.
CQ_HD double ct_kink_node(const TabPot& t, const GLRule& gl, double w, double beta, double Vmin,
                          double iE, double tsw, int m)
{
    const int k = m < gl.n ? m : m - gl.n;
    const double ta = m < gl.n ? tsw : 0.0, len = m < gl.n ? 1.0 - tsw : tsw;
    double smax = 0.0;
    int nonpos = 0;
    return gl.w[k] * len *
           ct_node<CT_ALL>(t, w, beta * beta, Vmin, iE, ta + len * gl.t[k], smax, nonpos);
}

// ------------------------------------------------------------------------
// Host-side set-up
// ------------------------------------------------------------------------
inline void make_ct_rule(CtRule* r)
{
    const long double pi = 3.14159265358979323846264338327950288L;
    long double x[CT_C];
    for (int j = 0; j < CT_C; ++j) x[j] = -0.5L * cosl((2 * j + 1) * pi / (2 * CT_C));
    for (int j = 0; j < CT_C; ++j) {
        // Lagrange polynomial of node j, expanded
        long double p[CT_C] = {1.0L}, den = 1.0L;
        int deg = 0;
        for (int i = 0; i < CT_C; ++i) {
            if (i == j) continue;
            den *= x[j] - x[i];
            for (int k = deg + 1; k > 0; --k) p[k] = p[k - 1] - x[i] * p[k];
            p[0] = -x[i] * p[0];
            ++deg;
        }
        for (int k = 0; k < CT_C; ++k) r->m[k][j] = (double)(p[k] / den);
        r->x[j] = (double)x[j];
    }
}

inline void make_ct_nodes(const GLRule& gl, CtNode* nd)
{
    for (int k = 0; k < gl.n; ++k) nd[k] = CtNode{1.0 - gl.t[k] * gl.t[k], 2.0 * gl.t[k] * gl.w[k]};
}
inline void make_ct_nodes(const GLRule& gl, CtNodeF* nd)
{
    for (int k = 0; k < gl.n; ++k) {
        const double u = 1.0 - gl.t[k] * gl.t[k];
        nd[k].uh = (float)u;
        nd[k].ul = (float)(u - (double)nd[k].uh);
        nd[k].t2 = (float)(gl.t[k] * gl.t[k]);
        nd[k].wt = (float)(2.0 * gl.t[k] * gl.w[k]);
    }
}

// Whether the table kernels take the potential: below the orbiting energy
// every root lies on the dispersion branch, and the table resolves V.  That is,
// at points between the interpolation nodes of every interval, within 2e-14 of
// the direct value relative to its terms' magnitude (the argon set: 4e-15).
// Where slow pairs are on the long-range side of that, 1e-12 does (the angle's
// own bound is 1e-9): of the dispersion sum at w < w_far (the argon set: 4e-16;
// shorter ranges of the damping leave more repulsion there) and of the table
// just above (longer ones bring w_far down).  The table's absolute error at these points sets *e_far, the
// energy from which it moves F = D(r(t)) by less than 2e-16 (twice the largest
// error found over 2e-16).
constexpr double CT_E_FAR = 0.05;   // most of the orbiting energy that e_far may be
inline bool ct_resolves(const Pot& P, const CtRule& rule, double* e_far)
{
    if (P.p.kind != DSMC_POT_JAGER || !(P.r_floor > 1.01 * P.r_sw)) return false;
    const CtScale s = ct_scale(P);
    double far_err = 0.0;
    for (int i = 0; i < CT_N; ++i) {
        double c[CT_C];
        ct_build(P, s, rule, i, c);
        for (int m = 0; m < 4; ++m) {
            const double x = -0.4 + 0.25 * m, k = (i < CT_LR ? i : i - CT_LR) + (0.5 + x);
            const double w = i < CT_LR ? k / s.inv_lr : s.w_sw + k / s.inv_sr;
            const double V = i < CT_LR ? ct_far(P, w) : ct_near(P, w);
            const double t = c[0] + x * (c[1] + x * (c[2] + x * (c[3] + x * (c[4] + x * c[5]))));
            double mag = fabs(V), d, e;
            if (i < CT_LR) {
                const double r = 1.0 / w;
                mag += 2.0 * P.p.A * exp(P.p.a1 * r + P.p.a2 * r * r + P.p.am1 * w + P.p.am2 * w * w);
            }
            if (w < s.w_far && !(fabs(ct_tail(P.p, w, d, e) - V) <= 1e-12 * mag)) return false;
            const double err = fabs(t - V);
            if (err <= 2e-14 * mag) continue;
            if (i >= CT_LR || !(w < s.w_far || err <= 1e-12 * mag)) return false;
            if (!(err <= far_err)) far_err = err;
        }
    }
    *e_far = 1e16 * far_err;
    return *e_far <= CT_E_FAR * P.e_scan;
}

}  // namespace dsmc
