// Helix-fit arithmetic shared by the forward fit and its adjoint.
//
// State p = (y, z, s = sin phi, t = tan lambda, w = q/pT) on a pad-row plane
// x, track oriented towards +x, curvature kappa = -c Bz w (counter-clockwise
// positive); covariance as the 15 entries of its lower triangle.
//
// Precision.  The forward filter (state, helix transport, Jacobian,
// covariance transport F C F^T and Kalman update) runs in the type R, double
// in the library: a short track's curvature is fixed by sub-micron
// sagittas, so single-precision transport of y alone moves q/pT by ~1e-4
// relative, and a single-precision covariance update loses up to all
// significant digits when the diffuse start covariance collapses onto the
// first hits (C - K H C cancels).  On gfx950 the FP64 vector FMA issues at the
// rate of the non-packed FP32 one, so double costs no more than float here.
// Reciprocals and square roots in the inner loop use the hardware estimates
// refined by Newton steps rather than the correctly rounded sequences.  So
// does the adjoint, with the second-order term (derivative of the Jacobian)
// in the closed forms that follow from the step's.
// No MFMA: a 5x5 symmetric update is not a dense contraction.
#pragma once

#include <hip/hip_runtime.h>

#define TPC_C_LIGHT 0.00299792458f

template <class R>
struct SymT {
    // lower triangle, row by row: 00 10 11 20 21 22 30 31 32 33 40 41 42 43 44
    R c00, c10, c11, c20, c21, c22, c30, c31, c32, c33, c40, c41, c42, c43, c44;
};

// Jacobian entries that differ from the identity.
struct StepJac {
    double f02, f04, f12, f13, f14, f24;
};

// What the derivatives of the Jacobian use of a step: 1/c, 1/c', T, 1/(c + c').
template <class R>
struct StepTrig {
    R ic1, ic2, T, iden;
};

// Reciprocal and square root of positive, finite, normal doubles for the
// filter's inner loop.  On the device: the hardware estimates refined by
// Newton-Raphson (reciprocal, two steps) and by one step of third order (the
// inverse square root) with a Newton correction of the root; within a few
// units of rounding, but not correctly rounded.  On the host: the library
// operations.
__host__ __device__ inline double recip_pos(double x) {
#if defined(__HIP_DEVICE_COMPILE__)
    double r = __builtin_amdgcn_rcp(x);
    double e = fma(-x, r, 1.0);
    r = fma(r, e, r);
    e = fma(-x, r, 1.0);
    return fma(r, e, r);
#else
    return 1.0 / x;
#endif
}

// sqrt(x), and 1/sqrt(x) in *inv.
__host__ __device__ inline double sqrt_pos(double x, double *inv) {
#if defined(__HIP_DEVICE_COMPILE__)
    const double y0 = __builtin_amdgcn_rsq(x);
    const double e = fma(-(x * y0), y0, 1.0);
    const double y = fma(y0 * e, fma(e, 0.375, 0.5), y0);
    const double g = x * y, d = fma(-g, g, x);
    if (inv) *inv = y;
    return fma(d, 0.5 * y, g);
#else
    const double g = sqrt(x);
    if (inv) *inv = 1.0 / g;
    return g;
#endif
}

// asin(u)/u = sum of a_k x^k, x = u^2, to x^N: the sum (g) and its derivative
// in x (d), so that the derivative in u is 2 u d.  What is left out is below
// 1e-17 and 7e-14 of them for N = 5, |u| < 0.05 (and below rounding at 0.025),
// below 1e-17 and 1e-16 for N = 10, |u| < 0.15.
// (e: half the second derivative, to x^(N - 2), if asked for.)
template <int N, class R>
__host__ __device__ inline void asin_series(R x, R &g, R &d, R *e = nullptr) {
    constexpr R a[14] = {1.0, 1.0 / 6, 3.0 / 40, 5.0 / 112, 35.0 / 1152, 63.0 / 2816, 231.0 / 13312, 143.0 / 10240,
                         6435.0 / 557056, 12155.0 / 1245184, 46189.0 / 5505024, 88179.0 / 12058624,
                         676039.0 / 104857600, 1300075.0 / 226492416};
    static_assert(N < 14, "coefficients");
    d = a[N];
    g = fma(a[N], x, a[N - 1]);
    if (e) *e = (R)0;
#pragma unroll
    for (int k = N - 2; k >= 0; --k) {
        if (e) *e = k == N - 2 ? d : fma(*e, x, d);
        d = fma(d, x, g);
        g = fma(g, x, a[k]);
    }
}

// asin(u)/u for |u| >= 0.05: asin(u) = 2 asin(u / sqrt(2 (1 + sqrt(1 - u^2))))
// until the series to u^2N holds (N = 13: below 0.25, three times at most; N =
// 5: below 0.05, five times; NaN beyond 1).  Rarely taken; a call of the
// library's asin made every fit keep what lives across it in the registers
// that calls leave alone.
template <int N = 13>
__host__ __device__ inline double asin_over_far(double u) {
    static_assert(N == 13 || N == 5, "where the series holds");
    double v = u, k = 1.0;
    while (fabs(v) >= (N == 13 ? 0.25 : 0.05)) {
        double h;
        sqrt_pos(2.0 + 2.0 * sqrt_pos((1.0 - v) * (1.0 + v), nullptr), &h);
        v *= h;
        k += k;
    }
    double g, d;
    asin_series<N>(v * v, g, d);
    return k * v * g / u;
}
// asin(u)/u in the state precision
template <int N = 13, class R>
__host__ __device__ inline R asin_over_r(R u) {
    if (fabs(u) < (R)0.05) {
        R g, d;
        asin_series<5>(u * u, g, d);
        return g;
    }
    return (R)asin_over_far<N>((double)u);
}

// Exact helix step from x to x + dx, state and Jacobian in precision R
// (double in the library: on gfx950 the FP64 vector FMA issues at the rate
// of the non-packed FP32 one, so a single-precision Jacobian would only add
// conversions).  Returns false when |sin phi| reaches max_sin before or
// after the step; the step is evaluated regardless (no early exit keeps the
// filter loop free of branches), so p and J are then meaningless.
// The plane distance dx and kbz = -c Bz come in precision K: single in the
// fit (adjacent planes), double where steps cross several planes.
//
// The filters are bound by this step's instructions (one wavefront per SIMD,
// every instruction of the chain counts), so it is written with few of them.
// With s' = s + kappa dx, cosines c, c', T = (s + s')/(c + c') and
// B = c + s T (= c' + s' T), the turned angle delta has sin delta =
// s'c - s c' = kappa dx B, so the path is dx B asin(v)/v with v = sin delta
// (no chord length), and the partial derivatives are
//   dT/ds = B/(c c'),            dT/dkappa = dx B / ((c + c') c'),
//   darc/ds = (1/c' - 1/c)/kappa = dx T/(c c'),
//   darc/dkappa = dx s dT/dkappa / cos delta + (dx B)^2 g'(v),
// g = asin(v)/v, 1/cos delta = g + v g'.  Turns of |v| >= 0.05 (and beyond 90
// degrees, where v falls again) take the half angle u = sin(delta/2) =
// kappa chord/2: arc = chord g(u), darc/dkappa = dx^2 T/((c + c') c') +
// chord^2 g'(u)/2, with 1/cos(delta/2) = chord/(dx B) in g'.  (A track's
// outermost steps may turn by 0.2, where it runs along the pad row: a series
// to u^20, short, as a wavefront takes it when one of its tracks does.  MID =
// 5 where its coefficients would take registers that are not there.)
template <class R, class K = float, int MID = 10>
__host__ __device__ inline bool helix_step(R p[5], K dx, K kbz, float max_sin, StepJac &J,
                                           StepTrig<R> *trig = nullptr) {
    // kbz = -c Bz, so kappa = kbz * w
    const R s = p[2], t = p[3], w = p[4], d = (R)dx, kb = (R)kbz;
    const R kap = kb * w, kd = kap * d;
    const R s2 = fma(kap, d, s);
    const bool ok = fabs(s) < (R)max_sin && fabs(s2) < (R)max_sin;
    R ic1, ic2;
    const R c1 = sqrt_pos(fma(-s, s, (R)1), &ic1);
    const R c2 = sqrt_pos(fma(-s2, s2, (R)1), &ic2);
    const R den = c1 + c2;
    const R iden = recip_pos(den);
    const R T = (s + s2) * iden;                  // tan of the chord direction
    const R B = c1 + s * T;
    const R dB = d * B, v = kd * B;
    const R dTk = dB * iden * ic2;                // dT/dkappa
    const R cc = ic1 * ic2;
    R arc, dark;                                  // signed transverse path length, darc/dkappa
    // (a turn of 90 degrees or more changes s by at least 1)
    if (fabs(v) < (R)0.05 && fabs(kd) < (R)1) {
        const R v2 = v * v;
        R g, h;
        asin_series<5>(v2, g, h);
        h += h;
        arc = dB * g;
        dark = d * s * dTk * fma(v2, h, g) + dB * dB * (v * h);
    } else {
        const R chord = d * sqrt_pos(fma(T, T, (R)1), nullptr);   // signed
        const R u = (R)0.5 * kap * chord;
        dark = (d * iden) * (d * ic2) * T;
        R g, h;
        if (fabs(u) < (R)(MID == 10 ? 0.15 : 0.05)) {
            asin_series<MID>(u * u, g, h);
            dark = fma(chord * chord, u * h, dark);
        } else {
            g = asin_over_far<MID == 10 ? 13 : 5>(u);
            dark += chord * (chord / dB - g) / kap;
        }
        arc = chord * g;
    }
    if (trig) *trig = StepTrig<R>{ic1, ic2, T, iden};
    J.f02 = dB * cc;
    J.f04 = d * kb * dTk;
    J.f12 = t * (d * T * cc);
    J.f13 = arc;
    J.f14 = t * (kb * dark);
    J.f24 = d * kb;
    p[0] += d * T;
    p[1] += t * arc;
    p[2] = s2;
    return ok;
}

// Symmetric transport with the sparse step Jacobian F = I + N:
//   transposed == false:  C <- F C F^T
//   transposed == true:   C <- F^T C F
template <class R, bool transposed>
__host__ __device__ inline void sym_transport(SymT<R> &C, const StepJac &J) {
    const R f02 = J.f02, f04 = J.f04, f12 = J.f12, f13 = J.f13, f14 = J.f14, f24 = J.f24;
    const R C00 = C.c00, C01 = C.c10, C02 = C.c20, C03 = C.c30, C04 = C.c40;
    const R C11 = C.c11, C12 = C.c21, C13 = C.c31, C14 = C.c41;
    const R C22 = C.c22, C23 = C.c32, C24 = C.c42;
    const R C33 = C.c33, C34 = C.c43, C44 = C.c44;
    if (!transposed) {
        // A = F C: rows 0..2 change, rows 3, 4 are those of C
        const R A00 = C00 + f02 * C02 + f04 * C04;
        const R A02 = C02 + f02 * C22 + f04 * C24;
        const R A04 = C04 + f02 * C24 + f04 * C44;
        const R A10 = C01 + f12 * C02 + f13 * C03 + f14 * C04;
        const R A11 = C11 + f12 * C12 + f13 * C13 + f14 * C14;
        const R A12 = C12 + f12 * C22 + f13 * C23 + f14 * C24;
        const R A13 = C13 + f12 * C23 + f13 * C33 + f14 * C34;
        const R A14 = C14 + f12 * C24 + f13 * C34 + f14 * C44;
        const R A20 = C02 + f24 * C04;
        const R A22 = C22 + f24 * C24;
        const R A24 = C24 + f24 * C44;
        // C' = A F^T
        C.c00 = A00 + f02 * A02 + f04 * A04;
        C.c10 = A10 + f02 * A12 + f04 * A14;
        C.c11 = A11 + f12 * A12 + f13 * A13 + f14 * A14;
        C.c20 = A20 + f02 * A22 + f04 * A24;
        C.c21 = (C12 + f24 * C14) + f12 * A22 + f13 * (C23 + f24 * C34) + f14 * A24;
        C.c22 = A22 + f24 * A24;
        C.c30 = C03 + f02 * C23 + f04 * C34;
        C.c31 = C13 + f12 * C23 + f13 * C33 + f14 * C34;
        C.c32 = C23 + f24 * C34;
        C.c40 = C04 + f02 * C24 + f04 * C44;
        C.c41 = C14 + f12 * C24 + f13 * C34 + f14 * C44;
        C.c42 = C24 + f24 * C44;
        // c33, c43, c44 unchanged
    } else {
        // Q = C F: columns 2..4 change (col2 += f02 col0 + f12 col1,
        // col3 += f13 col1, col4 += f04 col0 + f14 col1 + f24 col2)
        // then C' = F^T Q: rows change the same way.
        const R Q02 = C02 + f02 * C00 + f12 * C01;
        const R Q12 = C12 + f02 * C01 + f12 * C11;
        const R Q22 = C22 + f02 * C02 + f12 * C12;
        const R Q32 = C23 + f02 * C03 + f12 * C13;
        const R Q42 = C24 + f02 * C04 + f12 * C14;
        const R Q03 = C03 + f13 * C01;
        const R Q13 = C13 + f13 * C11;
        const R Q23 = C23 + f13 * C12;
        const R Q33 = C33 + f13 * C13;
        const R Q43 = C34 + f13 * C14;
        const R Q04 = C04 + f04 * C00 + f14 * C01 + f24 * C02;
        const R Q14 = C14 + f04 * C01 + f14 * C11 + f24 * C12;
        const R Q24 = C24 + f04 * C02 + f14 * C12 + f24 * C22;
        const R Q34 = C34 + f04 * C03 + f14 * C13 + f24 * C23;
        const R Q44 = C44 + f04 * C04 + f14 * C14 + f24 * C24;
        // rows 0, 1 of F^T Q are rows 0, 1 of Q
        C.c20 = Q02;
        C.c21 = Q12;
        C.c22 = Q22 + f02 * Q02 + f12 * Q12;
        C.c30 = Q03;
        C.c31 = Q13;
        C.c32 = Q23 + f02 * Q03 + f12 * Q13;
        C.c33 = Q33 + f13 * Q13;
        C.c40 = Q04;
        C.c41 = Q14;
        C.c42 = Q24 + f02 * Q04 + f12 * Q14;
        C.c43 = Q34 + f13 * Q14;
        C.c44 = Q44 + f04 * Q04 + f14 * Q14 + f24 * Q24;
        (void)Q32; (void)Q42; (void)Q43;
        // c00, c10, c11 unchanged
    }
}

// Kalman update with measurement (my, mz), in two halves: kalman_gain forms
// the gain K = C H^T S^-1 from the predicted covariance, updates the state
// and returns the chi2 increment (negative if the residual covariance is not
// positive definite; everything is evaluated regardless, and p, C are then
// meaningless); kalman_cov applies C -= K H C.  The filter loop runs the
// covariance half of one step next to the helix step of the next, which
// does not need it.  Columns 0 and 1 of the updated covariance are K V, V =
// diag(vy, vz): C - K (S - V) = K V there, one product instead of two
// multiply-adds and no cancellation.  The other six entries need K and the
// rows H C, kept in a Gain.
template <class R>
struct Gain {
    R k00, k10, k11, k20, k21, k30, k31, k40, k41;   // K (k01 = k10 vy / vz is not used)
    R r02, r03, r04, r12, r13, r14;                   // rows 0 and 1 of C
    // the gain that leaves diag(vy, vz, *, *, *) as it is
    __host__ __device__ static Gain none() {
        Gain g = {};
        g.k00 = g.k11 = (R)1;
        return g;
    }
};

template <class R>
__host__ __device__ inline R kalman_gain(R p[5], const SymT<R> &C, R my, R mz, R vy, R vz, Gain<R> &G) {
    const R r0 = my - p[0], r1 = mz - p[1];
    const R S00 = C.c00 + vy, S01 = C.c10, S11 = C.c11 + vz;
    const R det = S00 * S11 - S01 * S01;
    const bool pd = det > (R)0;
    const R idet = recip_pos(det);
    const R i00 = S11 * idet, i01 = -S01 * idet, i11 = S00 * idet;
    // p += C[:, 0:2] S^-1 r
    const R a0 = i00 * r0 + i01 * r1, a1 = i01 * r0 + i11 * r1;
    p[0] = p[0] + C.c00 * a0 + C.c10 * a1;
    p[1] = p[1] + C.c10 * a0 + C.c11 * a1;
    p[2] = p[2] + C.c20 * a0 + C.c21 * a1;
    p[3] = p[3] + C.c30 * a0 + C.c31 * a1;
    p[4] = p[4] + C.c40 * a0 + C.c41 * a1;
    // K = C[:, 0:2] S^-1
    G.k00 = C.c00 * i00 + C.c10 * i01;
    G.k10 = C.c10 * i00 + C.c11 * i01; G.k11 = C.c10 * i01 + C.c11 * i11;
    G.k20 = C.c20 * i00 + C.c21 * i01; G.k21 = C.c20 * i01 + C.c21 * i11;
    G.k30 = C.c30 * i00 + C.c31 * i01; G.k31 = C.c30 * i01 + C.c31 * i11;
    G.k40 = C.c40 * i00 + C.c41 * i01; G.k41 = C.c40 * i01 + C.c41 * i11;
    G.r02 = C.c20; G.r03 = C.c30; G.r04 = C.c40;
    G.r12 = C.c21; G.r13 = C.c31; G.r14 = C.c41;
    const R chi = r0 * a0 + r1 * a1;
    return pd ? chi : (R)-1;
}

// C -= K H C for the gain G of a measurement with variances vy, vz
template <class R>
__host__ __device__ inline void kalman_cov(SymT<R> &C, const Gain<R> &G, R vy, R vz) {
    C.c00 = G.k00 * vy;
    C.c10 = G.k10 * vy;
    C.c11 = G.k11 * vz;
    C.c20 = G.k20 * vy;
    C.c21 = G.k21 * vz;
    C.c22 = C.c22 - G.k20 * G.r02 - G.k21 * G.r12;
    C.c30 = G.k30 * vy;
    C.c31 = G.k31 * vz;
    C.c32 = C.c32 - G.k30 * G.r02 - G.k31 * G.r12;
    C.c33 = C.c33 - G.k30 * G.r03 - G.k31 * G.r13;
    C.c40 = G.k40 * vy;
    C.c41 = G.k41 * vz;
    C.c42 = C.c42 - G.k40 * G.r02 - G.k41 * G.r12;
    C.c43 = C.c43 - G.k40 * G.r03 - G.k41 * G.r13;
    C.c44 = C.c44 - G.k40 * G.r04 - G.k41 * G.r14;
}

template <class R>
__host__ __device__ inline R kalman_update(R p[5], SymT<R> &C, R my, R mz, R vy, R vz) {
    Gain<R> G;
    const R chi = kalman_gain(p, C, my, mz, vy, vz, G);
    kalman_cov(C, G, vy, vz);
    return chi;
}

// Exact circle through C (innermost), B, A (outermost): state at A, computed
// in precision R.  Returns false if the points are degenerate or the
// direction at A is not towards +x with |sin phi| < max_sin.
template <class R, class K = float>
__host__ __device__ inline bool helix_start(R xa, R ya, R za, R xb, R yb, R xc, R yc, R zc,
                                            K kbz, float max_sin, R p[5]) {
    const R bcx = xb - xc, bcy = yb - yc;
    const R abx = xa - xb, aby = ya - yb;
    const R acx = xa - xc, acy = ya - yc;
    const R lbc = sqrt(bcx * bcx + bcy * bcy);
    const R lab = sqrt(abx * abx + aby * aby);
    const R lac = sqrt(acx * acx + acy * acy);
    const R prod = lbc * lab * lac;
    const R cross = bcx * aby - bcy * abx;
    if (!(prod > (R)0)) return false;
    const R kap = (R)2 * cross / prod;
    const R ua = (R)0.5 * kap * lab, uc = (R)0.5 * kap * lac;
    if (!(fabs(ua) < (R)1) || !(fabs(uc) < (R)1)) return false;
    // direction at A: chord angle plus half the turning angle over B -> A,
    // whose sine is ua (the sum's sine and cosine without the angles)
    const R ca = sqrt(((R)1 - ua) * ((R)1 + ua)), ilab = (R)1 / lab;
    const R sn = (aby * ca + abx * ua) * ilab, cs = (abx * ca - aby * ua) * ilab;
    if (!(cs > (R)0) || !(fabs(sn) < (R)max_sin)) return false;
    p[0] = ya;
    p[1] = za;
    p[2] = sn;
    p[3] = (za - zc) / (lac * asin_over_r(uc));
    p[4] = kap / (R)kbz;          // w = -kappa / (c Bz) = kappa / kbz
    return true;
}

// ---------------------------------------------------------------------------
// Adjoint (reverse mode), written out by hand.  A symmetric matrix argument
// has a symmetric adjoint Mbar with dL = <Mbar, dM> for symmetric dM.

// d<G, F(p)>/dp for p = (s, t, w) of the state a step of Jacobian F starts
// from: the second partial derivatives of (T, arc) of helix_step.  With
// cc = 1/(c c') and the logarithmic derivatives of cc, 1/c' and 1/(c + c'),
//   d2T/ds2 = cc (dB/ds + B (s/c^2 + s'/c'^2)),   dB/ds = T + s dT/ds - s/c,
//   d2T/dsdk = cc (s dT/dk + B dx s'/c'^2),
//   d2T/dk2 = dT/dk dx/c' (T + s'/c'),
//   d2arc/ds2 = dx cc (dT/ds + T (s/c^2 + s'/c'^2)),
//   d2arc/dsdk = dx cc (dT/dk + T dx s'/c'^2),
// and d2arc/dk2 from arc = dB g(v), v = kappa dB, dB = dx B (near), or from
// darc/dk = (dx/c' - arc)/kappa (far; the same limit as helix_step's).
template <class R, class K>
__host__ __device__ inline void helix_jac_adjoint(const R p[5], K dx, K kbz, R arc, const StepTrig<R> &q, R G02, R G04,
                                                  R G12, R G13, R G14, R &bs, R &bt, R &bw) {
    const R s = p[2], t = p[3], d = (R)dx, kb = (R)kbz, kap = kb * p[4], kd = kap * d;
    const R s2 = fma(kap, d, s), T = q.T;
    const R u1 = s * q.ic1, u2 = s2 * q.ic2;            // s/c, s'/c'
    const R B = fma(-s, s, (R)1) * q.ic1 + s * T;
    const R cc = q.ic1 * q.ic2, dB = d * B, v = kd * B;
    const R Ts = B * cc, Tk = dB * q.iden * q.ic2;
    const R l1 = u1 * q.ic1 + u2 * q.ic2, l2 = d * u2 * q.ic2;   // d ln cc/ds, d ln cc/dkappa
    const R Tss = cc * (T + s * Ts - u1 + B * l1);
    const R Tsk = cc * (s * Tk + B * l2);
    const R Tkk = Tk * (d * q.ic2) * (T + u2);
    const R dcc = d * cc;
    const R as = dcc * T, ass = dcc * (Ts + T * l1), ask = dcc * (Tk + T * l2);
    R ak, akk;
    if (fabs(v) < (R)0.05 && fabs(kd) < (R)1) {
        const R v2 = v * v;
        R g, h, hh;
        asin_series<5>(v2, g, h, &hh);
        const R gd = (R)2 * v * h, gdd = (R)2 * h + (R)8 * v2 * hh;
        const R Bk = d * s * Tk, Bkk = d * s * Tkk;     // of dB
        const R vk = dB + kap * Bk, vkk = (R)2 * Bk + kap * Bkk;
        ak = Bk * g + dB * gd * vk;
        akk = Bkk * g + (R)2 * Bk * gd * vk + dB * (gdd * vk * vk + gd * vkk);
    } else {
        const R ik = (R)1 / kap;
        ak = (d * q.ic2 - arc) * ik;
        akk = (d * l2 * q.ic2 - (R)2 * ak) * ik;
    }
    const R G4 = G04 * kb, G14t = G14 * t * kb;
    bs = d * (G02 * Tss + G4 * Tsk) + G12 * t * ass + G13 * as + G14t * ask;
    bw = kb * (d * (G02 * Tsk + G4 * Tkk) + G12 * t * ask + G13 * ak + G14t * akk);
    bt = G12 * as + G14 * kb * ak;
}

// Reverse of one filter step (propagate by dx, then update with (my, mz)).
// In: the state (pb, Cb) the step started from, the adjoints (pbar, Cbar)
// of its result, chibar = dL/dchi2.  Out: pbar, Cbar become the adjoints of
// (pb, Cb); (mby, mbz) receive dL/d(my, mz).
//
// The update from the propagated (x, P): with K its gain, A = I - K H and
// a = S^-1 r, dC = A dP A^T, dx' = A (dx + dP H^T a) + K dm and dchi2 =
// 2 a^T dr - a^T H dP H^T a, so
//   Pbar = A^T Cbar A + sym(A^T pbar (H^T a)^T) - chibar (H^T a)(H^T a)^T,
//   mbar = 2 chibar a + K^T pbar,  xbar = pbar - H^T mbar,
// where A^T Cbar A differs from Cbar in rows and columns 0 and 1 only.
template <class R>
__host__ __device__ inline void step_adjoint(const R pb[5], const SymT<R> &Cb, float dx, float kbz,
                                             R my, R mz, R vy, R vz, R chibar, R pbar[5],
                                             SymT<R> &Cbar, R &mby, R &mbz) {
    // recompute the step
    R pp[5] = {pb[0], pb[1], pb[2], pb[3], pb[4]};
    StepJac J;
    StepTrig<R> trig;
    helix_step<R, float, 5>(pp, dx, kbz, 2.0f, J, &trig);
    SymT<R> Pb = Cbar;
    R q0, q1;
    {
        SymT<R> P = Cb;
        sym_transport<R, false>(P, J);
        const R r0 = my - pp[0], r1 = mz - pp[1];
        const R S00 = P.c00 + vy, S01 = P.c10, S11 = P.c11 + vz;
        const R idet = recip_pos(S00 * S11 - S01 * S01);
        const R i00 = S11 * idet, i01 = -S01 * idet, i11 = S00 * idet;
        const R a0 = i00 * r0 + i01 * r1, a1 = i01 * r0 + i11 * r1;
        const R B0[5] = {P.c00, P.c10, P.c20, P.c30, P.c40};
        const R B1[5] = {P.c10, P.c11, P.c21, P.c31, P.c41};
        const R Cb_[25] = {Cbar.c00, Cbar.c10, Cbar.c20, Cbar.c30, Cbar.c40,
                           Cbar.c10, Cbar.c11, Cbar.c21, Cbar.c31, Cbar.c41,
                           Cbar.c20, Cbar.c21, Cbar.c22, Cbar.c32, Cbar.c42,
                           Cbar.c30, Cbar.c31, Cbar.c32, Cbar.c33, Cbar.c43,
                           Cbar.c40, Cbar.c41, Cbar.c42, Cbar.c43, Cbar.c44};
        R K0[5], K1[5], kp0 = 0, kp1 = 0;       // K, K^T pbar
#pragma unroll
        for (int i = 0; i < 5; ++i) {
            K0[i] = B0[i] * i00 + B1[i] * i01;
            K1[i] = B0[i] * i01 + B1[i] * i11;
            kp0 += K0[i] * pbar[i];
            kp1 += K1[i] * pbar[i];
        }
        R CK0[5], CK1[5];                       // Cbar K
#pragma unroll
        for (int i = 0; i < 5; ++i) {
            R x0 = 0, x1 = 0;
#pragma unroll
            for (int k = 0; k < 5; ++k) {
                x0 += Cb_[i * 5 + k] * K0[k];
                x1 += Cb_[i * 5 + k] * K1[k];
            }
            CK0[i] = x0;
            CK1[i] = x1;
        }
        R k00 = 0, k01 = 0, k11 = 0;            // K^T Cbar K
#pragma unroll
        for (int k = 0; k < 5; ++k) {
            k00 += K0[k] * CK0[k];
            k01 += K0[k] * CK1[k];
            k11 += K1[k] * CK1[k];
        }
        const R u0 = pbar[0] - kp0, u1 = pbar[1] - kp1;        // A^T pbar
        const R h0 = (R)0.5 * a0, h1 = (R)0.5 * a1;
        Pb.c00 += (k00 - (R)2 * CK0[0]) + a0 * (u0 - chibar * a0);
        Pb.c10 += (k01 - CK0[1] - CK1[0]) + h0 * u1 + h1 * u0 - chibar * a0 * a1;
        Pb.c11 += (k11 - (R)2 * CK1[1]) + a1 * (u1 - chibar * a1);
        Pb.c20 += h0 * pbar[2] - CK0[2];
        Pb.c21 += h1 * pbar[2] - CK1[2];
        Pb.c30 += h0 * pbar[3] - CK0[3];
        Pb.c31 += h1 * pbar[3] - CK1[3];
        Pb.c40 += h0 * pbar[4] - CK0[4];
        Pb.c41 += h1 * pbar[4] - CK1[4];
        mby = (R)2 * chibar * a0 + kp0;
        mbz = (R)2 * chibar * a1 + kp1;
        q0 = pbar[0] - mby;
        q1 = pbar[1] - mbz;
    }
    const R q2 = pbar[2], q3 = pbar[3], q4 = pbar[4];
    // Fbar = 2 Pbar F Cb, entries (0,2) (0,4) (1,2) (1,3) (1,4).  Rows 0, 1 of
    // Pbar F: column j of F adds the columns listed in sym_transport.
    const R PF00 = Pb.c00, PF01 = Pb.c10;
    const R PF02 = Pb.c20 + J.f02 * Pb.c00 + J.f12 * Pb.c10;
    const R PF03 = Pb.c30 + J.f13 * Pb.c10;
    const R PF04 = Pb.c40 + J.f04 * Pb.c00 + J.f14 * Pb.c10 + J.f24 * Pb.c20;
    const R PF10 = Pb.c10, PF11 = Pb.c11;
    const R PF12 = Pb.c21 + J.f02 * Pb.c10 + J.f12 * Pb.c11;
    const R PF13 = Pb.c31 + J.f13 * Pb.c11;
    const R PF14 = Pb.c41 + J.f04 * Pb.c10 + J.f14 * Pb.c11 + J.f24 * Pb.c21;
    const R Cc2[5] = {Cb.c20, Cb.c21, Cb.c22, Cb.c32, Cb.c42};     // column 2 of Cb
    const R Cc3[5] = {Cb.c30, Cb.c31, Cb.c32, Cb.c33, Cb.c43};
    const R Cc4[5] = {Cb.c40, Cb.c41, Cb.c42, Cb.c43, Cb.c44};
    const R r0v[5] = {PF00, PF01, PF02, PF03, PF04};
    const R r1v[5] = {PF10, PF11, PF12, PF13, PF14};
    R G02 = 0, G04 = 0, G12 = 0, G13 = 0, G14 = 0;
#pragma unroll
    for (int k = 0; k < 5; ++k) {
        G02 += r0v[k] * Cc2[k];
        G04 += r0v[k] * Cc4[k];
        G12 += r1v[k] * Cc2[k];
        G13 += r1v[k] * Cc3[k];
        G14 += r1v[k] * Cc4[k];
    }
    // Cbar_b = F^T Pbar F
    Cbar = Pb;
    sym_transport<R, true>(Cbar, J);
    // pbar_b = F^T q + second-order term of the Jacobian
    R bs, bt, bw;
    helix_jac_adjoint(pb, dx, kbz, J.f13, trig, (R)2 * G02, (R)2 * G04, (R)2 * G12, (R)2 * G13, (R)2 * G14, bs, bt, bw);
    pbar[0] = q0;
    pbar[1] = q1;
    pbar[2] = q2 + J.f02 * q0 + J.f12 * q1 + bs;
    pbar[3] = q3 + J.f13 * q1 + bt;
    pbar[4] = q4 + J.f04 * q0 + J.f14 * q1 + J.f24 * q2 + bw;
}

// Reverse of helix_start: adjoint of the start state -> adjoints of the
// measurements of A (outermost), B and C (innermost).
template <class R>
__host__ __device__ inline void start_adjoint(R xa, R ya, R za, R xb, R yb, R xc, R yc, R zc,
                                              float kbz, const R pbar[5], R &bya, R &bza, R &byb,
                                              R &byc, R &bzc) {
    const R bcx = xb - xc, bcy = yb - yc;
    const R abx = xa - xb, aby = ya - yb;
    const R acx = xa - xc, acy = ya - yc;
    const R lbc = sqrt(bcx * bcx + bcy * bcy);
    const R lab = sqrt(abx * abx + aby * aby);
    const R lac = sqrt(acx * acx + acy * acy);
    const R prod = lbc * lab * lac;
    const R cross = bcx * aby - bcy * abx;
    const R kap = (R)2 * cross / prod;
    const R ua = (R)0.5 * kap * lab, uc = (R)0.5 * kap * lac;
    const R ca = sqrt(((R)1 - ua) * ((R)1 + ua));       // of half the turning angle, as in helix_start
    const R guc = asin_over_r<5>(uc);
    const R D = lac * guc;
    const R t = (za - zc) / D;
    const R bphi = pbar[2] * (abx * ca - aby * ua) / lab;
    const R lab2 = lab * lab;
    R b_aby = bphi * abx / lab2;
    const R b_ua = bphi / ca;
    bya = pbar[0];
    bza = pbar[1] + pbar[3] / D;
    bzc = -pbar[3] / D;
    const R b_D = -pbar[3] * t / D;
    R b_lac = b_D * guc;
    // d(asin(u)/u)/du
    R gp;
    if (fabs(uc) < (R)0.05) {
        const R u2 = uc * uc;
        gp = uc * ((R)1 / 3 + u2 * ((R)3 / 10 + u2 * ((R)15 / 56 + u2 * ((R)35 / 144))));
    } else {
        gp = ((R)1 / sqrt(((R)1 - uc) * ((R)1 + uc)) - guc) / uc;
    }
    const R b_uc = b_D * lac * gp;
    const R b_kap = pbar[4] / (R)kbz + b_ua * (R)0.5 * lab + b_uc * (R)0.5 * lac;
    R b_lab = b_ua * (R)0.5 * kap;
    b_lac += b_uc * (R)0.5 * kap;
    const R b_cross = (R)2 * b_kap / prod;
    const R b_prod = -b_kap * kap / prod;
    const R b_lbc = b_prod * lab * lac;
    b_lab += b_prod * lbc * lac;
    b_lac += b_prod * lbc * lab;
    b_aby += b_cross * bcx;
    R b_bcy = -b_cross * abx;
    b_bcy += b_lbc * bcy / lbc;
    b_aby += b_lab * aby / lab;
    const R b_acy = b_lac * acy / lac;
    (void)acx;
    byb = b_bcy - b_aby;
    byc = -b_bcy - b_acy;
    bya += b_aby + b_acy;
}
