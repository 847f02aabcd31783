// ks_geodesic.hpp -- null geodesics of the Kerr metric in Kerr-Schild coordinates.
//
// State y = (t~, r, theta, phi~, k^t, k^r, k^theta, k^phi), integrated with the
// classical fourth-order Runge-Kutta scheme (Sec. 2.2.1 of Bronzwaer et al. 2018) of
// dx/dlambda = k, dk/dlambda = -Gamma k k (Sec. 2.2) with the paper's adaptive step
// (Sec. 2.2) written in the logarithmic KS chart (x1 = ln r, x2 = theta/pi, x3 = phi).
//
// The connection term is evaluated in closed form in registers.  With the metric depending
// on (r, theta) only,
//     Gamma^a_{mn} k^m k^n = g^{ab} ( Gdot_{bn} k^n - 1/2 (d_b g_{mn}) k^m k^n ),
//     Gdot_{bn} = k^r d_r g_{bn} + k^theta d_theta g_{bn},
// which is the connection formula of Sec. 2.1 contracted with k twice.  The Kerr-Schild form
// of the metric (Sec. 2.1) is used to contract it: g = g0 + z l l with z = 2 M r / Sigma, the
// null covector l = (1, 1, 0, -a sin^2) and g0 flat space in oblate spheroidal coordinates, so
// that F_b splits into a short flat-space part and a z l l part built from z, its two
// derivatives and l.k; the inverse metric is used in its closed form.
#pragma once
#include "rt_math.hpp"

// Every fused multiply-add of this file is written out and the compiler's own contraction is off, so
// that each kernel variant rounds alike whatever the code around an expression.
#pragma clang fp contract(off)

namespace rk {

// Per-ray constants of the spacetime.
template <class T>
struct Spin {
    T a, a2, M;
    T twoM, m2a, twoa2;   // 2 M, -2 a, 2 a^2
};

template <class T>
__host__ __device__ inline Spin<T> make_spin(T a, T M)
{
    Spin<T> s;
    s.a = a;
    s.a2 = a * a;
    s.M = M;
    s.twoM = T(2.0) * M;
    s.m2a = T(-2.0) * a;
    s.twoa2 = T(2.0) * s.a2;
    return s;
}

// dk/dlambda = -Gamma k k at state y, given s = sin(theta), c = cos(theta).
// F_b = Gdot_{bn} k^n - 1/2 (d_b g_mn) k^m k^n for g = g0 + z l l:
//   z l l part:  zd l_b L + z (k.d l_b) L + z l_b Ld - 1/2 (d_b z) L^2 - z L (d_b l_m) k^m,
//   with L = l.k, zd = k^r dz/dr + k^theta dz/dtheta, and d_theta l_phi = -2 a s c the only
//   derivative of l (Ld = k^theta (d_theta l_phi) k^phi);
//   flat part:   g0 = diag(-1, 1, Sigma) with g0_{r phi} = l_phi, g0_{phi phi} = (r^2 + a^2) sin^2;
// then raised with the closed-form inverse metric.
//
// The order and the fusing of these operations are fixed (LATE: how the third and fourth RK4 stage
// and the second-order steps fuse a^2 cos^2 and 2 M r): images keep them.  Where the orbital flow
// turns null just outside the horizon one sample can hold most of an image's light, and the last bit
// of a trajectory is amplified to as much as 1e-9 of it (FP32 transfer: 1e-8, by how the sample's
// float coefficients round): another order of the same operations moved a 7 x 187 image by 8e-10 of
// its norm and the 512^2 FP32 image of a = 0, i = 85 deg by 1.3e-8 (see ks_accel_short).
// If F_h_out is given, it gets F_theta and *isig_out 1/Sigma, and dk[2] is left to the caller.
template <bool LATE, class T>
__host__ __device__ inline void ks_accel(const Spin<T>& sp, const T* y, T s, T c, T* dk, T* F_h_out = nullptr,
                                         T* isig_out = nullptr)
{
    using namespace rt;
    const T a = sp.a, a2 = sp.a2;
    const T r = y[1];
    const T kt = y[4], kr = y[5], kh = y[6], kp = y[7];
    const T s2 = s * s, sc = s * c, c2 = c * c;
    const T r2 = r * r;
    const T a2c2 = a2 * c2;
    const T sig = LATE ? fma_(a2, c2, r2) : fma_(r, r, a2c2);
    const T dif = LATE ? fma_(a2, c2, -r2) : a2c2 - r2;
    const T w = rcp_nr(sig * s2);                           // 1/(Sigma sin^2)
    const T isig = w * s2;                                  // 1/Sigma
    const T twoMr = sp.twoM * r;
    const T z = twoMr * isig;                               // 2 M r / Sigma
    const T zr = sp.twoM * dif * (isig * isig);             // dz/dr
    const T zt = z * (sp.twoa2 * sc) * isig;                // dz/dtheta
    const T lp = -a * s2;                                   // l_phi
    const T dl = sp.m2a * sc;                               // d l_phi / dtheta
    const T L = fma_(lp, kp, kt + kr);                      // l.k
    const T ld = kh * dl;                                   // k^c d_c l_phi
    const T Ld = ld * kp;
    const T zd = fma_(kr, zr, kh * zt);                     // k^c d_c z
    const T L2 = L * L;
    const T zL = z * L;
    const T khh = kh * kh, kpp = kp * kp;
    const T ra = fma_(r, r, a2);
    const T F1t = fma_(Ld, z, L * zd);                      // z l l part of F_t (the flat part is 0)
    const T F_r = fma_(-L2, T(0.5) * zr, F1t) + fma_(-r, fma_(kpp, s2, khh), Ld);
    T F_h = fma_(kh, (r + r) * kr, -(L2 * (T(0.5) * zt)));
    F_h = fma_(-(dl * kp), fma_(L, z, kr), F_h);
    F_h = fma_(-fma_(a2, khh, ra * kpp), sc, F_h);
    T F_p = fma_(ld, zL, lp * F1t);
    F_p = fma_(kr, fma_(kp, (r + r) * s2, ld), F_p);
    F_p = fma_(kp, kh * ((ra + ra) * sc), F_p);
    // inverse metric: g^tt = -(1+z), g^tr = z, g^rr = Delta/Sigma, g^rp = a/Sigma,
    // g^hh = 1/Sigma, g^pp = 1/(Sigma sin^2)
    const T gi_rr = (LATE ? fma_(-sp.twoM, r, ra) : ra - twoMr) * isig;
    const T ai = a * isig;
    dk[0] = fma_(z, F1t - F_r, F1t);
    dk[1] = -fma_(ai, F_p, fma_(z, F1t, gi_rr * F_r));
    if (F_h_out) {
        *F_h_out = F_h;
        *isig_out = isig;
    } else {
        dk[2] = -isig * F_h;
    }
    dk[3] = -fma_(ai, F_r, w * F_p);
}

// The same connection term in fewer operations, for the thin-disk test, whose rays carry no such
// amplification to their results (they move by 1e-14).
// F_b = Gdot_{bn} k^n - 1/2 (d_b g_mn) k^m k^n splits for g = g0 + z l l into l_b G + R_b, with
// L = l.k, X = z L + k^r (the k_r of the z l l part plus the flat g0_{r phi} cross term) and
//   G   = (k.d z) L + z Ld,  Ld = k^theta (d_theta l_phi) k^phi,
//   R_t = 0,
//   R_r = -1/2 (d_r z) L^2 + Ld - r ((k^theta)^2 + sin^2 (k^phi)^2),
//   R_h = -1/2 (d_theta z) L^2 + 2 r k^r k^theta
//         - sin cos (a^2 (k^theta)^2 + k^phi ((r^2 + a^2) k^phi - 2 a X)),
//   R_p = 2 k^phi r sin^2 k^r + 2 sin cos k^theta ((r^2 + a^2) k^phi - a X).
// Raising uses g^ab = g0^ab - z l^a l^b with l^a = (-1, 1, 0, 0) null, so that l_b G raises to
// l^a G and only R_r meets the z l l part:
//   dk^t = G - z R_r,  dk^r = -dk^t - ((r^2 + a^2) R_r + a R_p) / Sigma,
//   dk^h = -R_h / Sigma,  dk^p = -a R_r / Sigma - R_p / (Sigma sin^2).
// The derivatives of z share the factor 2 M / Sigma^2, which multiplies L once.  57 FP64
// instructions and the reciprocal, against 71 and the reciprocal for raising the whole of F_b
// with the assembled inverse metric.
__host__ __device__ inline void ks_accel_short(const Spin<double>& sp, const double* y, double s, double c, double* dk)
{
    using namespace rt;
    using T = double;
    const T a = sp.a, a2 = sp.a2;
    const T r = y[1];
    const T kt = y[4], kr = y[5], kh = y[6], kp = y[7];
    const T s2 = s * s, sc = s * c;
    const T r2 = r * r;
    const T a2c2 = fma_(-a2, s2, a2);                       // a^2 cos^2
    const T sig = r2 + a2c2, ra = r2 + a2, u = a2c2 - r2;
    const T w = rcp_nr(sig * s2);                           // 1/(Sigma sin^2)
    const T isig = w * s2;                                  // 1/Sigma
    const T mi = sp.twoM * isig;                            // 2 M / Sigma
    const T z = mi * r;                                     // 2 M r / Sigma; d_r z = u mi / Sigma
    const T s2kp = s2 * kp;
    const T L = fma_(-a, s2kp, kt + kr);                    // l.k
    const T X = fma_(z, L, kr);
    const T pL = mi * isig * L;                             // (2 M / Sigma^2) L
    const T H = T(0.5) * pL * L;
    const T t2 = T(2.0) * sc * kh;                          // 2 sin cos k^theta
    const T at2 = a * t2;
    const T mLd = at2 * kp;                                 // -Ld
    const T G = fma_(pL, fma_(a * r, at2, u * kr), -(z * mLd));
    const T R_r = fma_(-u, H, fma_(-r, fma_(s2kp, kp, kh * kh), -mLd));
    const T aX = a * X;
    const T Y = fma_(ra, kp, -aX);
    const T br = fma_(sp.twoa2 * r, H, fma_(kp, Y - aX, a2 * (kh * kh)));
    const T rk = T(2.0) * r * kr;
    const T R_h = fma_(rk, kh, -(sc * br));
    const T R_p = fma_(t2, Y, s2kp * rk);
    dk[0] = fma_(-z, R_r, G);
    dk[1] = fma_(-isig, fma_(ra, R_r, a * R_p), -dk[0]);
    dk[2] = -(isig * R_h);
    dk[3] = -fma_(w, R_p, a * isig * R_r);
}

// f = dy/dlambda (the full eight-component right-hand side).
template <class T>
__host__ __device__ inline void ks_rhs(const Spin<T>& sp, const T* y, T* f)
{
    T s, c;
    rt::sincos_(y[2], &s, &c);
    f[0] = y[4];
    f[1] = y[5];
    f[2] = y[6];
    f[3] = y[7];
    ks_accel<false>(sp, y, s, c, f + 4);
}

// sin and cos of theta + d from s0 = sin(theta), c0 = cos(theta): Taylor polynomials of sin d
// (through d^9) and cos d (through d^10), whose truncation errors for |d| <= 0.1 are below
// 3e-18 relative and 3e-21 absolute, and the angle-addition formulas; larger |d| falls back to
// a full sincos.  With the step rule's eps = 0.05 a stage moves theta by at most about 0.08.
// The polynomials are summed as power sums, each coefficient a multiplicand: a coefficient that
// is an FMA addend must be copied into vector registers first, one multiplicand is read from
// scalar registers as it is.
template <class T>
__host__ __device__ inline void sincos_add(T th, T d, T s0, T c0, T* s, T* c);

template <class T>
__host__ __device__ inline void sincos_shift(T th0, T s0, T c0, T th, T* s, T* c)
{
    sincos_add(th, th - th0, s0, c0, s, c);
}

// The same with the angle th and its offset d from the angle of (s0, c0) given separately (d
// computed by the caller without cancellation); th is used only by the fallback.
template <class T>
__host__ __device__ inline void sincos_add(T th, T d, T s0, T c0, T* s, T* c)
{
    using namespace rt;
    if (fabs_(d) > T(0.1)) {
        sincos_small(th, s, c);
        return;
    }
    // smallest terms first
    const T d2 = d * d, d4 = d2 * d2, d6 = d4 * d2, d8 = d4 * d4;
    T ps = fma_(T(1.0 / 362880.0), d8, T(-1.0 / 5040.0) * d6);
    ps = fma_(T(1.0 / 120.0), d4, ps);
    ps = fma_(T(-1.0 / 6.0), d2, ps);            // sin d / d - 1
    const T sd = fma_(d, ps, d);
    T cdm1 = T(-1.0 / 3628800.0) * (d8 * d2);
    cdm1 = fma_(T(1.0 / 40320.0), d8, cdm1);
    cdm1 = fma_(T(-1.0 / 720.0), d6, cdm1);
    cdm1 = fma_(T(1.0 / 24.0), d4, cdm1);
    cdm1 = fma_(T(-0.5), d2, cdm1);              // cos d - 1
    *s = s0 + fma_(s0, cdm1, c0 * sd);
    *c = c0 + fma_(c0, cdm1, -(s0 * sd));
}

// The same for a half step (|d| <= 0.05, about twice the largest half-step move of theta at
// eps = 0.05): sin d through d^7 and cos d through d^8, truncation below 2e-18 relative and
// 3e-20 absolute.
template <class T>
__host__ __device__ inline void sincos_shift_half(T th0, T s0, T c0, T th, T* s, T* c)
{
    using namespace rt;
    const T d = th - th0;
    if (fabs_(d) > T(0.05)) {
        sincos_small(th, s, c);
        return;
    }
    const T d2 = d * d, d4 = d2 * d2, d6 = d4 * d2;
    T ps = T(-1.0 / 5040.0) * d6;
    ps = fma_(T(1.0 / 120.0), d4, ps);
    ps = fma_(T(-1.0 / 6.0), d2, ps);            // sin d / d - 1
    const T sd = fma_(d, ps, d);
    T cdm1 = fma_(T(1.0 / 40320.0), d4 * d4, T(-1.0 / 720.0) * d6);
    cdm1 = fma_(T(1.0 / 24.0), d4, cdm1);
    cdm1 = fma_(T(-0.5), d2, cdm1);              // cos d - 1
    *s = s0 + fma_(s0, cdm1, c0 * sd);
    *c = c0 + fma_(c0, cdm1, -(s0 * sd));
}

// Positive step size of the adaptive rule (Sec. 2.2),
//   1/dl = (|k^x1| + d)/eps + (|k^x2| + d)/(eps min(x2, 1 - x2)) + (|k^x3| + d)/eps
// with k^x1 = k^r / r, k^x2 = k^theta / pi, x2 = theta / pi, k^x3 = k^phi, evaluated with a
// single division.  `edge` is floored at 1e-12.
template <class T>
__host__ __device__ inline T step_size(T eps, const T* y)
{
    using namespace rt;
    const T d = T(1e-40);
    const T r = y[1];
    const T edge = fmax_(fmin_(y[2] * T(M_1_PI), fma_(y[2], T(-M_1_PI), T(1.0))), T(1e-12));
    T den = fma_(r, d, fabs_(y[5])) * edge;
    den = fma_(r, fma_(fabs_(y[6]), T(M_1_PI), d), den);
    den = fma_(r * (fabs_(y[7]) + d), edge, den);
    return eps * r * edge * rcp_nr(den);
}

// The work count treats sincos_shift and sincos_shift_half as one sine-cosine evaluation.
inline void sincos_shift(rt::OpCounted th0, rt::OpCounted s0, rt::OpCounted c0, rt::OpCounted th,
                         rt::OpCounted* s, rt::OpCounted* c)
{
    (void)th0; (void)s0; (void)c0;
    rt::sincos_(th, s, c);
}
inline void sincos_shift_half(rt::OpCounted th0, rt::OpCounted s0, rt::OpCounted c0, rt::OpCounted th,
                              rt::OpCounted* s, rt::OpCounted* c)
{
    sincos_shift(th0, s0, c0, th, s, c);
}

// One classical RK4 step of size dl (negative: away from the camera) on y = (x, k).  s0, c0
// are sin and cos of y[2]; the three later stages get theirs with sincos_shift (the two
// half-step stages with its shorter half-step form).  The position
// derivative of a stage is that stage's wave vector, so only dk/dlambda is evaluated.
template <class T>
__host__ __device__ inline void rk4_step(const Spin<T>& sp, T* y, T dl, T s0, T c0)
{
    using namespace rt;
    T t[8], acc[8], dk[4];
    T s, c;
    ks_accel<false>(sp, y, s0, c0, dk);
    const T h2 = T(0.5) * dl;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        acc[i] = y[4 + i];
        acc[4 + i] = dk[i];
        t[i] = fma_(h2, y[4 + i], y[i]);
        t[4 + i] = fma_(h2, dk[i], y[4 + i]);
    }
    sincos_shift_half(y[2], s0, c0, t[2], &s, &c);
    ks_accel<false>(sp, t, s, c, dk);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        acc[i] = fma_(T(2.0), t[4 + i], acc[i]);
        acc[4 + i] = fma_(T(2.0), dk[i], acc[4 + i]);
        t[i] = fma_(h2, t[4 + i], y[i]);
        t[4 + i] = fma_(h2, dk[i], y[4 + i]);
    }
    sincos_shift_half(y[2], s0, c0, t[2], &s, &c);
    ks_accel<true>(sp, t, s, c, dk);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        acc[i] = fma_(T(2.0), t[4 + i], acc[i]);
        acc[4 + i] = fma_(T(2.0), dk[i], acc[4 + i]);
        t[i] = fma_(dl, t[4 + i], y[i]);
        t[4 + i] = fma_(dl, dk[i], y[4 + i]);
    }
    sincos_shift(y[2], s0, c0, t[2], &s, &c);
    T F_h, isig;
    ks_accel<true>(sp, t, s, c, dk, &F_h, &isig);
    const T h6 = dl * T(1.0 / 6.0);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        y[i] = fma_(h6, acc[i] + t[4 + i], y[i]);
        y[4 + i] = fma_(h6, i == 2 ? fma_(-isig, F_h, acc[4 + i]) : acc[4 + i] + dk[i], y[4 + i]);
    }
}

// rk4_step and the sine and cosine of the new theta as one basic block: bit for bit rk4_step with
// its shifts of the angle, without their branches.  The size tests of the four shifts are made
// together before y is written; false (y untouched) if one fails, which at eps = 0.05 none does.
// The trace kernel is bound by vector-instruction issue and, with few rays, by the length of the
// step's chain: the branches cost both scalar instructions and the overlap of one stage's angle with
// the other's connection term.
__host__ __device__ inline bool rk4_try_block(const Spin<double>& sp, double* y, double dl, double* sin_th,
                                              double* cos_th)
{
    using namespace rt;
    const double s0 = *sin_th, c0 = *cos_th, h2 = 0.5 * dl, h6 = dl * (1.0 / 6.0);
    double t[8], acc[8], dk[4], s, c, F_h, isig;
    const auto half = [&](double d) {
        const double d2 = d * d, d4 = d2 * d2, d6 = d4 * d2;
        const double ps = fma_(-1.0 / 6.0, d2, fma_(1.0 / 120.0, d4, (-1.0 / 5040.0) * d6));
        const double sd = fma_(d, ps, d);
        double cm = fma_(1.0 / 40320.0, d4 * d4, (-1.0 / 720.0) * d6);
        cm = fma_(-0.5, d2, fma_(1.0 / 24.0, d4, cm));
        s = s0 + fma_(s0, cm, c0 * sd);
        c = c0 + fma_(c0, cm, -(s0 * sd));
    };
    const auto full = [&](double d) {
        const double d2 = d * d, d4 = d2 * d2, d6 = d4 * d2, d8 = d4 * d4;
        double ps = fma_(1.0 / 362880.0, d8, (-1.0 / 5040.0) * d6);
        ps = fma_(-1.0 / 6.0, d2, fma_(1.0 / 120.0, d4, ps));
        const double sd = fma_(d, ps, d);
        double cm = fma_(1.0 / 40320.0, d8, (-1.0 / 3628800.0) * (d8 * d2));
        cm = fma_(1.0 / 24.0, d4, fma_(-1.0 / 720.0, d6, cm));
        cm = fma_(-0.5, d2, cm);
        s = s0 + fma_(s0, cm, c0 * sd);
        c = c0 + fma_(c0, cm, -(s0 * sd));
    };
    const auto stage = [&](double h) {   // the wave vector and the radius of the next stage
        const double kr = t[5];
#pragma unroll
        for (int i = 0; i < 4; ++i) t[4 + i] = fma_(h, dk[i], y[4 + i]);
        t[1] = fma_(h, kr, y[1]);
    };
    ks_accel<false>(sp, y, s0, c0, dk);
    const double d1 = fma_(h2, y[6], y[2]) - y[2];
    half(d1);
    t[5] = y[5];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        acc[i] = y[4 + i];
        acc[4 + i] = dk[i];
    }
    stage(h2);
    ks_accel<false>(sp, t, s, c, dk);
    const double d2 = fma_(h2, t[6], y[2]) - y[2];
    half(d2);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        acc[i] = fma_(2.0, t[4 + i], acc[i]);
        acc[4 + i] = fma_(2.0, dk[i], acc[4 + i]);
    }
    stage(h2);
    ks_accel<true>(sp, t, s, c, dk);
    const double d3 = fma_(dl, t[6], y[2]) - y[2];
    full(d3);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        acc[i] = fma_(2.0, t[4 + i], acc[i]);
        acc[4 + i] = fma_(2.0, dk[i], acc[4 + i]);
    }
    stage(dl);
    ks_accel<true>(sp, t, s, c, dk, &F_h, &isig);
    const double th = fma_(h6, acc[2] + t[6], y[2]);
    const double d4 = th - y[2];
    full(d4);
    if (!(fmax_(fabs_(d1), fabs_(d2)) <= 0.05 && fmax_(fabs_(d3), fabs_(d4)) <= 0.1)) return false;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        y[i] = i == 2 ? th : fma_(h6, acc[i] + t[4 + i], y[i]);
        y[4 + i] = fma_(h6, i == 2 ? fma_(-isig, F_h, acc[4 + i]) : acc[4 + i] + dk[i], y[4 + i]);
    }
    *sin_th = s;
    *cos_th = c;
    return true;
}

// sin and cos of an angle d away from the one of (s0, c0), from sd = sin d and cm = cos d - 1.
__host__ __device__ inline void rotate(double sd, double cm, double s0, double c0, double* s, double* c)
{
    using namespace rt;
    *s = fma_(c0, sd, fma_(s0, cm, s0));
    *c = fma_(-s0, sd, fma_(c0, cm, c0));
}

// Rotation by |d| <= ROT_HALF, about the largest half-step move of theta at eps = 0.05 (0.039) with
// some margin: sin d through d^7, cos d through d^8 (truncation below 2e-18 and 3e-20).
constexpr double ROT_HALF = 0.05;
__host__ __device__ inline void rotate_half(double d, double s0, double c0, double* s, double* c)
{
    using namespace rt;
    const double d2 = d * d, d4 = d2 * d2, d6 = d4 * d2;
    double ps = (-1.0 / 5040.0) * d6;
    ps = fma_((1.0 / 120.0), d4, ps);
    ps = fma_((-1.0 / 6.0), d2, ps);             // sin d / d - 1
    double cm = (1.0 / 40320.0) * (d4 * d4);
    cm = fma_((-1.0 / 720.0), d6, cm);
    cm = fma_((1.0 / 24.0), d4, cm);
    cm = fma_((-0.5), d2, cm);                   // cos d - 1
    rotate(fma_(d, ps, d), cm, s0, c0, s, c);
}

// Rotation by |d| <= ROT_SMALL: sin d through d^5, cos d through d^4 (truncation below 1e-18
// relative and 5e-18 absolute).
constexpr double ROT_SMALL = 0.00390625;
__host__ __device__ inline void rotate_small(double d, double s0, double c0, double* s, double* c)
{
    using namespace rt;
    const double d2 = d * d, d3 = d * d2, d4 = d2 * d2;
    double sd = (1.0 / 120.0) * (d3 * d2);
    sd = fma_((-1.0 / 6.0), d3, sd);
    double cm = (1.0 / 24.0) * d4;
    cm = fma_((-0.5), d2, cm);
    rotate(d + sd, cm, s0, c0, s, c);
}

// Rotation by |d| <= ROT_TINY: sin d through d^3, cos d through d^2 (truncation below 1e-18
// relative and 5e-18 absolute).
constexpr double ROT_TINY = 1e-4;
__host__ __device__ inline void rotate_tiny(double d, double s0, double c0, double* s, double* c)
{
    const double d2 = d * d;
    rotate(rt::fma_((-1.0 / 6.0) * d, d2, d), -0.5 * d2, s0, c0, s, c);
}

// One RK4 step as rk4_step, and sin and cos of the new theta: s, c are those of y[2] on entry and
// on return.  The angles of a step are chained: from y to the first half-step stage (a half-step
// move), on to the second (whose offset is h^2/4 dk^theta, second order in the step), on to the
// full-step stage (a half-step move), and on to the new theta, whose offset from that stage is
// dl^2/6 times the second difference of the stages' derivatives (fourth order).  Each move takes
// the shortest polynomials for its size, and each offset is formed as the product it is rather
// than as the difference of two angles.  The position update needs the sum of the first three
// derivatives only (a stage's position derivative is its wave vector, itself y's plus a
// derivative).  The whole step is one basic block: the four size tests are made together before
// y is written.  A lane that fails one takes rk4_step and the full-size shift instead: at eps = 0.05
// 3e-5 of the steps do (near the axis and at large curvature); with an eps above EPS_CHAINED, where
// ordinary steps begin to, every step takes that form at once.
// 339 FP64 instructions against 459 for rk4_step and its shifts.
constexpr double EPS_CHAINED = 0.0625;
__host__ __device__ inline bool rk4_try_chained(const Spin<double>& sp, double* y, double dl, double* sin_th,
                                                double* cos_th)
{
    using namespace rt;
    const double h2 = 0.5 * dl, dl6 = dl * (1.0 / 6.0);
    const double s0 = *sin_th, c0 = *cos_th;
    double t[8], k1[4], k2[4], k3[4], k4[4];
    double s, c;
    ks_accel_short(sp, y, s0, c0, k1);
    const double d1 = h2 * y[6];
    rotate_half(d1, s0, c0, &s, &c);
    const double e1 = h2 * k1[2];                       // the second stage's k^theta less y's
    t[1] = fma_(h2, y[5], y[1]);
    t[4] = fma_(h2, k1[0], y[4]);
    t[5] = fma_(h2, k1[1], y[5]);
    t[6] = y[6] + e1;
    t[7] = fma_(h2, k1[3], y[7]);
    ks_accel_short(sp, t, s, c, k2);
    const double d2 = h2 * e1;
    rotate_small(d2, s, c, &s, &c);
    const double e2 = h2 * k2[2];
    const double t6 = t[6];
    t[1] = fma_(h2, t[5], y[1]);
    t[4] = fma_(h2, k2[0], y[4]);
    t[5] = fma_(h2, k2[1], y[5]);
    t[6] = y[6] + e2;
    t[7] = fma_(h2, k2[3], y[7]);
    ks_accel_short(sp, t, s, c, k3);
    const double d3 = h2 * fma_(2.0, t[6], -t6);        // dl t6(3) - h2 t6(2)
    rotate_half(d3, s, c, &s, &c);
    t[1] = fma_(dl, t[5], y[1]);
    t[4] = fma_(dl, k3[0], y[4]);
    t[5] = fma_(dl, k3[1], y[5]);
    t[6] = fma_(dl, k3[2], y[6]);
    t[7] = fma_(dl, k3[3], y[7]);
    ks_accel_short(sp, t, s, c, k4);
    double k23[4], k123[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        k23[i] = k2[i] + k3[i];
        k123[i] = k1[i] + k23[i];
    }
    const double d4 = dl * fma_(dl6, k123[2], -e2);
    rotate_tiny(d4, s, c, &s, &c);
    if (!(fmax_(fabs_(d1), fabs_(d3)) <= ROT_HALF && fabs_(d2) <= ROT_SMALL && fabs_(d4) <= ROT_TINY)) return false;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        y[i] = fma_(dl, fma_(dl6, k123[i], y[4 + i]), y[i]);
        y[4 + i] = fma_(dl6, k123[i] + (k23[i] + k4[i]), y[4 + i]);
    }
    *sin_th = s;
    *cos_th = c;
    return true;
}

// One RK4 step and the sine and cosine of theta with it (those of y[2] on entry and on return):
// SHORT the chained form, else rk4_step's own operations; `block`: eps is small enough for either.
template <bool SHORT = true>
__host__ __device__ inline void rk4_step_angles(const Spin<double>& sp, double* y, double dl, bool block,
                                                double* sin_th, double* cos_th)
{
    if (block && (SHORT ? rk4_try_chained(sp, y, dl, sin_th, cos_th) : rk4_try_block(sp, y, dl, sin_th, cos_th)))
        return;
    const double th0 = y[2], s0 = *sin_th, c0 = *cos_th;
    rk4_step(sp, y, dl, s0, c0);
    sincos_shift(th0, s0, c0, y[2], sin_th, cos_th);
}

// One second-order Runge-Kutta (midpoint) step: dk/dlambda at y and at y + (dl/2) f(y), then
// y + dl f(midpoint).  The paper names RK2 for its timing runs without spelling it out; the
// midpoint rule is the reading taken.
template <class T>
__host__ __device__ inline void rk2_step(const Spin<T>& sp, T* y, T dl, T s0, T c0)
{
    using namespace rt;
    T t[8], dk[4];
    T s, c;
    ks_accel<true>(sp, y, s0, c0, dk);
    const T h2 = T(0.5) * dl;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        t[i] = fma_(h2, y[4 + i], y[i]);
        t[4 + i] = fma_(h2, dk[i], y[4 + i]);
    }
    sincos_shift_half(y[2], s0, c0, t[2], &s, &c);
    ks_accel<true>(sp, t, s, c, dk);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        y[i] = fma_(dl, t[4 + i], y[i]);
        y[4 + i] = fma_(dl, dk[i], y[4 + i]);
    }
}

// One velocity-Verlet step (Sec. 2.2.2) with A = dk/dlambda at y carried in acc:
//   x' = x + k dl + A dl^2/2,  k_p = k + A dl,  A' = accel(x', k_p),  k' = k + (A + A') dl/2,
// with the corrector A' = accel(x', k') and k' recomputed once more.  acc returns the last
// evaluated derivative.  One connection evaluation per step (two with the corrector).
template <class T>
__host__ __device__ inline void verlet_step(const Spin<T>& sp, T* y, T* acc, T dl, bool corrector, T s0, T c0)
{
    using namespace rt;
    T t[8], dk[4];
    T s, c;
    const T hh = T(0.5) * dl * dl;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        t[i] = fma_(hh, acc[i], fma_(y[4 + i], dl, y[i]));
        t[4 + i] = fma_(acc[i], dl, y[4 + i]);
    }
    sincos_shift(y[2], s0, c0, t[2], &s, &c);
    const T h2 = T(0.5) * dl;
    for (int pass = 0; pass < (corrector ? 2 : 1); ++pass) {
        T F_h, isig;
        ks_accel<true>(sp, t, s, c, dk, &F_h, &isig);
        dk[2] = -isig * F_h;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            t[4 + i] = fma_(h2, i == 2 ? fma_(-isig, F_h, acc[2]) : acc[i] + dk[i], y[4 + i]);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        y[i] = t[i];
        y[4 + i] = t[4 + i];
        acc[i] = dk[i];
    }
}

// Virtual camera (Sec. 2.3) at radius r_cam and polar angle incl, impact parameters
// (alpha, beta): E = 1, L = -alpha sin(i), Q = beta^2 + cos^2(i)(alpha^2 - a^2),
// k_theta = sign(beta) sqrt|Q - L^2 cot^2(i) + a^2 cos^2(i)|, k_r > 0 from the null
// condition with the Boyer-Lindquist inverse metric, raised and mapped to KS with the
// appendix matrix (k^t~ = k^t + 2 M r/Delta k^r, k^phi~ = k^phi + a/Delta k^r).
// CameraFrame: what the pixels of an image share, formed once per image.
template <class T>
struct CameraFrame {
    T r, incl, t_init, a2, sin_i, cos_i, c2, a2ci, cot;
    T gtt, gtp, gpp, grr, ghh, igrr;   // Boyer-Lindquist inverse metric at the camera, 1 / g^rr
    T ht, hp;                          // 2 M r / Delta, a / Delta
};

template <class T>
__host__ __device__ inline CameraFrame<T> camera_frame(T a, T M, T r, T incl, T sin_i, T cos_i, T t_init)
{
    using namespace rt;
    CameraFrame<T> f;
    f.r = r;
    f.incl = incl;
    f.t_init = t_init;
    const T a2 = a * a;
    f.a2 = a2;
    f.sin_i = sin_i;
    f.cos_i = cos_i;
    f.c2 = cos_i * cos_i;
    f.a2ci = a2 * cos_i;
    f.cot = cos_i * rcp(sin_i);
    const T s2 = sin_i * sin_i;
    const T sig = fma_(r, r, a2 * f.c2);
    const T del = fma_(a, a, fma_(r, r, -(T(2.0) * M * r)));
    const T ra = fma_(r, r, a2);
    const T isd = rcp(sig * del);
    f.gtt = -fma_(ra, ra, -(a2 * del * s2)) * isd;
    f.gtp = -T(2.0) * M * a * r * isd;
    f.gpp = fma_(-a2, s2, del) * isd * rcp(s2);
    f.ghh = rcp(sig);
    f.grr = del * f.ghh;
    f.igrr = rcp(f.grr);
    const T idel = rcp(del);
    f.ht = T(2.0) * M * r * idel;
    f.hp = a * idel;
    return f;
}

template <class T>
__host__ __device__ inline void camera_ray(const CameraFrame<T>& f, T alpha, T beta, T* y)
{
    using namespace rt;
    const T L = -alpha * f.sin_i;
    const T Q = fma_(beta, beta, fma_(alpha, alpha, -f.a2) * f.c2);
    // at beta = 0 the radicand cancels to rounding: its operations and their order decide k_theta
    const T rad = fma_(f.cos_i, f.a2ci, fma_(-f.cot, f.cot * (L * L), Q));
    const T kth = (beta >= T(0.0) ? T(1.0) : T(-1.0)) * sqrt_(fabs_(rad));
    // g^tt k_t^2 + 2 g^tp k_t k_p + g^pp k_p^2 + g^hh k_h^2 + g^rr k_r^2 = 0, k_t = -1
    const T kh_up = f.ghh * kth;
    const T rest = fma_(kth, kh_up, fma_(L, f.gpp * L, fma_(T(-2.0) * f.gtp, L, f.gtt)));
    const T kr_up = f.grr * sqrt_(fmax_(-rest * f.igrr, T(0.0)));
    y[0] = f.t_init;
    y[1] = f.r;
    y[2] = f.incl;
    y[3] = T(0.0);
    y[4] = fma_(f.ht, kr_up, fma_(f.gtp, L, -f.gtt));
    y[5] = kr_up;
    y[6] = kh_up;
    y[7] = fma_(f.hp, kr_up, fma_(f.gpp, L, -f.gtp));
}

// Pole crossing: (theta, phi) -> (-theta, phi + pi) or (2 pi - theta, phi + pi) is the same
// point and the polar velocity changes sign.  Returns 1 if the state was reflected.
template <class T>
__host__ __device__ inline int reflect_pole(T* y)
{
    if (y[2] < T(0.0)) {
        y[2] = -y[2];
    } else if (y[2] > T(M_PI)) {
        y[2] = T(2.0 * M_PI) - y[2];
    } else {
        return 0;
    }
    y[3] = y[3] + T(M_PI);
    y[6] = -y[6];
    return 1;
}

}  // namespace rk

#pragma clang fp contract(fast)
