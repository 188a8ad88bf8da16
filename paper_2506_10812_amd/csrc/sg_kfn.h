// sg_kfn.h -- device evaluation of F(x) = e^x [K1(x) - K0(x)] and of the
// exact kernel in its Cartesian and log-polar (App. C) forms.
//
// F(x) is the function of App. A (there at argument x/4) that carries the
// whole distance dependence of the exact kernel (Sect. 2.2):
//     K_ab(s) = pi^{-1/2} H_ab^{-2} (d/8) F(d^2/8),  d = s/H_ab.
// Evaluation never forms e^x K1(x) and e^x K0(x) separately at large x (their
// difference cancels and e^x overflows, the NaN problem noted in Sect. 5.3):
//   double
//     x < 1/16          power series of I0, I1, K0, K1 (Abramowitz & Stegun
//           9.6.10, 9.6.11), F = e^x (K1 - K0);
//     1/16 <= x < 256   local polynomials of 12 terms on 8 intervals per
//           octave (gen_cheb64.cpp -> sg_cheb64.h, fitted at build time in
//           long double), within 4e-16 of F, with no square root or division;
//     x >= 256          the asymptotic series F = (sqrt(2 pi)/4) x^{-3/2}
//           sum_n c_n x^-n, c_0 = 1, c_n = -c_{n-1} (4 n^2 - 1)/(8 n) (its
//           first three terms are the expansion printed in Sect. 5.3) through
//           c_7: the remainder is below the first omitted term, 6e-18.
//     The same three branches give D(x) = -x F' - 3/2 F (what the derivatives
//     with respect to the scale heights need; the difference of its two terms
//     would lose log10(x) digits), G0(x) = e^x K0(x) (the potential's kernel)
//     and E(x) = 2 x F - G0 (its derivative).  A block copies the one table
//     it needs (9 KB) into LDS.  Per wave an evaluation is 12 LDS reads and 11
//     FMAs in a dependent chain; the Chebyshev series of 27 terms used before
//     took 27 reads and 53 operations, and below 32 only.
//   float
//     x < 1             the same power series;
//     1 <= x < 32       F = sqrt(2) x^{-3/2} J(x),  J(x) = int_0^inf v^2 e^{-v^2}
//           (1 + v^2/(2x))^{-1/2} dv, obtained from the integral
//           representation K_nu(x) = int_0^inf e^{-x cosh t} cosh(nu t) dt by
//           the substitution sinh(t/2) = v / sqrt(2x).  The integrand is even
//           and analytic for |Im v| < sqrt(2x), so the trapezoidal rule on a
//           fixed grid converges geometrically, its error ~ exp(-2 pi
//           sqrt(2x) / step): step 1/2 and 9 nodes (2e-8 at x = 1, below a
//           float ulp; the tail beyond v = 4.5 is e^{-20});
//     x >= 32           the asymptotic series through c_5.
// The float trapezoidal weights e^{-v_k^2} and the double tables are copied
// once per workgroup into LDS (sg_fill_weights, sg_fill64).
#pragma once
#include "sg_internal.h"
#include "sg_cheb64.h"

#define SG_EULER_GAMMA 0.57721566490153286061

// LDS table of TABLE entries.  Float: w[k-1] = exp(-(k STEP)^2), k = 1..NODES.
// Double: the local polynomials of one function.
enum { SG_FN_F = 0, SG_FN_D = 1, SG_FN_G0 = 2, SG_FN_E = 3 };
template <typename R> struct FQuad;
template <> struct FQuad<double> {
    static constexpr int TABLE = SG_POLY_NI * SG_POLY_NC;
};
template <> struct FQuad<float> {
    static constexpr int NODES = 9;
    static constexpr float STEP = 0.5f;
    static constexpr int TABLE = NODES;
};

// Reciprocal and reciprocal square root of the working type.  Float takes the
// hardware v_rcp_f32 / v_rsq_f32 (about 1 ulp; arguments here are normal and
// positive): rsqrt() has only a double overload, so a float argument would be
// promoted to the double sequence, and '/' costs the full IEEE division.
__device__ inline float sg_rcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ inline double sg_rcp(double x) { return 1.0 / x; }
__device__ inline float sg_rsqrt(float x) { return __builtin_amdgcn_rsqf(x); }
__device__ inline double sg_rsqrt(double x) { return rsqrt(x); }

// Call from every thread, then sync.  fn: the function of a double table
// (uniform over the block).
__device__ inline void sg_fill64(double *w, int fn)
{
    for (int k = threadIdx.x; k < FQuad<double>::TABLE; k += blockDim.x) w[k] = sg_poly64[fn * FQuad<double>::TABLE + k];
}
template <typename R> __device__ inline void sg_fill_weights(R *w, int fn = SG_FN_F)
{
    if constexpr (sizeof(R) == 8) {
        sg_fill64(w, fn);
    } else {
        for (int k = threadIdx.x; k < FQuad<R>::TABLE; k += blockDim.x) {
            const double v = (k + 1) * (double)FQuad<float>::STEP;
            w[k] = (R)exp(-v * v);
        }
    }
}

// Series branch, small x.  NT terms.
template <typename R, int NT>
__device__ inline void sg_F_series(R x, R &F, R *dF)
{
    const R y = x * x * R(0.25);
    const R Lg = log(x * R(0.5)) + R(SG_EULER_GAMMA);
    R tk = R(1), sk = R(1), Hk = R(0);
    R I0 = R(0), I1s = R(0), K0s = R(0), K1s = R(0);
#pragma unroll
    for (int k = 0; k < NT; ++k) {
        const R Hk1 = Hk + R(1) / R(k + 1);
        I0 += tk;
        I1s += sk;
        K0s += Hk * tk;
        K1s += (Hk + Hk1) * sk;
        tk *= y * (R(1) / R((k + 1) * (k + 1)));  // constant reciprocals, folded
        sk *= y * (R(1) / R((k + 1) * (k + 2)));
        Hk = Hk1;
    }
    const R ix = sg_rcp(x);
    const R I1 = x * R(0.5) * I1s;
    const R K0 = -Lg * I0 + K0s;
    const R K1 = ix + Lg * I1 - x * R(0.25) * K1s;
    const R ex = exp(x);
    F = ex * (K1 - K0);
    if (dF) *dF = ex * (R(2) * (K1 - K0) - K1 * ix);
}

// Trapezoidal branch, x >= 2: F = sqrt(2) x^-3/2 J, F' from J' =
// int v^2 e^{-v^2} v^2/(4x^2) (1 + v^2/(2x))^{-3/2} dv.
template <typename R>
__device__ inline void sg_F_quad(R x, const R *w, R &F, R *dF)
{
    const R ix = sg_rcp(x);
    const R i2x = R(0.5) * ix;
    R J = R(0), Jd = R(0);
#pragma unroll
    for (int k = 1; k <= FQuad<R>::NODES; ++k) {
        const R v2 = R(k * k) * (FQuad<R>::STEP * FQuad<R>::STEP);
        const R rho = sg_rsqrt(R(1) + v2 * i2x);
        const R base = w[k - 1] * v2 * rho;
        J += base;
        if (dF) Jd += base * rho * rho * v2;
    }
    J *= FQuad<R>::STEP;
    const R x32 = sg_rsqrt(x) * ix;  // x^-3/2
    F = R(SG_SQRT2) * x32 * J;
    if (dF) {
        const R Jp = Jd * FQuad<R>::STEP * R(0.25) * (ix * ix);
        *dF = R(SG_SQRT2) * x32 * (Jp - R(1.5) * J * ix);
    }
}

// Asymptotic branch (float), x >= 32.
struct AsymCoef {
    float c[6];
    constexpr AsymCoef() : c{}
    {
        double v = 1.0;
        c[0] = 1.0f;
        for (int n = 1; n < 6; ++n) {
            v = -v * (4.0 * n * n - 1.0) / (8.0 * n);
            c[n] = (float)v;
        }
    }
};

__device__ inline float sg_F_asym(float x)
{
    constexpr AsymCoef C;
    const float u = sg_rcp(x);
    float s = C.c[5];
#pragma unroll
    for (int n = 4; n >= 0; --n) s = s * u + C.c[n];
    const float J = float(SG_SQRT_PI * 0.25) * s;
    const float rx = sg_rsqrt(x);
    return float(SG_SQRT2) * rx * u * J;
}

// Wave-uniform branches: the series and the asymptotic form each run only
// when some lane of the wave needs them, every lane keeping its own branch's
// value.  SG_NO_SPECULATE, an empty asm statement that emits no instruction,
// keeps the compiler from if-converting such branches into straight-line code
// that evaluates every branch for every lane.
#define SG_NO_SPECULATE() asm volatile("")

// Series branch of the double functions (x < 1/16: y = x^2/4 < 1e-3, so 5
// terms leave y^5/(5!)^2 < 1e-19).
template <int FN> __device__ inline double sg_series64(double x);
template <typename R, int NT> __device__ inline R sg_G0_series(R x);

// Asymptotic coefficients n = 0..7 of F / ((sqrt(2 pi)/4) x^{-3/2}), of D over
// the same (n c_n), of G0 / sqrt(pi/(2x)) (a_n = -a_{n-1} (2n - 1)^2/(8n)) and
// of E over the same (c_n - a_n).
template <int FN> struct Asym64 {
    double c[8];
    constexpr Asym64() : c{}
    {
        double v = 1.0, g = 1.0;
        for (int n = 0; n < 8; ++n) {
            if (n) {
                v = -v * (4.0 * n * n - 1.0) / (8.0 * n);
                g = -g * (2.0 * n - 1.0) * (2.0 * n - 1.0) / (8.0 * n);
            }
            c[n] = FN == SG_FN_F ? v : FN == SG_FN_D ? n * v : FN == SG_FN_G0 ? g : v - g;
        }
    }
};

// The function FN at x > 0; w: its table.  Lanes outside the polynomials'
// range (whose value is discarded) are clamped to an interval.
template <int FN> __device__ inline double sg_fn64(double x, const double *w)
{
    static_assert(SG_POLY_SUB == 8 && SG_POLY_NC == 12, "index arithmetic below");
    const int hi = __double2hiint(x);
    const int k = min(max((hi >> 17) - ((1023 + SG_POLY_OCT0) << 3), 0), SG_POLY_NI - 1);
    // the 3 leading mantissa bits are in k; the rest as v in [1, 1 + 1/8), t = 16 v - 17
    const double t = fma(16.0, __hiloint2double((hi & 0x1ffff) | 0x3ff00000, __double2loint(x)), -17.0);
    const double2 *c = (const double2 *)(w + k * SG_POLY_NC);
    double2 q[6];
#pragma unroll
    for (int j = 0; j < 6; ++j) q[j] = c[j];
    double f = q[5].y;
#pragma unroll
    for (int j = 5; j >= 0; --j) {
        if (j < 5) f = fma(f, t, q[j].y);
        f = fma(f, t, q[j].x);
    }
    if (__any(!(x < 256.0))) {  // NaN included
        SG_NO_SPECULATE();
        constexpr Asym64<FN> A;
        const double r = rsqrt(x), u = r * r;
        double s = A.c[7];
#pragma unroll
        for (int n = 6; n >= 0; --n) s = fma(s, u, A.c[n]);
        s *= FN == SG_FN_F || FN == SG_FN_D ? (SG_SQRT2 * SG_SQRT_PI * 0.25) * (u * r) : (SG_SQRT_PI / SG_SQRT2) * r;
        f = x < 256.0 ? f : s;
    }
    if (__any(x < 0.0625)) {
        SG_NO_SPECULATE();
        const double s = sg_series64<FN>(x);
        f = x < 0.0625 ? s : f;
    }
    return f;
}

__device__ inline double sg_F64(double x, const double *w) { return sg_fn64<SG_FN_F>(x, w); }
__device__ inline double sg_D64(double x, const double *w) { return sg_fn64<SG_FN_D>(x, w); }
__device__ inline double sg_G0_64(double x, const double *w) { return sg_fn64<SG_FN_G0>(x, w); }
__device__ inline double sg_E64(double x, const double *w) { return sg_fn64<SG_FN_E>(x, w); }

// Float: each branch runs only when some lane of the wave needs it, and each
// lane keeps its own branch's value (a wave whose lanes all fall in one range
// pays for one branch).
__device__ inline float sg_F32(float x, const float *w)
{
    const bool ser = x < 1.0f, asy = x >= 32.0f, quad = !ser && !asy;
    float F = 0.0f, t;
    if (__any(ser)) {
        SG_NO_SPECULATE();
        sg_F_series<float, 8>(x, t, nullptr);
        F = ser ? t : F;
    }
    if (__any(quad)) {
        SG_NO_SPECULATE();
        sg_F_quad<float>(x, w, t, nullptr);
        F = quad ? t : F;
    }
    if (__any(asy)) {
        SG_NO_SPECULATE();
        t = sg_F_asym(x);
        F = asy ? t : F;
    }
    return F;
}

// ------------------------------------------------------------------------
// G0(x) = e^x K0(x), the kernel of the conservative potential (Sect. 5.5,
// appendix "Conservative force"): P_ab(s) = -G0(d^2/8) / (2 sqrt(pi) H_ab).
// Double: sg_fn64 above.  Float:
//   x < 1   A&S series of I0 and K0, G0 = e^x K0;
//   1 <= x < 32  G0 = sqrt(2/x) int_0^inf e^{-v^2}
//        (1 + v^2/(2x))^{-1/2} dv (the same substitution as for F; the
//        trapezoid's v = 0 node has value 1 and weight STEP/2);
//   x >= 32  sqrt(pi/(2x)) sum_n a_n x^-n, a_0 = 1,
//        a_n = -a_{n-1} (2n - 1)^2 / (8 n), through a_5.
// ------------------------------------------------------------------------
template <typename R, int NT> __device__ inline R sg_G0_series(R x)
{
    const R y = x * x * R(0.25);
    const R Lg = log(x * R(0.5)) + R(SG_EULER_GAMMA);
    R tk = R(1), Hk = R(0), I0 = R(0), K0s = R(0);
#pragma unroll
    for (int k = 0; k < NT; ++k) {
        I0 += tk;
        K0s += Hk * tk;
        tk *= y * (R(1) / R((k + 1) * (k + 1)));
        Hk += R(1) / R(k + 1);
    }
    return exp(x) * (-Lg * I0 + K0s);
}

template <typename R> __device__ inline R sg_G0_quad(R x, const R *w)
{
    const R i2x = R(0.5) * sg_rcp(x);
    R acc = R(0.5);
#pragma unroll
    for (int k = 1; k <= FQuad<R>::NODES; ++k) {
        const R v2 = R(k * k) * (FQuad<R>::STEP * FQuad<R>::STEP);
        acc += w[k - 1] * sg_rsqrt(R(1) + v2 * i2x);
    }
    return acc * FQuad<R>::STEP * R(SG_SQRT2) * sg_rsqrt(x);
}

struct AsymCoefG0 {
    float c[6];
    constexpr AsymCoefG0() : c{}
    {
        double v = 1.0;
        c[0] = 1.0f;
        for (int n = 1; n < 6; ++n) {
            v = -v * (2.0 * n - 1.0) * (2.0 * n - 1.0) / (8.0 * n);
            c[n] = (float)v;
        }
    }
};

template <int FN> __device__ inline double sg_series64(double x)
{
    if constexpr (FN == SG_FN_G0) {
        return sg_G0_series<double, 5>(x);
    } else {
        double F, dF;
        sg_F_series<double, 5>(x, F, FN == SG_FN_D ? &dF : nullptr);
        if constexpr (FN == SG_FN_F) return F;
        else if constexpr (FN == SG_FN_D) return -x * dF - 1.5 * F;
        else return 2.0 * x * F - sg_G0_series<double, 5>(x);
    }
}

// Branches as in sg_F32: run only when some lane of the wave needs them.
__device__ inline float sg_G0_32(float x, const float *w)
{
    const bool ser = x < 1.0f, asy = x >= 32.0f, quad = !ser && !asy;
    float G = 0.0f;
    if (__any(ser)) {
        SG_NO_SPECULATE();
        const float t = sg_G0_series<float, 8>(x);
        G = ser ? t : G;
    }
    if (__any(quad)) {
        SG_NO_SPECULATE();
        const float t = sg_G0_quad<float>(x, w);
        G = quad ? t : G;
    }
    if (__any(asy)) {
        SG_NO_SPECULATE();
        constexpr AsymCoefG0 C;
        const float u = sg_rcp(x);
        float s = C.c[5];
#pragma unroll
        for (int n = 4; n >= 0; --n) s = s * u + C.c[n];
        const float t = float(SG_SQRT_PI / SG_SQRT2) * sg_rsqrt(x) * s;
        G = asy ? t : G;
    }
    return G;
}

// ------------------------------------------------------------------------
// Log-polar (App. C) kernels for H_f = h_f r, double precision:
//   h^2(X) = (h_a^2 e^{-X} + h_b^2 e^{X}) / 2,  x = (cosh X - cos phi)/(4 h^2),
//   K_r   = F(x) e^{-3X/2} h^{-3} (e^X - cos phi) / (8 sqrt(pi)),
//   K_phi = F(x) e^{-3X/2} h^{-3} sin phi / (8 sqrt(pi)),
// (App. C's L/(pi d^2) [e^{-X}/h^2]^{3/2} with L = sqrt(pi) x F(x), x = d^2/8).
// cosh X - cos phi = 2 sinh^2(X/2) + 2 sin^2(phi/2) and e^X - cos phi =
// expm1(X) + 2 sin^2(phi/2) avoid cancellation near the origin.
// which = 1, 2: derivatives with respect to h_a, h_b:
//   dK/d(h^2) = K-prefactor (h^2)^{-5/2} D(x), D = -x F'(x) - 3/2 F(x),
//   d(h^2)/dh_a = h_a e^{-X},  d(h^2)/dh_b = h_b e^{X}.
// sin(phi/2), sin(phi) are passed in so callers can use exact arguments.
// w: the table of F (which = 0) or D (which = 1, 2).
// ------------------------------------------------------------------------
// The factors of sg_conv_kernel64 (which = 0) that depend on the row alone
// (X, h_a, h_b): a semi-spectral operator row samples the kernel at N/2 + 1
// azimuths with these fixed, so they are formed once per row.
struct ConvRow64 {
    double two_sxh2;  // 2 sinh^2(X/2) = cosh X - 1
    double em1;       // e^X - 1
    double inv4h2;    // 1 / (4 h_ab^2(X))
    double pref;      // e^{-3X/2} / (8 sqrt(pi) h_ab^3)
};

// e^{X/2} and e^{-X/2} from one sinh (the larger as cosh + |sinh|, without
// cancellation, the other as its reciprocal).
__device__ inline void sg_exp_half(double X, double &s, double &ep, double &em)
{
    s = sinh(0.5 * X);
    const double big = sqrt(1.0 + s * s) + fabs(s), inv = 1.0 / big;
    ep = X >= 0.0 ? big : inv;
    em = X >= 0.0 ? inv : big;
}

__device__ inline ConvRow64 sg_conv_row64(double X, double ha, double hb)
{
    double s, ep, em;
    sg_exp_half(X, s, ep, em);
    const double rs = rsqrt(0.5 * (ha * ha * (em * em) + hb * hb * (ep * ep))), r2 = rs * rs;
    ConvRow64 c;
    c.two_sxh2 = 2.0 * s * s;
    c.em1 = 2.0 * s * ep;
    c.inv4h2 = 0.25 * r2;
    c.pref = em * em * em * (1.0 / (8.0 * SG_SQRT_PI)) * (r2 * rs);
    return c;
}

// sg_conv_kernel64 (which = 0) at one azimuth of a row.
__device__ inline void sg_conv_kernel64_row(const ConvRow64 &c, double sphi_half, double sphi, const double *w,
                                            double &Kr, double &Kp)
{
    const double two_s2 = 2.0 * sphi_half * sphi_half;
    const double p = sg_F64((c.two_sxh2 + two_s2) * c.inv4h2, w) * c.pref;
    Kr = p * (c.em1 + two_s2);
    Kp = p * sphi;
}

__device__ inline void sg_conv_kernel64(double X, double sphi_half, double sphi, double ha,
                                        double hb, int which, const double *w, double &Kr,
                                        double &Kp)
{
    double s, ep, em;
    sg_exp_half(X, s, ep, em);
    const double rs = rsqrt(0.5 * (ha * ha * (em * em) + hb * hb * (ep * ep))), r2 = rs * rs;
    const double two_s2 = 2.0 * sphi_half * sphi_half;
    const double x = 0.25 * (2.0 * s * s + two_s2) * r2;  // (cosh X - cos phi) / (4 h^2)
    const double emc = 2.0 * s * ep + two_s2;             // e^X - cos phi
    double p = em * em * em * (1.0 / (8.0 * SG_SQRT_PI)) * (r2 * rs);
    if (which == 0)
        p *= sg_F64(x, w);
    else
        p *= sg_D64(x, w) * r2 * (which == 1 ? ha * (em * em) : hb * (ep * ep));
    Kr = p * emc;
    Kp = p * sphi;
}

// Both h derivatives at once (one D evaluation per azimuth): the row's
// factors and one sample, (Kr1, Kp1) = d/dh_a, (Kr2, Kp2) = d/dh_b, as
// sg_conv_kernel64 with which = 1 and 2.
struct ConvRowDh64 {
    double two_sxh2, em1, inv4h2;  // as in ConvRow64
    double p1, p2;                 // e^{-3X/2} / (8 sqrt(pi) h^5) times d(h^2)/dh_a, d(h^2)/dh_b
};

__device__ inline ConvRowDh64 sg_conv_row64_dh(double X, double ha, double hb)
{
    double s, ep, em;
    sg_exp_half(X, s, ep, em);
    const double rs = rsqrt(0.5 * (ha * ha * (em * em) + hb * hb * (ep * ep))), r2 = rs * rs;
    const double g = em * em * em * (1.0 / (8.0 * SG_SQRT_PI)) * (r2 * r2 * rs);
    ConvRowDh64 c;
    c.two_sxh2 = 2.0 * s * s;
    c.em1 = 2.0 * s * ep;
    c.inv4h2 = 0.25 * r2;
    c.p1 = g * ha * (em * em);
    c.p2 = g * hb * (ep * ep);
    return c;
}

__device__ inline void sg_conv_kernel64_dh(const ConvRowDh64 &c, double sphi_half, double sphi, const double *w,
                                           double &Kr1, double &Kp1, double &Kr2, double &Kp2)
{
    const double two_s2 = 2.0 * sphi_half * sphi_half, emc = c.em1 + two_s2;
    const double D = sg_D64((c.two_sxh2 + two_s2) * c.inv4h2, w);
    const double d1 = D * c.p1, d2 = D * c.p2;
    Kr1 = d1 * emc;
    Kp1 = d1 * sphi;
    Kr2 = d2 * emc;
    Kp2 = d2 * sphi;
}

// X-symmetrised radial kernel used by the self-cell average.
__device__ inline double sg_sym_kr64(double X, double phi, double ha, double hb, int which,
                                     const double *w)
{
    const double sh = sin(0.5 * phi), s = sin(phi);
    double k1, k2, t;
    sg_conv_kernel64(X, sh, s, ha, hb, which, w, k1, t);
    sg_conv_kernel64(-X, sh, s, ha, hb, which, w, k2, t);
    return 0.5 * (k1 + k2);
}
