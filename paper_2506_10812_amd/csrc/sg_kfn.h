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
//     and E(x) = 2 x F - G0 (its derivative).  The series of D and E begin at
//     n = 1 and so go through n = 9: first omitted terms 1.3e-17 and 2e-18 of
//     them (through n = 7 3e-14 and 5e-15).  A block copies the one table
//     it needs (9 KB) into LDS.  Per wave an evaluation is 12 LDS reads and 11
//     FMAs in a dependent chain; the Chebyshev series of 27 terms used before
//     took 27 reads and 53 operations, and below 32 only.
//   The direct sums (float and double) evaluate many pairs per wave and take
//   F as F(x) h^-3 = s'^-3 V(u), u = 1/x = h^2/s'^2 (s'^2 = s^2/8), V(u) =
//   u^{-3/2} F(1/u): one reciprocal square root per source serves every pair
//   of fluids.  V (and Vg(u) = u^{-1/2} G0(1/u) for the potential) has local
//   polynomials on the octaves of u, the asymptotic series' polynomial in u
//   below them and the power series above.  Float F and G0 follow from V, Vg;
//   float V is within 1.2e-7.
#pragma once
#include "sg_internal.h"
#include "sg_cheb64.h"

#define SG_EULER_GAMMA 0.57721566490153286061

// LDS tables of TABLE entries: the local polynomials of one function.
enum { SG_FN_F = 0, SG_FN_D = 1, SG_FN_G0 = 2, SG_FN_E = 3 };  // of x, double
enum { SG_FN_V = 0, SG_FN_VG = 1 };                            // of u = 1/x
template <typename R> struct FQuad;
template <> struct FQuad<double> {
    static constexpr int TABLE = SG_POLY_NI * SG_POLY_NC;
};
template <> struct FQuad<float> {
    static constexpr int TABLE = SG_POLYF_NI * (SG_POLYF_NC + 1);
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
// The same for V (fn = SG_FN_V) or Vg.
__device__ inline void sg_fill_v(double *w, int fn)
{
    for (int k = threadIdx.x; k < FQuad<double>::TABLE; k += blockDim.x) w[k] = sg_polyu64[fn * FQuad<double>::TABLE + k];
}
__device__ inline void sg_fill_v(float *w, int fn)
{
    for (int k = threadIdx.x; k < FQuad<float>::TABLE; k += blockDim.x) w[k] = sg_polyu32[fn * FQuad<float>::TABLE + k];
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

// Asymptotic coefficients n = 0..N-1 of F / ((sqrt(2 pi)/4) x^{-3/2}), of D over
// the same (n c_n), of G0 / sqrt(pi/(2x)) (a_n = -a_{n-1} (2n - 1)^2/(8n)) and
// of E over the same (c_n - a_n).
template <int FN> struct Asym64 {
    static constexpr int N = FN == SG_FN_F || FN == SG_FN_G0 ? 8 : 10;
    double c[N];
    constexpr Asym64() : c{}
    {
        double v = 1.0, g = 1.0;
        for (int n = 0; n < N; ++n) {
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
        double s = A.c[A.N - 1];
#pragma unroll
        for (int n = A.N - 2; n >= 0; --n) s = fma(s, u, A.c[n]);
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

// ------------------------------------------------------------------------
// G0(x) = e^x K0(x), the kernel of the conservative potential (Sect. 5.5,
// appendix "Conservative force"): P_ab(s) = -G0(d^2/8) / (2 sqrt(pi) H_ab).
// Double: sg_fn64 above; both types: Vg below.
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

// ------------------------------------------------------------------------
// V(u) and Vg(u), u = 1/x > 0; w: the table of fn.  u below the polynomials
// (x > 256, float 64) takes the asymptotic series, alone when the whole wave
// is there; u >= 16 (x <= 1/16) the power series.
// ------------------------------------------------------------------------
template <int FN, typename R> __device__ inline R sg_v_asym(R u)
{
    constexpr int NT = sizeof(R) == 8 ? 8 : 5;
    constexpr Asym64<FN == SG_FN_V ? SG_FN_F : SG_FN_G0> A;
    R s = R(A.c[NT - 1]);
#pragma unroll
    for (int n = NT - 2; n >= 0; --n) s = s * u + R(A.c[n]);
    return s * R(FN == SG_FN_V ? SG_SQRT2 * SG_SQRT_PI * 0.25 : SG_SQRT_PI / SG_SQRT2);
}

template <int FN, typename R> __device__ inline R sg_v_series(R u)
{
    const R x = sg_rcp(u);
    if constexpr (FN == SG_FN_VG) {
        return sqrt(x) * sg_G0_series<R, 5>(x);
    } else {
        R F;
        sg_F_series<R, 5>(x, F, (R *)nullptr);
        return x * sqrt(x) * F;
    }
}

template <int FN> __device__ inline double sg_v(double u, const double *w)
{
    constexpr double lo = SG_POLYU_OCT0 == -8 ? 0x1p-8 : -1.0;
    static_assert(lo > 0.0 && SG_POLY_SUB == 8 && SG_POLY_NC == 12, "index arithmetic below");
    if (__all(u < lo)) return sg_v_asym<FN>(u);
    const int hi = __double2hiint(u);
    const int k = min(max((hi >> 17) - ((1023 + SG_POLYU_OCT0) << 3), 0), SG_POLY_NI - 1);
    const double t = fma(16.0, __hiloint2double((hi & 0x1ffff) | 0x3ff00000, __double2loint(u)), -17.0);
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
    if (__any(u < lo)) {
        SG_NO_SPECULATE();
        const double s = sg_v_asym<FN>(u);
        f = u < lo ? s : f;
    }
    if (__any(!(u < 16.0))) {  // NaN included
        SG_NO_SPECULATE();
        const double s = sg_v_series<FN>(u);
        f = u < 16.0 ? f : s;
    }
    return f;
}

template <int FN> __device__ inline float sg_v(float u, const float *w)
{
    constexpr float lo = SG_POLYF_OCT0 == -6 ? 0x1p-6f : -1.0f;
    static_assert(lo > 0.0f && SG_POLYF_SUB == 4 && SG_POLYF_NC == 7, "index arithmetic below");
    if (__all(u < lo)) return sg_v_asym<FN>(u);
    const int bits = __float_as_int(u);
    const int k = min(max((bits >> 21) - ((127 + SG_POLYF_OCT0) << 2), 0), SG_POLYF_NI - 1);
    // the 2 leading mantissa bits are in k; the rest as v in [1, 1 + 1/4), t = 8 v - 9
    const float t = fmaf(8.0f, __int_as_float((bits & 0x1fffff) | 0x3f800000), -9.0f);
    const float4 *c = (const float4 *)(w + k * (SG_POLYF_NC + 1));
    const float4 c0 = c[0], c1 = c[1];
    float f = c1.z;
    f = fmaf(f, t, c1.y);
    f = fmaf(f, t, c1.x);
    f = fmaf(f, t, c0.w);
    f = fmaf(f, t, c0.z);
    f = fmaf(f, t, c0.y);
    f = fmaf(f, t, c0.x);
    if (__any(u < lo)) {
        SG_NO_SPECULATE();
        const float s = sg_v_asym<FN>(u);
        f = u < lo ? s : f;
    }
    if (__any(!(u < 16.0f))) {  // NaN included
        SG_NO_SPECULATE();
        const float s = sg_v_series<FN>(u);
        f = u < 16.0f ? f : s;
    }
    return f;
}

// Float F(x) and G0(x) over the whole range of x; w: the table of V or Vg.
// The power series gives them below 1/16: u^{3/2} overflows from x = 2e-26 down.
__device__ inline float sg_F32(float x, const float *w)
{
    const bool ser = x < 0.0625f;
    const float u = sg_rcp(x);
    float f = u * sg_rsqrt(x) * sg_v<SG_FN_V>(ser ? 1.0f : u, w);
    if (__any(ser)) {
        SG_NO_SPECULATE();
        float s;
        sg_F_series<float, 5>(x, s, nullptr);
        f = ser ? s : f;
    }
    return f;
}
__device__ inline float sg_G0_32(float x, const float *w)
{
    const bool ser = x < 0.0625f;
    float g = sg_rsqrt(x) * sg_v<SG_FN_VG>(ser ? 1.0f : sg_rcp(x), w);
    if (__any(ser)) {
        SG_NO_SPECULATE();
        const float s = sg_G0_series<float, 5>(x);
        g = ser ? s : g;
    }
    return g;
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

// The row of one of K, dK/dh_a, dK/dh_b (which = 0, 1, 2): K_r = fn(x) pref
// (e^X - cos phi) with fn = F or D.
__device__ inline ConvRow64 sg_conv_row64(double X, double ha, double hb, int which)
{
    if (which == 0) return sg_conv_row64(X, ha, hb);
    const ConvRowDh64 d = sg_conv_row64_dh(X, ha, hb);
    ConvRow64 c;
    c.two_sxh2 = d.two_sxh2;
    c.em1 = d.em1;
    c.inv4h2 = d.inv4h2;
    c.pref = which == 1 ? d.p1 : d.p2;
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
