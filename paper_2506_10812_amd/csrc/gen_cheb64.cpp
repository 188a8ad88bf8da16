// gen_cheb64.cpp -- host build step: writes the tables of sg_cheb64.h.
//
// The kernel functions (the force kernel's of Sect. 2.2 and App. A, its
// derivative's and the potential kernel's of Sect. 5.5) are
//     F(x)  = e^x [K1(x) - K0(x)],   G0(x) = e^x K0(x),
//     D(x)  = -x F'(x) - 3/2 F(x),   E(x)  = 2 x F(x) - G0(x).
// Values come from the integral representation of the Macdonald functions,
// K_nu(x) = int_0^inf e^{-x cosh t} cosh(nu t) dt, which gives
//     F(x)  =  int_0^inf e^{-x (cosh t - 1)} (cosh t - 1) dt,
//     F'(x) = -int_0^inf e^{-x (cosh t - 1)} (cosh t - 1)^2 dt,
//     D(x)  = -1/2 int_0^inf e^{-x (cosh t - 1)} tanh^3(t/2) sinh t dt
//             (the two terms of D cancel to O(1/x) of themselves, the integral
//             does not),
//     G0(x) =  int_0^inf e^{-x (cosh t - 1)} dt,
//     E(x)  =  int_0^inf e^{-x (cosh t - 1)} (2 x (cosh t - 1) - 1) dt,
// evaluated in long double with the trapezoid rule: the integrands are even,
// entire and decay doubly exponentially, so the rule converges geometrically
// in 1/step (step 1/64 here, far below what 64-bit mantissas need).
//
// The tables (all of the header, written with --header):
//   sg_poly64   F, D, G0, E: PSUB intervals per octave from 2^POCT0 to
//               2^POCT1, PNC monomial coefficients each in the local variable
//               t in [-1, 1), from the Chebyshev interpolant on the interval
//               (its last coefficients are checked to be below 1e-15 of the
//               value; the dropped ones are below 3e-17);
//   sg_polyu64  V(u) = u^{-3/2} F(1/u) and Vg(u) = u^{-1/2} G0(1/u) of the
//               direct sums likewise, on the octaves of u = 1/x from 2^UOCT0 to
//               2^UOCT1;
//   sg_polyu32  the same in float, FSUB intervals per octave with FNC terms;
//   sg_tw64     the double twiddles of the table builds' transforms.
// Without --header they follow Chebyshev series of F, F' and G0 on the dyadic
// intervals [2^(k-1), 2^k), k = 0 .. NI - 1 (M = 27 terms from the discrete
// cosine transform at NN points of the first kind, truncated below 1e-17 of
// an interval's largest value), which check the integrals' evaluation over
// whole octaves; the library does not use them.
#include <cmath>
#include <cstdio>
#include <cstdlib>

static const int NI = 6;   // intervals [1/2,1), [1,2), [2,4), ..., [16,32)
static const int M = 27;   // terms kept
static const int NN = 48;  // Chebyshev points per interval

static const int PSUB = 8, POCT0 = -4, POCT1 = 8, PNC = 12, PNN = 24;

// F, D, G0 and E by the same trapezoid rule.
static void fdg(long double x, long double (&v)[4])
{
    const long double h = 1.0L / 64.0L;
    v[0] = v[1] = v[2] = v[3] = 0.0L;
    for (int k = 0;; ++k) {
        const long double t = k * h, sh = sinhl(0.5L * t), th = tanhl(0.5L * t);
        const long double c = 2.0L * sh * sh, e = expl(-x * c) * (k == 0 ? 0.5L : 1.0L) * h;
        v[0] += e * c;
        v[1] -= 0.5L * e * th * th * th * sinhl(t);
        v[2] += e;
        v[3] += e * (2.0L * x * c - 1.0L);
        if (x * c > 60.0L) break;
    }
}

static const int UOCT0 = -8, UOCT1 = 4;               // double: PSUB intervals, PNC terms
static const int FSUB = 4, FOCT0 = -6, FOCT1 = 4, FNC = 7;  // float, rows of FNC + 1

// Monomial coefficients of the NF functions' fits on the interval [a, a + w);
// tol: largest last coefficient over the function's value.
template <int NF, int NC, typename Fn>
static bool poly_fit(Fn fn, long double a, long double w, long double tol, double (&out)[NF][NC])
{
    const long double pi = 3.141592653589793238462643383279502884L;
    long double val[NF][PNN], top[NF] = {};
    for (int j = 0; j < PNN; ++j) {
        long double v[NF];
        fn(a + 0.5L * w * (1.0L + cosl(pi * (j + 0.5L) / PNN)), v);
        for (int f = 0; f < NF; ++f) {
            val[f][j] = v[f];
            top[f] = fmaxl(top[f], fabsl(v[f]));
        }
    }
    for (int f = 0; f < NF; ++f) {
        long double mono[NC] = {}, t0[NC] = {}, t1[NC] = {}, last = 0.0L;
        t0[0] = 1.0L;
        t1[1] = 1.0L;
        for (int m = 0; m < NC; ++m) {
            long double c = 0.0L;
            for (int j = 0; j < PNN; ++j) c += val[f][j] * cosl(pi * m * (j + 0.5L) / PNN);
            c *= (m == 0 ? 1.0L : 2.0L) / PNN;
            last = c;
            for (int i = 0; i < NC; ++i) mono[i] += c * t0[i];
            long double t2[NC];  // T_{m+2} = 2 t T_{m+1} - T_m
            for (int i = 0; i < NC; ++i) t2[i] = (i ? 2.0L * t1[i - 1] : 0.0L) - t0[i];
            for (int i = 0; i < NC; ++i) {
                t0[i] = t1[i];
                t1[i] = t2[i];
            }
        }
        if (fabsl(last) > tol * top[f]) return false;  // the next one is 34 (float: 18) times smaller
        for (int i = 0; i < NC; ++i) out[f][i] = (double)mono[i];
    }
    return true;
}

static void fdf(long double x, long double &F, long double &dF, long double &G)
{
    const long double h = 1.0L / 64.0L;
    long double s = 0.0L, sd = 0.0L, sg = 0.0L;
    for (int k = 0;; ++k) {
        const long double t = k * h;
        const long double sh = sinhl(0.5L * t);
        const long double c = 2.0L * sh * sh;  // cosh t - 1 without the cancellation
        const long double e = expl(-x * c);
        const long double wgt = k == 0 ? 0.5L : 1.0L;
        s += wgt * e * c;
        sd += wgt * e * c * c;
        sg += wgt * e;
        if (x * c > 60.0L) break;  // e^{-60} ~ 1e-26
    }
    F = s * h;
    dF = -sd * h;
    G = sg * h;
}

int main(int argc, char **)
{
    const bool header = argc > 1;  // --header
    static double cf[NI][M], cd[NI][M], cg[NI][M];
    const long double pi = 3.141592653589793238462643383279502884L;
    for (int k = 0; k < NI; ++k) {
        const long double a = ldexpl(1.0L, k - 1);
        long double fv[NN], dv[NN], gv[NN];
        long double fmax = 0.0L, dmax = 0.0L, gmax = 0.0L;
        for (int j = 0; j < NN; ++j) {
            const long double t = cosl(pi * (j + 0.5L) / NN);
            fdf(a * (3.0L + t) / 2.0L, fv[j], dv[j], gv[j]);
            fmax = fmaxl(fmax, fabsl(fv[j]));
            dmax = fmaxl(dmax, fabsl(dv[j]));
            gmax = fmaxl(gmax, fabsl(gv[j]));
        }
        for (int m = 0; m < M; ++m) {
            long double sf = 0.0L, sd = 0.0L, sg = 0.0L;
            for (int j = 0; j < NN; ++j) {
                const long double c = cosl(pi * m * (j + 0.5L) / NN);
                sf += fv[j] * c;
                sd += dv[j] * c;
                sg += gv[j] * c;
            }
            const long double sc = (m == 0 ? 1.0L : 2.0L) / NN;
            cf[k][m] = (double)(sf * sc);
            cd[k][m] = (double)(sd * sc);
            cg[k][m] = (double)(sg * sc);
        }
        // the dropped tail: the last kept terms bound it (geometric decay)
        if (fabsl((long double)cf[k][M - 1]) > 1e-17L * fmax || fabsl((long double)cd[k][M - 1]) > 1e-17L * dmax ||
            fabsl((long double)cg[k][M - 1]) > 1e-17L * gmax) {
            fprintf(stderr, "gen_cheb64: interval %d: last coefficients %g %g %g too large\n", k, cf[k][M - 1],
                    cd[k][M - 1], cg[k][M - 1]);
            return 1;
        }
    }
    printf("// sg_cheb64.h -- written by gen_cheb64.cpp at build time; do not edit.\n");
    printf("#pragma once\n");
    if (!header) printf("#define SG_CHEB_NI %d\n#define SG_CHEB_M %d\n", NI, M);
    const char *names[3] = {"sg_cheb_f", "sg_cheb_df", "sg_cheb_g0"};
    double(*tabs[3])[M] = {cf, cd, cg};
    for (int q = 0; q < 3 && !header; ++q) {
        printf("static constexpr double %s[SG_CHEB_NI * SG_CHEB_M] = {\n", names[q]);
        for (int k = 0; k < NI; ++k)
            for (int m = 0; m < M; ++m) printf("    %.17e,\n", tabs[q][k][m]);
        printf("};\n");
    }
    const int pni = (POCT1 - POCT0) * PSUB;
    printf("#define SG_POLY_SUB %d\n#define SG_POLY_OCT0 %d\n#define SG_POLY_NI %d\n#define SG_POLY_NC %d\n", PSUB, POCT0,
           pni, PNC);
    static double poly[4][(POCT1 - POCT0) * PSUB][PNC];
    for (int i = 0; i < pni; ++i) {
        const long double oct = ldexpl(1.0L, POCT0 + i / PSUB), w = oct / PSUB;
        double c[4][PNC];
        if (!poly_fit<4, PNC>([](long double x, long double(&v)[4]) { fdg(x, v); }, oct + w * (i % PSUB), w, 1e-15L,
                              c)) {
            fprintf(stderr, "gen_cheb64: local polynomial %d: truncation too large\n", i);
            return 1;
        }
        for (int f = 0; f < 4; ++f)
            for (int m = 0; m < PNC; ++m) poly[f][i][m] = c[f][m];
    }
    // one array [F, D, G0, E][interval][coefficient]
    printf("static __device__ const double sg_poly64[4 * SG_POLY_NI * SG_POLY_NC] = {\n");
    for (int f = 0; f < 4; ++f)
        for (int i = 0; i < pni; ++i)
            for (int m = 0; m < PNC; ++m) printf("    %.17e,\n", poly[f][i][m]);
    printf("};\n");
    auto vvg = [](long double u, long double(&v)[2]) {
        long double f[4];
        fdg(1.0L / u, f);
        v[0] = f[0] / (u * sqrtl(u));
        v[1] = f[2] / sqrtl(u);
    };
    const int uni = (UOCT1 - UOCT0) * PSUB, fni = (FOCT1 - FOCT0) * FSUB;
    static double pu[2][(UOCT1 - UOCT0) * PSUB][PNC];
    static double pf[2][(FOCT1 - FOCT0) * FSUB][FNC];
    for (int i = 0; i < uni; ++i) {
        const long double oct = ldexpl(1.0L, UOCT0 + i / PSUB), w = oct / PSUB;
        double c[2][PNC];
        if (!poly_fit<2, PNC>(vvg, oct + w * (i % PSUB), w, 1e-15L, c)) {
            fprintf(stderr, "gen_cheb64: V polynomial %d: truncation too large\n", i);
            return 1;
        }
        for (int f = 0; f < 2; ++f)
            for (int m = 0; m < PNC; ++m) pu[f][i][m] = c[f][m];
    }
    for (int i = 0; i < fni; ++i) {
        const long double oct = ldexpl(1.0L, FOCT0 + i / FSUB), w = oct / FSUB;
        double c[2][FNC];
        if (!poly_fit<2, FNC>(vvg, oct + w * (i % FSUB), w, 1e-7L, c)) {
            fprintf(stderr, "gen_cheb64: float V polynomial %d: truncation too large\n", i);
            return 1;
        }
        for (int f = 0; f < 2; ++f)
            for (int m = 0; m < FNC; ++m) pf[f][i][m] = c[f][m];
    }
    printf("#define SG_POLYU_OCT0 %d\n#define SG_POLYF_SUB %d\n#define SG_POLYF_OCT0 %d\n#define SG_POLYF_NI %d\n"
           "#define SG_POLYF_NC %d\n", UOCT0, FSUB, FOCT0, fni, FNC);
    printf("static __device__ const double sg_polyu64[2 * SG_POLY_NI * SG_POLY_NC] = {\n");
    for (int f = 0; f < 2; ++f)
        for (int i = 0; i < uni; ++i)
            for (int m = 0; m < PNC; ++m) printf("    %.17e,\n", pu[f][i][m]);
    printf("};\n");
    printf("static __device__ const float sg_polyu32[2 * SG_POLYF_NI * (SG_POLYF_NC + 1)] = {\n");
    for (int f = 0; f < 2; ++f)
        for (int i = 0; i < fni; ++i) {
            for (int m = 0; m < FNC; ++m) printf("    %.9ef,\n", pf[f][i][m]);
            printf("    0.0f,\n");
        }
    printf("};\n");
    // cos and sin of 2 pi k / 4096 (the first octant's values, mirrored)
    printf("#define SG_TW64_N 4096\nstatic __device__ const double sg_tw64[2 * SG_TW64_N] = {\n");
    for (int k = 0; k < 4096; ++k) {
        const long double a = 2.0L * pi / 4096.0L;
        const int q = k % 1024, m = q <= 512 ? q : 1024 - q;
        long double c = cosl(a * m), sn = sinl(a * m);
        if (q > 512) {
            const long double t = c;
            c = sn;
            sn = t;
        }
        const long double x[4] = {c, -sn, -c, sn}, y[4] = {sn, c, -sn, -c};
        printf("    %.17e, %.17e,\n", (double)x[k / 1024], (double)y[k / 1024]);
    }
    printf("};\n");
    return 0;
}
