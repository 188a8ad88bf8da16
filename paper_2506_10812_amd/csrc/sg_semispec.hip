// sg_semispec.hip -- the semi-spectral solver: azimuthal FFT plus a direct
// radial sum per azimuthal mode (Sect. 5.2), for scale heights that are any
// function of radius (it lifts the H = h r condition of the full log-polar
// FFT, whose cost App. D quantifies).
//
// With H_a = H_a(r) the kernel between source ring i' and target ring i
// still depends on the azimuths only through phi = phi_target - phi_source,
// so for every ring pair the field is a circular convolution in phi:
//   g_c^{b}(i, j) = - du dphi sum_a sum_i' sum_j' Sigma_a(i', j')
//                   K_c(X_ii', (j - j') dphi; h_a = H_a(r_i')/r_i', h_b = H_b(r_i)/r_i)
// with X_ii' = u_i - u_i' and K_c the convolution-form kernels of App. C
// (there with constant h; the pair enters them only through
// h_ab^2 = (h_a^2 e^{-X} + h_b^2 e^X)/2 = H_ab^2 / (r r'), so the same
// formulas hold ring by ring).  In phi-Fourier space mode m decouples:
//   g^_c^{b}(m, i) = sum_a sum_i' T_c^{ab}(m, i, i') Sigma~_a(m, i'),
// an n_r x n_r operator per (m, pair).  K_r is even and K_phi odd in phi, so
// T_r is real and T_phi = i t_phi with t_phi real.
//
// Table (sg_ss_table, double precision, rounded to float at the end):
//   1. self-cell averages Kbar_r per (pair, ring) with h = H/r at the ring
//      (offset X = 0, phi = 0; zero with SG_SELF_CELL_EXCLUDE);
//   2. per row (b, a, i', i): samples K_r + i K_phi at phi = q dphi for
//      q <= n_phi/2, mirrored (K_r even, K_phi odd), one complex transform
//      (shared by two rows, whose transforms are real),
//      T_r(m) = (Z[m] + Z[-m])/2, t_phi(m) = (Z[-m] - Z[m])/2,
//      scaled by -du dphi / n_phi (the inverse transform of the last pass is
//      unnormalised); rows are written [row][m] to a chunk buffer.  Ring
//      pairs far apart take fewer samples (SsClass below);
//   3. a tiled transpose moves each chunk into the table: full modes keep
//      every (i', i) entry, banded modes the diagonals |i' - i| <= w (the
//      band rule is in sg_internal.h; dropped couplings are below about
//      2^-30 of the axisymmetric one, and SG_SS_FULL keeps every entry).
// SG_INDIRECT folds the indirect term (Sect. 5.4 and its appendix) into
// mode 1: in the same convolution form it is Sigma convolved with
//   r_i'^2 sqrt(2) K_a(d_i') (cos phi, -sin phi),  d_i' = r_i' / H_a(r_i'),
// whose transform at m = 1 adds r_i'^2 sqrt(2) K_a(d) n_phi / 2 to both T_r
// and t_phi before scaling.
//
// SG_POTENTIAL builds the operators of the potential instead (Sect. 5.5 and
// the appendix on the conservative force): Phi_b(i, j) = sum Sigma_a A_i'
// P_ab(s), P_ab = -e^y K0(y) / (2 sqrt(pi) H_ab), y = s^2 / (8 H_ab^2), with
// the own-cell integral of P at zero offset.  P is even in phi, so T_r carries
// its real spectrum and t_phi = 0: the solve writes Phi to g_r (and rounding
// noise of the inverse transform to g_phi).
//
// Solve (sg_field_fft with discs flagged SG_SEMI_SPECTRAL): pass 1 and pass 3
// of the FFT path (phi transforms), and k_ss_pass in place of pass 2.
#include <algorithm>
#include <vector>

#include "sg_kfn.h"
#include "sg_semispec.h"
#include "sg_adjoint.h"
#include "sg_table.h"
#include "sg_hat.h"

// ------------------------------------------------------------ table: rows
struct SsRowArgs {
    int nr, nrt, nf, excl, ind, pot, lin, second;
    double lnrmin, du, dphi, rmin, dr;  // du: log grid; rmin, dr: uniform radial grid
    GLNodes gl;                         // second: the polar rules' nodes
};

// SG_SECOND_ORDER rows: the sample at (P, q) = (i - i', q) becomes the
// hat-weighted weight W_c(P, q) of the FFT path's table with the row's
// aspect ratios h_a = H_a(r_i')/r_i', h_b = H_b(r_i)/r_i held across the hat
// (for H = h r this is the FFT path's table; otherwise the variation of h
// across the hat is odd in s and enters at second order only).  Within
// SG_SS_HAT_NEAR of the larger cell side from the singular point the weight
// is integrated (sg_hat_weight_part); beyond, it is the point value plus the
// second moments of the hats, W = K + (D_X^2 K + D_phi^2 K)/12, with central
// second differences over one cell (D_phi from the neighbouring samples of
// the row, D_X from two extra samples at X +- du): the remainder is
// O((cell/distance)^4), below 3e-6 of the entry at 32 cells.  The integrated
// samples are computed by the whole group, one after the other (each
// thread takes every T-th quadrature node; the owner of the sample adds the
// parts in thread order), so that no single lane carries a polar rule.
#define SG_SS_HAT_NEAR 32.0

// Band-limited rows.  The kernels between rings |X| apart are analytic in phi
// within |Im phi| < |X|, so their Fourier coefficients fall off as e^{-m|X|}
// and M samples give every mode m <= M/2 to e^{-(M-m)|X|} of the axisymmetric
// coupling.  A row takes the smallest power of two M >= SG_SS_MIN_M with
// M |X| >= SG_SS_ALIAS instead of n_phi samples: aliases and the modes above
// M/2, which stay zero, are below e^{-40} = 4e-18, under the rounding of a
// double transform.  Most ring pairs are far apart: on the 1200 x 2048 grid
// the rows take 0.17 of the samples.  SG_SS_FULL keeps n_phi throughout.
//
// The rows of one M form a class: by units of SG_SS_TI consecutive target
// rings i (tile t) at one offset k = i' - i, whose last ring lies
// x1 <= |X| < x2 from its source ring (on the log grid |X| = |k| du for the
// whole unit; on a uniform grid |X| falls with i, so the last is the
// nearest).  Row index = ((pair n_t + t) n_k + offset) SG_SS_TI + i % SG_SS_TI:
// rows of a unit are consecutive entries of a diagonal in the banded modes'
// layout, and the units of one tile lie together for the full modes' (the
// scatter goes through them in that order).
// The gradient's rows, whose result is a double, take 96: aliases below e^{-48}.
// (A margin: the h derivatives' singularities at phi = +-i X are simple poles
// like the kernel's, and e^{-40} would do; the table's derivative rows take 80.)
#define SG_SS_ALIAS_GRAD 96.0
#define SG_SS_TI 16

struct SsClass {
    int on;          // 0: every row, in the plain (b, a, i', i) order
    int nt;          // tiles of target rings
    int K1, K2;      // |k| of the class in [K1, K2) (K1 = 0: all of -K2 < k < K2)
    int nk;          // offsets: 2 K2 - 1 or 2 (K2 - K1); half: K2 - K1
    int half;        // offsets k >= 0 only
    double x1, x2;   // the class's range of |X| (x2 infinite in the last)
};

__device__ inline int ss_class_offset(const SsClass &C, int q)
{
    if (C.half) return C.K1 + q;
    if (C.K1 == 0) return q - (C.K2 - 1);
    const int half = C.K2 - C.K1;
    return q < half ? C.K1 + q : -(C.K1 + q - half);
}

// |X| of the last ring of tile t at offset k on a uniform grid (infinite where
// the source ring would lie inside the centre).
__device__ __host__ inline double ss_tile_dist(double rmin, double dr, int t, int k)
{
    const double r = rmin + (t * SG_SS_TI + (SG_SS_TI - 0.5)) * dr, rp = r + k * dr;
    return rp > 0.0 ? fabs(log(rp / r)) : INFINITY;
}

template <int N> struct SsRowShape {
    static constexpr int P = FftShape<N>::P, T = FftShape<N>::T;
    static constexpr int WGS = T > 256 ? T : 256;
    static constexpr int G = WGS / T;
};

// sin and cos of half the azimuth 2 pi q / N, q <= N/2.
template <int N> __device__ inline void ss_half_angle(int q, double &s, double &c)
{
    static_assert(SG_TW64_N % (2 * N) == 0, "sine table");
    const double2 v = ((const double2 *)sg_tw64)[q * (SG_TW64_N / (2 * N))];
    c = v.x;
    s = v.y;
}

// Whether tile t at offset k belongs to the class.
__device__ inline bool ss_in_class(const SsRowArgs &A, const SsClass &C, int t, int k)
{
    const int ak = abs(k);
    if (ak < C.K1 || ak >= C.K2) return false;
    if (!A.lin) return true;
    const double x = ss_tile_dist(A.rmin, A.dr, t, k);
    return x >= C.x1 && x < C.x2;
}

// Row idx of a class (or of the plain order): its ring pair.  False where
// there is none (the caller drops the row; in the plain order i may be the
// padding column of an odd n_r).
__device__ inline bool ss_row(const SsRowArgs &A, const SsClass &C, uint32_t idx, int &b, int &a, int &ip, int &i)
{
    uint32_t rest;  // (at most 16 pairs x 2048 rings x 4095 offsets)
    bool ok = true;
    if (!C.on) {
        i = (int)(idx % A.nrt);
        rest = idx / A.nrt;
        ip = (int)(rest % A.nr);
        rest /= A.nr;
    } else {
        const uint32_t unit = idx / SG_SS_TI;
        const int k = ss_class_offset(C, (int)(unit % C.nk));
        rest = unit / C.nk;
        const int t = (int)(rest % C.nt);
        rest /= C.nt;
        i = t * SG_SS_TI + (int)(idx % SG_SS_TI);
        ip = i + k;
        ok = i < A.nr && ip >= 0 && ip < A.nr && ss_in_class(A, C, t, k);
    }
    a = (int)(rest % A.nf);
    b = (int)(rest / A.nf);
    return ok && b < A.nf;
}

// Second-order sample away from the singular point: the point value plus the
// second moments of the hats, W = K + (D_X^2 K + D_phi^2 K)/12.
__device__ inline void ss_far_weight(const ConvRow64 &c0, const ConvRow64 &c1, const ConvRow64 &c2, double phi_pi,
                                     double step_pi, const double *wq, double &kr, double &kp)
{
    double r[5], p[5];
#pragma unroll 1
    for (int k = 0; k < 5; ++k) {
        double sh, ch;  // half angle
        sincospi(0.5 * (phi_pi + (k == 3 ? step_pi : k == 4 ? -step_pi : 0.0)), &sh, &ch);
        sg_conv_kernel64_row(k == 1 ? c1 : k == 2 ? c2 : c0, sh, 2.0 * sh * ch, wq, r[k], p[k]);
    }
    kr = r[0] + (r[1] + r[2] + r[3] + r[4] - 4.0 * r[0]) / 12.0;
    kp = p[0] + (p[1] + p[2] + p[3] + p[4] - 4.0 * p[0]) / 12.0;
}

// A group of T threads takes RPG consecutive rows r0 + row of a class (or of
// the plain (b, a, i', i) order, i fastest).  Point-sampled rows go two to a group (RPG = 2): a row's
// samples z = K_r + i K_phi are Hermitian in phi, so its transform Z is real,
// and the group transforms z_A + i z_B once, reading Z_A from the real part
// and Z_B from the imaginary part.  The row count is even (n_rt is) and so
// is every chunk, so the two rows are always i and i + 1 of one (b, a, i').
// N: the samples of the rows, n_phi or a class's M.  SO: 0 point samples; 1
// second-order rows with samples to integrate (one row per group), 3 the same
// on long cells (sg_hat_long); 2 second-order rows beyond SG_SS_HAT_NEAR, whose
// samples are the weights of ss_far_weight.  out: [nrows][mc] float2 (T_r, t_phi), m < mc <= N/2 + 1.
template <int N, int SO>
__global__ void __launch_bounds__(SsRowShape<N>::WGS)
k_ss_rows(const double *H, const double *self, SsRowArgs A, SsClass C, size_t r0, int nrows, int mc, float2 *out)
{
    using S = SsRowShape<N>;
    constexpr int P = S::P, T = S::T, G = S::G, W = LdsPlane<double>::elems(N);
    constexpr int NC = N / 2 + 1;
    constexpr int RPG = (SO & 1) ? 1 : 2;
    __shared__ __attribute__((aligned(16))) double2 lds[W * G];
    __shared__ __attribute__((aligned(16))) double wq[FQuad<double>::TABLE];
    __shared__ double2 qres[(SO & 1) ? NC * G : 1];  // SO: the group's integrated samples
    __shared__ int qmax_wg;                         // SO: last integrated sample of any group
    const int g = threadIdx.x / T, t = threadIdx.x % T;
    const LdsPlane<double> pl{lds + W * g};
    const int row = (blockIdx.x * G + g) * RPG;  // the group's first row
    // per row of the group: ring pair (padding and missing rows take the first
    // ring and stay zero), radii, aspect ratios and X
    bool live_[RPG];
    int ic_[RPG], ip_[RPG], a = 0, b = 0;
    bool any = false;
#pragma unroll
    for (int u = 0; u < RPG; ++u) {
        int ur = row + u, ua, ub;
        const bool in = ur < nrows;
        live_[u] = ss_row(A, C, (uint32_t)r0 + (in ? ur : 0), ub, ua, ip_[u], ic_[u]) && in && ic_[u] < A.nr;
        if (live_[u]) {
            a = ua;  // one pair per group: units and plain rows pair up within it
            b = ub;
        } else {
            ic_[u] = ip_[u] = 0;
        }
        any = any || live_[u];
    }
    const bool valid = row < nrows;
    if (!__syncthreads_or(any || (valid && !C.on) ? 1 : 0)) return;
    sg_fill64(wq, A.pot ? SG_FN_G0 : SG_FN_F);
    double ri_[RPG], rp_[RPG], ha_[RPG], hb_[RPG], X_[RPG];
#pragma unroll
    for (int u = 0; u < RPG; ++u) {
        ri_[u] = A.lin ? A.rmin + (ic_[u] + 0.5) * A.dr : exp(A.lnrmin + (ic_[u] + 0.5) * A.du);
        rp_[u] = A.lin ? A.rmin + (ip_[u] + 0.5) * A.dr : exp(A.lnrmin + (ip_[u] + 0.5) * A.du);
        ha_[u] = H[a * A.nr + ip_[u]] / rp_[u];
        hb_[u] = H[b * A.nr + ic_[u]] / ri_[u];
        X_[u] = A.lin ? log(ri_[u] / rp_[u]) : (double)(ic_[u] - ip_[u]) * A.du;
    }
    const bool live = live_[0];
    const int ic = ic_[0], ip = ip_[0];
    const double ha = ha_[0], hb = hb_[0], X = X_[0];
    __syncthreads();
    if constexpr ((SO & 1) != 0) {
        // 1'. hat-weighted samples (see SG_SS_HAT_NEAR): point values of K go
        // to the plane for the neighbours' second differences, the weights
        // stay in registers until every neighbour has been read
        constexpr int J = (N / 2 + 1 + T - 1) / T;
        double2 val[J];
        unsigned taylor = 0u;
        const int Pr = ic - ip;
        const double rn = SG_SS_HAT_NEAR * fmax(A.du, A.dphi), xq = Pr * A.du;
        // integrated samples: q <= qn (qn = -1: none); the predicate below is
        // the one the sample loop uses
        int qn = -1;
        if (live && xq * xq < rn * rn)
            while (qn < N / 2 && xq * xq + ((qn + 1) * A.dphi) * ((qn + 1) * A.dphi) < rn * rn) ++qn;
        if (threadIdx.x == 0) qmax_wg = -1;
        __syncthreads();
        if (t == 0 && qn >= 0) atomicMax(&qmax_wg, qn);
        __syncthreads();
        const int qm = qmax_wg;  // uniform over the workgroup: every group meets the same barriers
        for (int q = 0; q <= qm; ++q) {
            double wr = 0.0, wp = 0.0;
            if (q <= qn) sg_hat_weight_part<SO == 3>(Pr, q, A.du, A.dphi, ha, hb, 0, A.gl, wq, t, T, wr, wp);
            pl.st(t, make_double2(wr, wp));
            __syncthreads();
            if (q <= qn && t == 0) {
                double sr = 0.0, sp = 0.0;
                for (int k = 0; k < T; ++k) {
                    const double2 v = pl.ld(k);
                    sr += v.x;
                    sp += v.y;
                }
                qres[g * NC + q] = make_double2(sr, sp);
            }
            __syncthreads();
        }
        // the row-only factors at X and at the D_X neighbours X +- du
        const ConvRow64 c0 = sg_conv_row64(X, ha, hb), c1 = sg_conv_row64(X + A.du, ha, hb),
                        c2 = sg_conv_row64(X - A.du, ha, hb);
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int q = t + T * j;
            val[j] = make_double2(0.0, 0.0);
            if (q > N / 2) continue;
            double sh, ch;
            ss_half_angle<N>(q, sh, ch);
            const double s2 = 2.0 * sh * ch;
            double kr = 0.0, kp = 0.0;
            if (q <= qn) {
                val[j] = qres[g * NC + q];
                if (Pr != 0 || q != 0) sg_conv_kernel64_row(c0, sh, s2, wq, kr, kp);
            } else {
                double k1r, k1p, k2r, k2p;
                sg_conv_kernel64_row(c0, sh, s2, wq, kr, kp);
                sg_conv_kernel64_row(c1, sh, s2, wq, k1r, k1p);
                sg_conv_kernel64_row(c2, sh, s2, wq, k2r, k2p);
                val[j] = make_double2(kr + (k1r - 2.0 * kr + k2r) / 12.0, kp + (k1p - 2.0 * kp + k2p) / 12.0);
                taylor |= 1u << j;
            }
            pl.st(q, make_double2(kr, kp));
            if (q != 0 && q != N / 2) pl.st(N - q, make_double2(kr, -kp));
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int q = t + T * j;
            if (q > N / 2 || !((taylor >> j) & 1u)) continue;
            const double2 k0 = pl.ld(q), kl = pl.ld((q + N - 1) & (N - 1)), kh = pl.ld((q + 1) & (N - 1));
            val[j].x += (kl.x - 2.0 * k0.x + kh.x) / 12.0;
            val[j].y += (kl.y - 2.0 * k0.y + kh.y) / 12.0;
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int q = t + T * j;
            if (q > N / 2) continue;
            pl.st(q, val[j]);
            if (q != 0 && q != N / 2) pl.st(N - q, make_double2(val[j].x, -val[j].y));
        }
    } else {
    // 1. samples q in [0, N/2] of both rows, packed as z_A + i z_B and
    // mirrored into the upper half (z(-q) = conj z(q) for each row); the
    // factors that depend on a row alone are formed once
    ConvRow64 cr[RPG], cp1[SO == 2 ? RPG : 1], cp2[SO == 2 ? RPG : 1];
    double sx[RPG], Hab2[RPG], pot_pref[RPG];
#pragma unroll
    for (int u = 0; u < RPG; ++u) {
        cr[u] = sg_conv_row64(X_[u], ha_[u], hb_[u]);
        if constexpr (SO == 2) {
            cp1[u] = sg_conv_row64(X_[u] + A.du, ha_[u], hb_[u]);
            cp2[u] = sg_conv_row64(X_[u] - A.du, ha_[u], hb_[u]);
        }
        const double Ha = ha_[u] * rp_[u], Hb = hb_[u] * ri_[u];
        sx[u] = sinh(0.5 * X_[u]);
        Hab2[u] = 0.5 * (Ha * Ha + Hb * Hb);
        pot_pref[u] = rp_[u] * rp_[u] / (2.0 * SG_SQRT_PI * sqrt(Hab2[u]));
    }
#pragma unroll 1
    for (int q = t; q <= N / 2; q += T) {
        double sp, cp;
        ss_half_angle<N>(q, sp, cp);
        double kr[RPG], kp[RPG];
#pragma unroll
        for (int u = 0; u < RPG; ++u) {
            kr[u] = 0.0;
            kp[u] = 0.0;
            if (!live_[u]) continue;  // shares its transform with the other row
            if constexpr (SO == 2) {
                ss_far_weight(cr[u], cp1[u], cp2[u], 2.0 * q / N, A.dphi / SG_PI, wq, kr[u], kp[u]);
                continue;
            }
            if (ic_[u] == ip_[u] && q == 0) {
                kr[u] = A.excl ? 0.0 : self[(size_t)(a * A.nf + b) * A.nr + ic_[u]];
            } else if (A.pot) {
                // -r'^2 P_ab(s), so that the common scale -du dphi / N gives A_i' P / N
                const double s2 = 4.0 * ri_[u] * rp_[u] * (sx[u] * sx[u] + sp * sp);
                kr[u] = pot_pref[u] * sg_G0_64(s2 / (8.0 * Hab2[u]), wq);
            } else {
                sg_conv_kernel64_row(cr[u], sp, 2.0 * sp * cp, wq, kr[u], kp[u]);
            }
        }
        // (kr0 + i kp0) + i (kr1 + i kp1), and at -q (kr0 - i kp0) + i (kr1 - i kp1)
        pl.st(q, make_double2(kr[0] - kp[1], kp[0] + kr[1]));
        if (q != 0 && q != N / 2) pl.st(N - q, make_double2(kr[0] + kp[1], kr[1] - kp[0]));
    }
    }
    __syncthreads();
    double2 z[P];
#pragma unroll
    for (int p = 0; p < P; ++p) z[p] = pl.ld(t + T * p);
    __syncthreads();
    // 2. transform; Z = T_r - t_phi at m and T_r + t_phi at -m
    fft<N, false>(z, t, pl, TwPow64<N>{t});
#pragma unroll
    for (int p = 0; p < P; ++p) pl.st(t + T * p, z[p]);
    __syncthreads();
    if (!valid) return;
#pragma unroll
    for (int u = 0; u < RPG; ++u) {
        // the samples carry r'^2 (the log-grid measure per du dphi); the source
        // cell's measure is r'^2 wgt dphi with wgt = du, or dr / r' on a uniform grid
        const double rp = rp_[u], scale = -(A.lin ? A.dr / rp : A.du) * A.dphi / N;
        double ind = 0.0;
        if (A.ind) {
            // r'^2 sqrt(2) K_a(d) N / 2 (the convolution-form samples carry the
            // cell measure r'^2), K_a(d) = pi^{-1/2} H^{-2} (d/4) F(d^2/4)
            const double Ha = ha_[u] * rp, d = rp / Ha;
            ind = rp * rp * SG_SQRT2 * (1.0 / SG_SQRT_PI) / (Ha * Ha) * (0.25 * d) * sg_F64(0.25 * d * d, wq) *
                  (0.5 * N);
        }
        float2 *o = out + (size_t)(row + u) * mc;
        for (int m = t; m < mc; m += T) {
            float2 v = make_float2(0.f, 0.f);
            if (live_[u]) {
                const double2 wm = pl.ld(m), wn = pl.ld((N - m) & (N - 1));
                const double zm = u == 0 ? wm.x : wm.y, zn = u == 0 ? wn.x : wn.y;
                double tr = 0.5 * (zm + zn), tp = A.pot ? 0.0 : 0.5 * (zn - zm);
                if (m == 1) {
                    tr += ind;
                    tp += ind;
                }
                v = make_float2((float)(scale * tr), (float)(scale * tp));
            }
            gstore2(o, m, v);
        }
    }
}

// Point-sampled rows of a class on the log grid, a ring pair at a time: a row
// (b, a, i', i) and its mirror (a, b, i, i') are one even function of phi,
// S = F(x(phi)) (G0 for the potential), times
//   K_r = p (e^X - cos phi) = p ((e^X - 1) + (1 - cos phi)),  K_phi = p sin phi
// with p and X of the row, and the products with 1 - cos phi and sin phi are
// differences of neighbouring modes of S~ (exact for the sampled sequence).
// So a pair takes one evaluation per azimuth of half the circle and half a
// transform, where its rows took two and one; the table's entries are formed
// from S~, held in double, by k_ss_scatter_pairs.  The differences cost
// 1e-16/|X| of a row's largest coefficient (1e-16/dphi^2 for i' = i, whose
// own-cell sample enters as a constant of all modes), as an absolute error of
// all its entries: the smallest that are kept, 2^-30 of the largest, hold
// 1e-7/|X| of themselves where the transform alone would leave 1e-7.  The table
// holds floats, and a ring's sum is led by its near pairs' entries.
// C: offsets k >= 0 only.  out: [nrows][ld] double S~, m < ld <= N/2 + 1.
// 1200 x 2048 one fluid, all rows 2.74 -> 1.14 ms, whole build and solve 3.84
// -> 2.40 ms.
template <int N>
__global__ void __launch_bounds__(SsRowShape<N>::WGS)
k_ss_pairs(const double *H, SsRowArgs A, SsClass C, size_t r0, int nrows, int ld, double *out)
{
    using S = SsRowShape<N>;
    constexpr int P = S::P, T = S::T, G = S::G, W = LdsPlane<double>::elems(N);
    __shared__ __attribute__((aligned(16))) double2 lds[W * G];
    __shared__ __attribute__((aligned(16))) double wq[FQuad<double>::TABLE];
    const int g = threadIdx.x / T, t = threadIdx.x % T;
    const LdsPlane<double> pl{lds + W * g};
    const int row = (blockIdx.x * G + g) * 2;
    int ic[2], ip[2], a = 0, b = 0;
    bool live[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        int ua, ub;
        live[u] = ss_row(A, C, (uint32_t)r0 + (row + u < nrows ? row + u : 0), ub, ua, ip[u], ic[u]) && row + u < nrows;
        if (live[u]) {
            a = ua;  // a unit's rows are of one fluid pair
            b = ub;
        } else {
            ic[u] = ip[u] = 0;
        }
    }
    if (!__syncthreads_or(live[0] || live[1] ? 1 : 0)) return;
    sg_fill64(wq, A.pot ? SG_FN_G0 : SG_FN_F);
    // x(phi) = xa (x0 + 2 sin^2(phi / 2)), also the potential's s^2 / (8 H_ab^2)
    double x0[2], xa[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const double ri = exp(A.lnrmin + (ic[u] + 0.5) * A.du), rp = exp(A.lnrmin + (ip[u] + 0.5) * A.du);
        const ConvRow64 c = sg_conv_row64((double)(ic[u] - ip[u]) * A.du, H[a * A.nr + ip[u]] / rp,
                                          H[b * A.nr + ic[u]] / ri);
        x0[u] = c.two_sxh2;
        xa[u] = c.inv4h2;
    }
    __syncthreads();
#pragma unroll 1
    for (int q = t; q <= N / 2; q += T) {
        double sh, ch, v[2];
        ss_half_angle<N>(q, sh, ch);
        const double two_s2 = 2.0 * sh * sh;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            v[u] = 0.0;
            if (!live[u] || (ic[u] == ip[u] && q == 0)) continue;
            const double x = (x0[u] + two_s2) * xa[u];
            v[u] = A.pot ? sg_G0_64(x, wq) : sg_F64(x, wq);
        }
        const double2 z = make_double2(v[0], v[1]);
        pl.st(q, z);
        if (q != 0 && q != N / 2) pl.st(N - q, z);
    }
    __syncthreads();
    double2 z[P];
#pragma unroll
    for (int p = 0; p < P; ++p) z[p] = pl.ld(t + T * p);
    __syncthreads();
    fft<N, false>(z, t, pl, TwPow64<N>{t});
    if (row >= nrows) return;
    double *o = out + (size_t)row * ld;
#pragma unroll
    for (int p = 0; p <= P / 2; ++p) {
        const int m = t + T * p;
        if (m >= ld) break;
        o[m] = z[p].x;
        o[ld + m] = z[p].y;
    }
}

// ------------------------------------------------------- table: transpose
// src [nrows][ld] (rows r0 + row of a class or of the plain order) into the layouts of modes m0 <= m < ncol, in 32 x 32 tiles of
// rows and modes.  The 32 rows of a block are written as runs of consecutive
// target rings, so they are taken in the order of the modes' layout: in row
// order (a class's diagonals for the banded modes; the plain order, whose i'
// rows are the full modes'), or, for the full modes of a class (FULL), as two
// source rings i' times the 16 target rings of a tile, gathered from the rows
// of their offsets (each row is read as 256 contiguous bytes either way).
// Diagonals written across the order, 8 bytes at a time, took 1.9 of the 5.2
// ms of the 1200 x 2048 build.  A row's place costs several integer divisions,
// so a block goes through all its modes (blockIdx.y: every gridDim.y-th tile).
template <bool FULL>
__global__ void __launch_bounds__(256)
k_ss_scatter(const float2 *src, int ld, int nrows, int ncol, int m0, float2 *coef, const SsMode *modes,
             SsRowArgs A, SsClass C, size_t r0, int tile0)
{
    __shared__ float2 tile[32][33];
    __shared__ int srow[32];
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    int i, ip, a, b, row;
    bool ok;
    if constexpr (FULL) {
        // unit (pair, t, v): source ring number v of those that tile t meets in the class
        const int side = C.K1 == 0 ? 2 * C.K2 - 1 + (SG_SS_TI - 1) : C.K2 - C.K1 + (SG_SS_TI - 1);
        const int per = C.K1 == 0 ? side : 2 * side;
        const int half = (per + 1) / 2;  // blocks per tile
        const int pt = tile0 + (int)(blockIdx.x / half), v = 2 * (int)(blockIdx.x % half) + (tx >> 4);
        const int t = pt % C.nt, pair = pt / C.nt;
        a = pair % A.nf;
        b = pair / A.nf;
        i = t * SG_SS_TI + (tx & 15);
        if (C.K1 == 0) ip = t * SG_SS_TI - (C.K2 - 1) + v;
        else ip = v < side ? t * SG_SS_TI + C.K1 + v : t * SG_SS_TI + (SG_SS_TI - 1) - C.K1 - (v - side);
        const int k = ip - i;
        ok = b < A.nf && v < per && i < A.nr && ip >= 0 && ip < A.nr && ss_in_class(A, C, t, k);
        // a ring may come up on both sides; only its own side's offsets count
        if (C.K1 != 0) ok = ok && (v < side ? k > 0 : k < 0);
        const int q = C.K1 == 0 ? k + C.K2 - 1 : k > 0 ? k - C.K1 : (C.K2 - C.K1) - k - C.K1;
        const int64_t rr = (((int64_t)pt * C.nk + q) * SG_SS_TI + (tx & 15)) - (int64_t)r0;
        ok = ok && rr >= 0 && rr < nrows;
        row = ok ? (int)rr : 0;
    } else {
        row = blockIdx.x * 32 + tx;
        ok = ss_row(A, C, (uint32_t)r0 + (row < nrows ? row : 0), b, a, ip, i) && row < nrows;
        row = ok ? row : 0;
    }
    if (!__syncthreads_or(ok ? 1 : 0)) return;
    if (ty == 0) srow[tx] = row;
    const uint32_t pair = b * A.nf + a;
    for (int mb = m0 + blockIdx.y * 32; mb < ncol; mb += gridDim.y * 32) {
        __syncthreads();  // srow; the previous tile has been read
        const int m = mb + tx;
        float2 v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = gload2(src, (size_t)srow[ty + 8 * k] * ld + (m < ncol ? m : 0));
#pragma unroll
        for (int k = 0; k < 4; ++k) tile[ty + 8 * k][tx] = v[k];
        __syncthreads();
        if (!ok) continue;
        for (int k = ty; k < 32 && mb + k < ncol; k += 8) {
            const SsMode md = modes[mb + k];
            size_t dst;
            if (md.banded) {
                const int d = ip - i + md.w;
                if (d < 0 || d > 2 * md.w) continue;
                dst = md.off + (size_t)(pair * (2 * md.w + 1) + d) * A.nrt + i;
            } else {
                dst = md.off + (size_t)(pair * A.nr + ip) * A.nrt + i;
            }
            gstore2(coef, dst, tile[tx][k]);
        }
    }
}

// The entries of a class's ring pairs from their S~ (k_ss_pairs; src
// [nrows][ld], modes m0 <= m < m1 of rows of N samples), both rows of a pair.
// The banded modes (!FULL) go by 32 consecutive rows, whose targets, i and
// i + k, are runs of two diagonals.  The full modes go by a source ring times
// 16 target rings of a tile, gathered from the rows of their offsets: rows
// i' >= i by (tile of i, i'), their mirrors by (source i, tile of i').  Every
// block forms its rows' factors once and goes through all its modes, 32 and
// one neighbour on each side at a time.
template <bool FULL>
__global__ void __launch_bounds__(256)
k_ss_scatter_pairs(const double *src, int ld, int nrows, int N, int m0, int m1, float2 *coef, const SsMode *modes,
                   const double *H, const double *self, SsRowArgs A, SsClass C, size_t r0, int tile0)
{
    __shared__ double tile[32][35];
    __shared__ double fc[2][32], fp[2][32], fown[2][32], find[2][32];
    __shared__ int srow[32];
    __shared__ __attribute__((aligned(16))) double wq[FQuad<double>::TABLE];
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    int i, ip, a, b, row, edir = 0;
    bool ok;
    if constexpr (FULL) {
        const int n0 = C.nk + SG_SS_TI - 1;                                      // source rings of a tile's rows
        const int n1 = SG_SS_TI * ((C.nk + 2 * SG_SS_TI - 2) / SG_SS_TI);        // (source, tile) of their mirrors
        const int h0 = (n0 + 1) / 2, half = h0 + n1 / 2;                         // blocks per tile
        const int pt = tile0 + (int)(blockIdx.x / half), e = (int)(blockIdx.x % half), l = tx & 15;
        const int t = pt % C.nt, pair = pt / C.nt;
        a = pair % A.nf;
        b = pair / A.nf;
        edir = e >= h0 ? 1 : 0;
        const int v = 2 * (edir ? e - h0 : e) + (tx >> 4);
        if (!edir) {
            i = t * SG_SS_TI + l;
            ip = t * SG_SS_TI + C.K1 + v;
            ok = v < n0;
        } else {
            i = t * SG_SS_TI + (v & 15);
            ip = (((i + C.K1) & ~15) + 16 * (v >> 4)) + l;
            ok = v < n1;
        }
        const int k = ip - i;
        ok = ok && b < A.nf && i < A.nr && ip < A.nr && k >= C.K1 && k < C.K2 && !(edir && k == 0);
        const int64_t rr = (((int64_t)pt * C.nk + (k - C.K1)) * SG_SS_TI + (i & 15)) - (int64_t)r0;
        ok = ok && rr >= 0 && rr < nrows;
        row = ok ? (int)rr : 0;
    } else {
        row = blockIdx.x * 32 + tx;
        ok = ss_row(A, C, (uint32_t)r0 + (row < nrows ? row : 0), b, a, ip, i) && row < nrows;
        row = ok ? row : 0;
    }
    if (!__syncthreads_or(ok ? 1 : 0)) return;
    const bool ind = A.ind && m0 + (int)blockIdx.y * 32 <= 1;  // the block forms mode 1
    if (ind) {
        sg_fill64(wq, SG_FN_F);
        __syncthreads();
    }
    if (ty == 0) srow[tx] = row;
    if (ty < (FULL ? 1 : 2)) {
        const int dir = FULL ? edir : ty;
        const int ii = ok ? i : 0, jj = ok ? ip : 0, fa = ok ? a : 0, fb = ok ? b : 0;
        const int ti = dir ? jj : ii, si = dir ? ii : jj, tf = dir ? fa : fb, sf = dir ? fb : fa;  // target, source
        const double rt = exp(A.lnrmin + (ti + 0.5) * A.du), rs = exp(A.lnrmin + (si + 0.5) * A.du);
        const double Ht = H[tf * A.nr + ti], Hs = H[sf * A.nr + si];
        const double scale = -A.du * A.dphi / N;  // the source cell's measure r'^2 du dphi is in p
        const ConvRow64 c = sg_conv_row64((double)(ti - si) * A.du, Hs / rs, Ht / rt);
        fc[dir && !FULL][tx] = A.pot ? 1.0 : c.em1;
        fp[dir && !FULL][tx] =
            scale * (A.pot ? rs * rs / (2.0 * SG_SQRT_PI * sqrt(0.5 * (Hs * Hs + Ht * Ht))) : c.pref);
        fown[dir && !FULL][tx] = ti == si && !A.excl ? scale * self[(size_t)(sf * A.nf + tf) * A.nr + ti] : 0.0;
        double w = 0.0;
        if (ind) {
            // r'^2 sqrt(2) K_a(d) N / 2, K_a(d) = pi^{-1/2} H^{-2} (d/4) F(d^2/4)
            const double d = rs / Hs;
            w = scale * rs * rs * SG_SQRT2 * (1.0 / SG_SQRT_PI) / (Hs * Hs) * (0.25 * d) * sg_F64(0.25 * d * d, wq) *
                (0.5 * N);
        }
        find[dir && !FULL][tx] = w;
    }
    const double b1 = A.pot ? 0.0 : 1.0;
    const int k = ip - i;
    for (int mb = m0 + blockIdx.y * 32; mb < m1; mb += gridDim.y * 32) {
        __syncthreads();  // the rows' factors; the previous tile has been read
        for (int e = threadIdx.x; e < 32 * 34; e += 256) {
            const int r = e / 34, c = e - 34 * r;
            int m = abs(mb - 1 + c);           // S~(-1) = S~(1)
            m = m > N / 2 ? N - m : m;         // and S~(N/2 + 1) = S~(N/2 - 1)
            tile[r][c] = src[(size_t)srow[r] * ld + min(m, ld - 1)];
        }
        __syncthreads();
        if (!ok) continue;
        for (int q = ty; q < 32 && mb + q < m1; q += 8) {
            const int m = mb + q;
            const SsMode md = modes[m];
            if (md.banded && k > md.w) continue;
            const double sl = tile[tx][q], s0 = tile[tx][q + 1], sh = tile[tx][q + 2];
            const double B = b1 * (s0 - 0.5 * (sl + sh)), Cp = b1 * 0.5 * (sh - sl);
#pragma unroll
            for (int u = 0; u < (FULL ? 1 : 2); ++u) {
                const int dir = FULL ? edir : u;
                if (dir && k == 0) continue;
                const double add = m == 1 ? find[u][tx] : 0.0;
                const double tr = fp[u][tx] * (fc[u][tx] * s0 + B) + fown[u][tx] + add, tp = fp[u][tx] * Cp + add;
                const uint32_t pair = dir ? a * A.nf + b : b * A.nf + a;
                const int ti = dir ? ip : i, si = dir ? i : ip;
                const size_t dst = md.banded
                                       ? md.off + (size_t)(pair * (2 * md.w + 1) + (si - ti + md.w)) * A.nrt + ti
                                       : md.off + (size_t)(pair * A.nr + si) * A.nrt + ti;
                gstore2(coef, dst, make_float2((float)tr, A.pot ? 0.f : (float)tp));
            }
        }
    }
}

// Mode descriptors (one block; the same band rule as the host layout, with
// the host's du): thread t takes ncol/256 consecutive modes, the offsets come
// from a prefix sum over the threads (a single thread took 66 to 125 us for
// 513 to 1025 modes).
__global__ void __launch_bounds__(256) k_ss_modes(SsMode *modes, int ncol, int nr, int nrt, int nf, double du, int full)
{
    __shared__ uint64_t sum[256];
    const int per = (ncol + 255) / 256, m0 = threadIdx.x * per, m1 = min(ncol, m0 + per);
    auto rows = [&](int m, int &w) {
        w = sg_ss_band(m, nr, du, full != 0);
        return sg_ss_is_banded(w, nr) ? 2 * w + 1 : nr;
    };
    uint64_t mine = 0;
    int w;
    for (int m = m0; m < m1; ++m) mine += (uint64_t)rows(m, w);
    sum[threadIdx.x] = mine;
    __syncthreads();
    for (int o = 1; o < 256; o <<= 1) {
        const uint64_t v = (int)threadIdx.x >= o ? sum[threadIdx.x - o] : 0;
        __syncthreads();
        sum[threadIdx.x] += v;
        __syncthreads();
    }
    uint64_t off = sum[threadIdx.x] - mine;
    for (int m = m0; m < m1; ++m) {
        const int n = rows(m, w);
        SsMode md;
        md.off = off * ((uint64_t)nf * nf * nrt);
        md.w = w;
        md.banded = sg_ss_is_banded(w, nr) ? 1 : 0;
        modes[m] = md;
        off += (uint64_t)n;
    }
}

// Own-cell terms on a uniform radial grid, one item per (pair, ring): the
// cell spans X = ln(r'/r) in [ln(1 - dr/(2r)), ln(1 + dr/(2r))], no longer
// symmetric, so each side of X = 0 is integrated on its own (the integrand
// is integrable: ~1/rho for the field, logarithmic for the potential) with
// the Duffy triangles and geometric panels of the log-cell quadrature, and
// doubled for phi < 0 (both kernels are even in phi).  Output: the table
// sample I / (wgt dphi) (field, I = int K_r dX dphi) or -I / (wgt dphi)
// (potential, I = int P dA'), wgt = dr / r; which = 1, 2: their derivatives
// with respect to h_a, h_b instead.  per: cells per ring of H
// and out (1: one value per ring; n_phi: per cell, for the direct sum with
// per-cell H), item = pair * n_r * per + cell.
__global__ void __launch_bounds__(256)
k_ss_self_lin(const double *H, int nf, int nr, int per, double rmin, double dr, double dphi, int pot, int which,
              double *out, GLNodes gl)
{
    __shared__ __attribute__((aligned(16))) double wq[FQuad<double>::TABLE];
    __shared__ double red[256];
    sg_fill64(wq, pot ? (which ? SG_FN_E : SG_FN_G0) : (which ? SG_FN_D : SG_FN_F));
    __syncthreads();
    const int64_t cells = (int64_t)nr * per;
    const int64_t item = blockIdx.x;
    if (item >= nf * nf * cells) return;
    const int pair = (int)(item / cells), fa = pair / nf, fb = pair % nf;
    const int64_t c = item % cells;
    const int ir = (int)(c / per);
    const double r = rmin + (ir + 0.5) * dr;
    const double Ha = H[fa * cells + c], Hb = H[fb * cells + c];
    const double ha = Ha / r, hb = Hb / r, Hab = sqrt(0.5 * (Ha * Ha + Hb * Hb));
    const double b = 0.5 * dphi;
    double acc = 0.0;
    for (int sd = 0; sd < 2; ++sd) {
        const double sgn = sd == 0 ? 1.0 : -1.0;
        const double a = sd == 0 ? log1p(0.5 * dr / r) : -log1p(-0.5 * dr / r);
        const int nx = sg_own_nx(a, b, fmin(ha, hb)), n = nx * gl.ne;
        const OwnEta e0(a, b), e1(b, a);
        for (int idx = threadIdx.x; idx < n; idx += blockDim.x) {
            double xi, s, wn;
            sg_own_node(gl, nx, idx, xi, s, wn);
            wn *= a * b;
            for (int tri = 0; tri < 2; ++tri) {
                double wgt = wn, f;
                const double eta = (tri == 0 ? e0 : e1).at(s, wgt);
                const double X = sgn * (tri == 0 ? a * xi : a * xi * eta);
                const double phi = tri == 0 ? b * xi * eta : b * xi;
                if (pot) {
                    const double sx = sinh(0.5 * X), sp = sin(0.5 * phi);
                    const double s2 = r * r * exp(X) * 4.0 * (sx * sx + sp * sp);
                    const double y = s2 / (8.0 * Hab * Hab);
                    if (which == 0) {
                        f = -sg_G0_64(y, wq) / (2.0 * SG_SQRT_PI * Hab) * r * r * exp(2.0 * X);
                    } else {
                        // dP/dH_ab = -(2 y F(y) - G0(y)) / (2 sqrt(pi) H_ab^2), times dH_ab/dh
                        const double ch = (which == 1 ? Ha : Hb) * r / (2.0 * Hab);
                        f = -sg_E64(y, wq) / (2.0 * SG_SQRT_PI * Hab * Hab) * ch * r * r * exp(2.0 * X);
                    }
                } else {
                    double kr, kp;
                    sg_conv_kernel64(X, sin(0.5 * phi), sin(phi), ha, hb, which, wq, kr, kp);
                    f = kr;
                }
                acc += wgt * f;
            }
        }
    }
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const double I = 2.0 * red[0], w = (dr / r) * dphi;
        out[item] = pot ? -I / w : I / w;
    }
}

__global__ void k_ss_scale(double *p, int n, double f)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] *= f;
}

__global__ void k_ss_zero(float2 *p, size_t n)
{
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        gstore2(p, i, make_float2(0.f, 0.f));
}

__global__ void k_ss_header(sg_ss_header *hd, sg_ss_header proto)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) *hd = proto;
}

// ------------------------------------------------------------- table: host
#define SG_SS_CHUNK_BYTES ((size_t)128 << 20)
#define SG_SS_MAX_NR 2048

int sg_ss_max_nr() { return SG_SS_MAX_NR; }

static size_t ss_chunk_rows(const SsLayout &L)
{
    const size_t per = sizeof(float2) * (size_t)L.ncol;
    size_t rows = SG_SS_CHUNK_BYTES / per;
    rows = rows / 32 * 32;
    if (rows < 32) rows = 32;
    return rows < L.rows ? rows : L.rows;
}

size_t sg_ss_ws_bytes(int nr, int nphi, int nf)
{
    const SsLayout L = sg_ss_layout(nr, nphi, nf, 1.0, true);
    return sg_align256(sizeof(double) * (size_t)nf * nf * nr) +
           sg_align256(sizeof(float2) * L.ncol * ss_chunk_rows(L));
}

// The row classes of a build: one launch set each (kind: SO of k_ss_rows).
struct SsPart {
    int M, kind;
    SsClass C;
};

// full: no band limit.  alias: SG_SS_ALIAS or SG_SS_ALIAS_GRAD.
static std::vector<SsPart> ss_parts(const SsRowArgs &A, int nphi, bool full, double alias)
{
    std::vector<SsPart> out;
    SsClass C{};
    const bool split = A.nr >= 2 * SG_SS_TI && (A.second || (!full && nphi > SG_SS_MIN_M));
    if (!split) {
        out.push_back({nphi, A.second ? 1 : 0, C});
        return out;
    }
    const double inf = INFINITY, rn = A.second ? SG_SS_HAT_NEAR * fmax(A.du, A.dphi) : 0.0;
    C.on = 1;
    C.nt = (A.nr + SG_SS_TI - 1) / SG_SS_TI;
    auto add = [&](int M, int kind, double x1, double x2) {
        if (x1 >= x2) return;
        C.x1 = x1;
        C.x2 = x2;
        C.K1 = x1 == 0.0 ? 0 : A.nr;
        C.K2 = 0;
        if (!A.lin) {
            if (x1 > 0.0) C.K1 = (int)fmin(ceil(x1 / A.du), (double)A.nr);
            C.K2 = (int)fmin(ceil(fmin(x2 / A.du, 1e9)), (double)A.nr);
        } else {
            // offsets of which some tile falls into the class: the distance falls
            // with the tile, from the first to the last that has a ring pair
            C.K2 = x1 == 0.0 ? 1 : 0;
            for (int k = 1; k < A.nr; ++k) {
                const int last = (A.nr - 1 - k) / SG_SS_TI;
                const double hi = fmax(ss_tile_dist(A.rmin, A.dr, 0, k), ss_tile_dist(A.rmin, A.dr, k / SG_SS_TI, -k));
                const double lo = fmin(ss_tile_dist(A.rmin, A.dr, last, k),
                                       ss_tile_dist(A.rmin, A.dr, (A.nr - 1) / SG_SS_TI, -k));
                if (hi < x1 || lo >= x2) continue;
                if (k < C.K1 && x1 > 0.0) C.K1 = k;
                C.K2 = k + 1;
            }
        }
        if (C.K1 >= C.K2) return;
        C.nk = C.K1 == 0 ? 2 * C.K2 - 1 : 2 * (C.K2 - C.K1);
        out.push_back({M, kind, C});
    };
    if (A.second) add(nphi, 1, 0.0, rn);
    for (int M = nphi;; M /= 2) {
        const bool last = full || M / 2 < SG_SS_MIN_M;
        const double x1 = M == nphi ? 0.0 : alias / M, x2 = last ? inf : alias / (M / 2);
        add(M, A.second ? 2 : 0, fmax(x1, rn), fmax(x2, rn));
        if (last) break;
    }
    return out;
}

static size_t ss_class_rows(const SsRowArgs &A, const SsClass &C)
{
    return (size_t)A.nf * A.nf * C.nt * C.nk * SG_SS_TI;
}

template <int N>
static void launch_ss_rows(const double *H, const double *self, const SsRowArgs &A, const SsPart &P, size_t r0,
                           int nrows, int mc, float2 *out, hipStream_t s)
{
    using S = SsRowShape<N>;
    // the quadrature's registers stay out of the other rows; two rows per
    // group unless integrated (nrows is even: see k_ss_rows)
    const dim3 one((nrows + S::G - 1) / S::G), two((nrows + 2 * S::G - 1) / (2 * S::G));
    if (P.kind == 1 && sg_hat_long(A.du, A.dphi))
        hipLaunchKernelGGL((k_ss_rows<N, 3>), one, dim3(S::WGS), 0, s, H, self, A, P.C, r0, nrows, mc, out);
    else if (P.kind == 1)
        hipLaunchKernelGGL((k_ss_rows<N, 1>), one, dim3(S::WGS), 0, s, H, self, A, P.C, r0, nrows, mc, out);
    else if (P.kind == 2)
        hipLaunchKernelGGL((k_ss_rows<N, 2>), two, dim3(S::WGS), 0, s, H, self, A, P.C, r0, nrows, mc, out);
    else
        hipLaunchKernelGGL((k_ss_rows<N, 0>), two, dim3(S::WGS), 0, s, H, self, A, P.C, r0, nrows, mc, out);
}

static bool dispatch_ss_rows(const double *H, const double *self, const SsRowArgs &A, const SsPart &P, size_t r0,
                             int nrows, int mc, float2 *out, hipStream_t s)
{
#define SG_ROWS(N) \
    case N: launch_ss_rows<N>(H, self, A, P, r0, nrows, mc, out, s); return true;
    switch (P.M) {
        SG_ROWS(4) SG_ROWS(8) SG_ROWS(16) SG_ROWS(32) SG_ROWS(64) SG_ROWS(128) SG_ROWS(256) SG_ROWS(512)
        SG_ROWS(1024) SG_ROWS(2048)
    }
#undef SG_ROWS
    return false;
}

// S~ of a class's ring pairs and their entries, a chunk buffer at a time.
static bool build_pairs(const double *H, const double *self, const SsRowArgs &A, const SsPart &P, int mc, int mfull,
                        void *chunk, size_t cbytes, float2 *coef, const SsMode *modes, hipStream_t s)
{
    SsClass C = P.C;
    C.half = 1;
    C.nk = C.K2 - C.K1;
    const int N = P.M, ld = std::min(mc + 1, N / 2 + 1);  // one mode more, for the last one's difference
    const size_t rows = ss_class_rows(A, C);
    size_t crows = cbytes / (sizeof(double) * ld) / SG_SS_TI * SG_SS_TI;
    if (crows > (size_t)1 << 30) crows = (size_t)1 << 30;
    double *out = (double *)chunk;
    for (size_t r0 = 0; r0 < rows; r0 += crows) {
        const int n = (int)std::min(crows, rows - r0);
        switch (N) {
#define SG_PAIRS(M)                                                                                              \
    case M:                                                                                                      \
        hipLaunchKernelGGL(k_ss_pairs<M>, dim3((n / 2 + SsRowShape<M>::G - 1) / SsRowShape<M>::G),               \
                           dim3(SsRowShape<M>::WGS), 0, s, H, A, C, r0, n, ld, out);                             \
        break;
            SG_PAIRS(128) SG_PAIRS(256) SG_PAIRS(512) SG_PAIRS(1024) SG_PAIRS(2048)
#undef SG_PAIRS
        default: return false;
        }
        if (mfull < mc)
            hipLaunchKernelGGL(k_ss_scatter_pairs<false>, dim3((n + 31) / 32, (mc - mfull + 255) / 256), dim3(256), 0, s,
                               out, ld, n, N, mfull, mc, coef, modes, H, self, A, C, r0, 0);
        if (mfull > 0) {
            const size_t per_tile = (size_t)C.nk * SG_SS_TI;
            const int t0 = (int)(r0 / per_tile), t1 = (int)((r0 + n - 1) / per_tile) + 1;
            const int half = (C.nk + SG_SS_TI) / 2 + SG_SS_TI * ((C.nk + 2 * SG_SS_TI - 2) / SG_SS_TI) / 2;
            hipLaunchKernelGGL(k_ss_scatter_pairs<true>, dim3((unsigned)(half * (t1 - t0)), (mfull + 255) / 256),
                               dim3(256), 0, s, out, ld, n, N, 0, mfull, coef, modes, H, self, A, C, r0, t0);
        }
    }
    return true;
}

sg_status sg_ss_table_build(const sg_grid *grid, int nf, const double *d_H, uint32_t flags, void *d_table,
                            void *d_ws, hipStream_t s)
{
    const int nr = grid->n_r, nphi = grid->n_phi;
    const double du = sg_ss_du(*grid, flags);  // band rule (and log-grid spacing)
    const bool full = (flags & SG_SS_FULL) != 0;
    const bool lin = (flags & SG_LINEAR_R) != 0;
    const double dr = (grid->r_max - grid->r_min) / nr;
    const SsLayout L = sg_ss_layout(nr, nphi, nf, du, full);
    const double dphi = 2.0 * SG_PI / nphi;
    char *tb = (char *)d_table;
    double *self = (double *)d_ws;
    float2 *chunk = (float2 *)((char *)d_ws + sg_align256(sizeof(double) * (size_t)nf * nf * nr));
    const bool excl = (flags & SG_SELF_CELL_EXCLUDE) != 0;
    const bool second = (flags & SG_SECOND_ORDER) != 0;  // log grid, force operators

    hipLaunchKernelGGL(k_twiddles, dim3((nphi + 255) / 256), dim3(256), 0, s, (float2 *)(tb + L.off_tw_phi), nphi);
    SG_HIP(hipGetLastError());
    SsMode *modes = (SsMode *)(tb + L.off_modes);
    hipLaunchKernelGGL(k_ss_modes, dim3(1), dim3(256), 0, s, modes, L.ncol, nr, L.nrt, nf, du, full ? 1 : 0);
    SG_HIP(hipGetLastError());
    float2 *coef = (float2 *)(tb + L.off_coef);
    const bool pot = (flags & SG_POTENTIAL) != 0;
    SsRowArgs A;
    A.nr = nr;
    A.nrt = L.nrt;
    A.nf = nf;
    A.excl = excl ? 1 : 0;
    A.ind = (flags & SG_INDIRECT) ? 1 : 0;
    A.pot = pot ? 1 : 0;
    A.lnrmin = log(grid->r_min);
    A.du = du;
    A.dphi = dphi;
    A.lin = lin ? 1 : 0;
    A.rmin = grid->r_min;
    A.dr = dr;
    A.second = second ? 1 : 0;
    sg_gl_nodes(A.gl, du / dphi);
    const std::vector<SsPart> parts = ss_parts(A, nphi, full, SG_SS_ALIAS);
    if (L.max_w >= 0 || parts[0].C.on) {  // entries the scatter does not reach stay zero
        hipLaunchKernelGGL(k_ss_zero, dim3(2048), dim3(256), 0, s, coef, L.coef_elems);
        SG_HIP(hipGetLastError());
    }
    if (!excl && !second) {  // second order: the own cell is a hat weight of the rows
        // one item per (pair, ring): the per-cell quadratures with one cell per ring
        if (lin) {
            GLNodes gl;
            sg_gl_nodes(gl, sg_lin_aspect(*grid, dphi));
            hipLaunchKernelGGL(k_ss_self_lin, dim3(nf * nf * nr), dim3(256), 0, s, d_H, nf, nr, 1, grid->r_min, dr,
                               dphi, pot ? 1 : 0, 0, self, gl);
        } else if (pot) {
            sg_pot_cells<double>(d_H, nullptr, nf, nr, 1, log(grid->r_min), du, dphi, 0, self, 0, s);
            SG_HIP(hipGetLastError());
            // own-cell integral I of P: the sample -I / (du dphi) scales to I / N
            hipLaunchKernelGGL(k_ss_scale, dim3((nf * nf * nr + 255) / 256), dim3(256), 0, s, self, nf * nf * nr,
                               -1.0 / (du * dphi));
        } else {
            sg_self_cells<double>(d_H, nf, nr, 1, log(grid->r_min), du, dphi, self, s);
        }
        SG_HIP(hipGetLastError());
    }
    // the chunk buffer holds whole units of each class's rows
    const size_t cbytes = sizeof(float2) * (size_t)L.ncol * ss_chunk_rows(L);
    for (const SsPart &P : parts) {
        // modes that the class's nearest ring pairs keep (on a uniform grid the
        // band is counted in rings, so by M alone): full ones, and banded ones
        // whose band reaches them
        int mc = P.M / 2 + 1;
        if (P.C.on && !lin) {
            const int k1 = P.C.K1;
            while (mc > 1) {
                const int w = sg_ss_band(mc - 1, nr, du, full);
                if (!sg_ss_is_banded(w, nr) || w >= k1) break;
                --mc;
            }
        }
        int mfull = 0;  // the leading full modes
        while (mfull < mc && !sg_ss_is_banded(sg_ss_band(mfull, nr, du, full), nr)) ++mfull;
        if (P.C.on && P.kind == 0 && !lin) {
            if (!build_pairs(d_H, self, A, P, mc, mfull, chunk, cbytes, coef, modes, s)) return SG_ERR_UNSUPPORTED;
            SG_HIP(hipGetLastError());
            continue;
        }
        const size_t rows = P.C.on ? ss_class_rows(A, P.C) : L.rows;
        size_t crows = P.C.on ? cbytes / (sizeof(float2) * mc) / SG_SS_TI * SG_SS_TI : ss_chunk_rows(L);
        if (crows > (size_t)1 << 30) crows = (size_t)1 << 30;
        for (size_t r0 = 0; r0 < rows; r0 += crows) {
            const int n = (int)std::min(crows, rows - r0);
            if (!dispatch_ss_rows(d_H, self, A, P, r0, n, mc, chunk, s)) return SG_ERR_UNSUPPORTED;
            SG_HIP(hipGetLastError());
            const int ms = P.C.on ? mfull : 0;
            if (ms < mc)
                hipLaunchKernelGGL(k_ss_scatter<false>, dim3((n + 31) / 32, (mc - ms + 255) / 256), dim3(256), 0, s,
                                   chunk, mc, n, mc, ms, coef, (const SsMode *)modes, A, P.C, r0, 0);
            if (ms > 0) {
                const size_t per_tile = (size_t)P.C.nk * SG_SS_TI;
                const int t0 = (int)(r0 / per_tile), t1 = (int)((r0 + n - 1) / per_tile) + 1;
                const int side = P.C.K1 == 0 ? 2 * P.C.K2 - 1 + (SG_SS_TI - 1) : P.C.K2 - P.C.K1 + (SG_SS_TI - 1);
                const int half = ((P.C.K1 == 0 ? side : 2 * side) + 1) / 2;
                hipLaunchKernelGGL(k_ss_scatter<true>, dim3((unsigned)(half * (t1 - t0)), (ms + 255) / 256), dim3(256),
                                   0, s, chunk, mc, n, ms, 0, coef, (const SsMode *)modes, A, P.C, r0, t0);
            }
            SG_HIP(hipGetLastError());
        }
    }
    sg_ss_header proto{};
    proto.magic = SG_SS_MAGIC;
    proto.version = 1;
    proto.n_r = nr;
    proto.n_phi = nphi;
    proto.n_fluids = nf;
    proto.flags = flags | SG_SEMI_SPECTRAL;
    proto.r_min = grid->r_min;
    proto.r_max = grid->r_max;
    proto.du = du;
    proto.total_bytes = L.total;
    hipLaunchKernelGGL(k_ss_header, dim3(1), dim3(1), 0, s, (sg_ss_header *)tb, proto);
    SG_HIP(hipGetLastError());
    return SG_OK;
}

// ------------------------------------------------------------ middle pass
// 16-byte load of two consecutive complex values at element offset i of a
// wave-uniform base (i even); NT: non-temporal (the operators are read once
// per solve, so they need not displace Sigma~ and g^ in the caches).
template <bool NT>
__device__ inline void ss_ld4(const float2 *p, uint32_t i, float2 &x, float2 &y)
{
    const sg_gcv4f *q = (const sg_gcv4f *)((const char *)p + (i << 3));
    sg_v4f v;
    if constexpr (NT) v = __builtin_nontemporal_load(q);
    else v = *q;
    x = make_float2(v.x, v.y);
    y = make_float2(v.z, v.w);
}

// Workgroup job (disc, m, b, target block): 256 threads in S row splits of
// LN = 256 / S lanes; lane l owns targets i0 .. i0 + V - 1, i0 = block TB +
// V l (TB = LN V), and split s sums the operator rows k = s (mod S) of every
// source fluid (source rows of a full mode, diagonals of a banded one); the
// splits are combined through LDS.  Sigma~_a(m, .) is staged in LDS first:
// the whole column for a full mode; for a banded mode the window of sources
// the block's targets reach, from blk TB - w (zero outside the grid), so
// that target i0 + v reads source i0 + v + d - w at window index V l + v + d.  The operator rows
// are streamed once with 16-byte loads, U rows in flight: this pass is bound
// by reading the table.
template <int NF, int V, int S, bool NT, int U, int SRC>
__global__ void __launch_bounds__(256) k_ss_pass(const DiscDev *discs, const WJob *wj, int nj, const float2 *,
                                                 int kc, OneDisc one)
{
    extern __shared__ __attribute__((aligned(16))) float2 ssh[];
    constexpr int LN = 256 / S, TB = LN * V;
    static_assert(V % 2 == 0, "targets per lane come in 16-byte pairs");
    const int w = sg_uniform(sg_xcd_remap(blockIdx.x, kc));
    if (w >= nj) return;
    DiscDev D;
    const WJob job = pass_job<SG_PASS_SS, SRC>(discs, wj, one, w, 1, D);
    if (job.n == 0) return;  // cluster padding
    const int idx = job.base;
    const int nr = D.nr, nrt = (nr + 1) & ~1, nb = (nr + TB - 1) / TB;
    const int blk = idx % nb, mb = idx / nb, b = mb % NF, m = mb / NF;
    const size_t fs = sg_blk_field_elems(D.nphi, nr);
    const SsMode md = D.modes[m];
    const bool banded = sg_uniform(md.banded) != 0;
    const int bw = banded ? sg_uniform(md.w) : 0;
    // staged sources: a full mode's whole column, a banded mode's window
    // [blk TB - w, blk TB + TB + w + 4) (zero outside the grid)
    const int cs = banded ? TB + 2 * bw + 4 : nr;
    const int nk = banded ? 2 * bw + 1 : nr;        // operator rows per (b, a)
    const int base = banded ? blk * TB - bw : 0;
    if (banded && bw > D.ss_wmax) return;  // table not built for this grid: never overrun the LDS
    for (int e = threadIdx.x; e < NF * cs; e += 256) {
        const int a = e / cs, ip = e - a * cs + base;
        ssh[e] = (ip >= 0 && ip < nr) ? gld2(D.st + a * fs, (uint32_t)sg_blk_index(m, ip, nr))
                                      : make_float2(0.f, 0.f);
    }
    __syncthreads();
    const int ln = threadIdx.x % LN, sp = threadIdx.x / LN;
    const int i0 = blk * TB + V * ln;
    // column of each target pair (pairs past the last row read column 0) and
    // each target's staged index (targets past the last row read index 0)
    uint32_t col[V / 2];
    int ie[V];
#pragma unroll
    for (int v = 0; v < V; v += 2) col[v / 2] = i0 + v < nr ? (uint32_t)(i0 + v) : 0u;
#pragma unroll
    for (int v = 0; v < V; ++v) ie[v] = i0 + v < nr ? V * ln + v : 0;
    float2 ar[V], ap[V];
#pragma unroll
    for (int v = 0; v < V; ++v) ar[v] = ap[v] = make_float2(0.f, 0.f);
    const float2 *C = D.spec + md.off;
    for (int a = 0; a < NF; ++a) {
        const float2 *Tm = C + (size_t)(b * NF + a) * nk * nrt;
        const float2 *sa = ssh + a * cs;
        int k = sp;
        for (; k + S * (U - 1) < nk; k += S * U) {
            float2 t[U][V];
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int v = 0; v < V; v += 2)
                    ss_ld4<NT>(Tm, (uint32_t)(k + S * u) * nrt + col[v / 2], t[u][v], t[u][v + 1]);
#pragma unroll
            for (int u = 0; u < U; ++u) {
#pragma unroll
                for (int v = 0; v < V; ++v) {
                    // full: source row k (all targets); banded: diagonal k
                    const float2 s = banded ? sa[ie[v] + k + S * u] : sa[k + S * u];
                    ar[v].x += t[u][v].x * s.x;
                    ar[v].y += t[u][v].x * s.y;
                    ap[v].x += t[u][v].y * s.x;
                    ap[v].y += t[u][v].y * s.y;
                }
            }
        }
        for (; k < nk; k += S) {
            float2 t[V];
#pragma unroll
            for (int v = 0; v < V; v += 2) ss_ld4<NT>(Tm, (uint32_t)k * nrt + col[v / 2], t[v], t[v + 1]);
#pragma unroll
            for (int v = 0; v < V; ++v) {
                const float2 s = banded ? sa[ie[v] + k] : sa[k];
                ar[v].x += t[v].x * s.x;
                ar[v].y += t[v].x * s.y;
                ap[v].x += t[v].y * s.x;
                ap[v].y += t[v].y * s.y;
            }
        }
    }
    if constexpr (S > 1) {
        // combine the row splits: partials after the staged columns
        float2 *red = ssh + ((NF * cs + 1) & ~1);
        if (sp > 0) {
#pragma unroll
            for (int v = 0; v < V; ++v) {
                red[((sp - 1) * LN + ln) * 2 * V + 2 * v] = ar[v];
                red[((sp - 1) * LN + ln) * 2 * V + 2 * v + 1] = ap[v];
            }
        }
        __syncthreads();
        if (sp > 0) return;
#pragma unroll
        for (int q = 0; q < S - 1; ++q)
#pragma unroll
            for (int v = 0; v < V; ++v) {
                const float2 x = red[(q * LN + ln) * 2 * V + 2 * v], y = red[(q * LN + ln) * 2 * V + 2 * v + 1];
                ar[v].x += x.x;
                ar[v].y += x.y;
                ap[v].x += y.x;
                ap[v].y += y.y;
            }
    }
    float2 *gr = D.gh + (size_t)(b * 2) * fs, *gp = gr + fs;
#pragma unroll
    for (int v = 0; v < V; ++v) {
        const int i = i0 + v;
        if (i < nr) {
            const uint32_t o = (uint32_t)sg_blk_index(m, i, nr);
            gst2(gr, o, ar[v]);
            gst2(gp, o, make_float2(-ap[v].y, ap[v].x));  // i t_phi Sigma~
        }
    }
}

template <int NF, int V, int S, bool NT = false, int U = 8> static SsPassInfo ss_info()
{
    constexpr int LN = 256 / S;
    SsPassInfo k;
    k.fn = k_ss_pass<NF, V, S, NT, U, SG_SRC_BATCH>;
    k.fn_one = k_ss_pass<NF, V, S, NT, U, SG_SRC_ONE>;
    k.wgs = 256;
    k.tb = LN * V;
    k.lds_per_row = NF * (int)sizeof(float2);
    // column padded to an even count, then the split partials
    k.lds_fixed = (int)sizeof(float2) * (1 + (S > 1 ? (S - 1) * LN * 2 * V : 0));
    return k;
}

template <int NF> static bool ss_variant(int variant, SsPassInfo &out)
{
    switch (variant) {
    case 1: out = ss_info<NF, 2, 4, true>(); return true;
    case 2: out = ss_info<NF, 2, 1>(); return true;
    case 3: out = ss_info<NF, 4, 1>(); return true;
    case 4: out = ss_info<NF, 2, 4>(); return true;
    default: return false;
    }
}

bool sg_ss_pass_kernel(int nf, int variant, SsPassInfo &out)
{
    switch (nf) {
    case 1: return ss_variant<1>(variant, out);
    case 2: return ss_variant<2>(variant, out);
    case 3: return ss_variant<3>(variant, out);
    case 4: return ss_variant<4>(variant, out);
    default: return false;
    }
}

// Row splits with 128 targets per job and non-temporal operator loads
// measured fastest on every grid tried (256 x 512 to 1200 x 2048: many jobs
// per mode, short banded windows, Sigma~ and g^ kept in the caches); the
// autotuner tries the other shapes.
int sg_ss_default_variant(int) { return 1; }

// ------------------------------------------------ dL/dH (gradient in H(r))
// For L with dL/dg_r = lam_r, dL/dg_phi = lam_phi, the derivative with
// respect to the ring scale heights follows from differentiating every
// operator entry: T^{ab}(m, i, i') depends on h_a = H_a(r_i')/r_i' (source)
// and h_b = H_b(r_i)/r_i (target), the own-cell entry on both at its ring,
// and mode 1 on H_a(r_i') through the folded indirect term.  Since g is the
// inverse transform of the per-mode products,
//   dL/dtheta = sum_m w_m Re[conj(lam~_r) dT_r Sigma~ + conj(lam~_phi) i dt_phi Sigma~]
// (w_m = 1 for m = 0, n_phi/2 and 2 otherwise: the stored half of a
// Hermitian spectrum), accumulated per (b, a, i', i) row and added to
// dL/dh_a(i') and dL/dh_b(i) in double; finally dL/dH = (dL/dh) / r.  The
// derivative rows are sampled and transformed on the fly (the table's own
// construction with the kernels' h derivatives), never stored.

// Half spectra of lam rows (b, i) (r and phi parts) and of Sigma row pairs, by
// rings: lt [b][i][m] (lam_r~, lam_phi~) and st [a][i][m].  (The contraction
// reads them along m, once per ring pair; in the passes' tiles of 4 x 4, one
// 8-byte value from each 32-byte sector, those reads were a third of the
// kernel.)
template <int N>
__global__ void __launch_bounds__(SsRowShape<N>::WGS)
k_ssg_phi(const float *lam_r, const float *lam_p, const float *sigma, const float2 *tw, float4 *lt, float2 *st,
          int nr, int nf)
{
    using S = SsRowShape<N>;
    constexpr int P = S::P, T = S::T, G = S::G, W = LdsPlane<float>::elems(N), NC = N / 2 + 1;
    __shared__ __attribute__((aligned(16))) float2 lds[W * G];
    const int g = threadIdx.x / T, t = threadIdx.x % T;
    const int hp = (nr + 1) / 2, nl = nf * nr, count = nl + nf * hp;
    const int idx = blockIdx.x * G + g;
    const bool valid = idx < count;
    const int j = valid ? idx : 0;
    const LdsPlane<float> pl{lds + W * g};
    const float *x1, *x2;
    size_t r1, r2;  // rows of st
    if (j < nl) {
        x1 = lam_r + (size_t)j * N;
        x2 = lam_p + (size_t)j * N;
        r1 = r2 = (size_t)j;
    } else {
        const int q = j - nl, a = q / hp, jj = q % hp;
        r1 = (size_t)a * nr + 2 * jj;
        r2 = (size_t)a * nr + min(2 * jj + 1, nr - 1);
        x1 = sigma + r1 * N;
        x2 = sigma + r2 * N;
    }
    float2 z[P];
    p1_load<N>(x1, x2, z, t);
    fft<N, false>(z, t, pl, TwTable{tw});
#pragma unroll
    for (int p = 0; p < P; ++p) pl.st(t + T * p, z[p]);
    __syncthreads();
    if (!valid) return;
    for (int m = t; m < NC; m += T) {
        // the Hermitian split of pass 1
        const float2 Z = pl.ld(m), C = pl.ld((N - m) & (N - 1));
        const float2 v1 = make_float2(0.5f * (Z.x + C.x), 0.5f * (Z.y - C.y));
        const float2 v2 = make_float2(0.5f * (Z.y + C.y), -0.5f * (Z.x - C.x));
        if (j < nl) {
            lt[r1 * NC + m] = make_float4(v1.x, v1.y, v2.x, v2.y);
        } else {
            gstore2(st, r1 * NC + m, v1);
            gstore2(st, r2 * NC + m, v2);  // (an odd last row is its own partner)
        }
    }
}

// Contraction of one mode of the row with lam~ and Sigma~:
// Re[conj(lr) T_r s] + Re[conj(lp) i t_phi s] = T_r cr + t_phi cp.
__device__ inline void ssg_mode(const float4 *lt, const float2 *st, size_t ro, size_t so, int m, double &cr, double &cp)
{
    typedef float v4 __attribute__((ext_vector_type(4)));
    const v4 l = ((const __attribute__((address_space(1))) v4 *)lt)[ro + m];
    const float2 sv = gload2(st, so + m);
    cr = (double)l.x * sv.x + (double)l.y * sv.y;
    cp = -(double)l.z * sv.y + (double)l.w * sv.x;
}

// Point-sampled rows, a ring pair at a time.  Both h derivatives of both
// operators of a ring pair, (b, a, i', i) and its mirror (a, b, i, i'), are
// one even function of phi, S = D(x(phi)) (E for the potential), times
//   K_r = p (e^X - cos phi) = p ((e^X - 1) + (1 - cos phi)),  K_phi = p sin phi
// with p and X of the row and the derivative.  The products with 1 - cos phi
// and sin phi are differences of neighbouring modes of S~ (exact for the
// sampled sequences), so a ring pair takes one real transform where its two
// rows and two derivatives took four, and one evaluation per azimuth of half
// the circle where the rows took two; a group transforms two ring pairs at
// once as z_A + i z_B (S~ is real).  The differences cost digits of the double
// rounding: 1e-16/|X| of a row's largest coefficient, for i' = i 1e-16/dphi^2
// (dL/dH itself moved by 5e-13 of its largest at 600 x 1024; the float spectra
// of lam and Sigma leave 1e-7 of it).
// The own-cell sample of i = i' enters as a constant of all modes.
// On a uniform grid the classes of a row and of its mirror differ: rows then
// stand alone (both signs of k).  Index: as ss_row's with offsets k >= 0.
// The transforms bound it with the evaluations (both FP64 with LDS traffic).
// 600 x 1024 two-fluid, all rows: 3.86 -> 1.90 ms.
template <int N>
__global__ void __launch_bounds__(SsRowShape<N>::WGS)
k_ssg_pairs(const double *H, const double *dself, SsRowArgs A, SsClass C, int nphi, const float4 *lt,
            const float2 *st, size_t r0, int nrows, double *rowpart)
{
    using S = SsRowShape<N>;
    constexpr int P = S::P, T = S::T, G = S::G, W = LdsPlane<double>::elems(N);
    constexpr int NC = N / 2 + 1, SUB = T < 64 ? T : 64, NS = T / SUB;
    __shared__ __attribute__((aligned(16))) double2 lds[W * G];
    __shared__ __attribute__((aligned(16))) double wq[FQuad<double>::TABLE];
    __shared__ double red[G * NS * 4];
    __shared__ double ext[G * 4];  // cr + cp of mode 1 (the indirect term), by ring pair and direction
    const int g = threadIdx.x / T, t = threadIdx.x % T;
    const LdsPlane<double> pl{lds + W * g};
    const int row = (blockIdx.x * G + g) * 2;
    int ic[2], ip[2], a = 0, b = 0;
    bool live[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        int ua, ub;
        live[u] = ss_row(A, C, (uint32_t)r0 + (row + u < nrows ? row + u : 0), ub, ua, ip[u], ic[u]) && row + u < nrows;
        if (live[u]) {
            a = ua;  // a unit's rows are of one fluid pair
            b = ub;
        } else {
            ic[u] = ip[u] = 0;
        }
    }
    if (!__syncthreads_or(live[0] || live[1] ? 1 : 0)) return;
    sg_fill64(wq, A.pot ? SG_FN_E : SG_FN_D);
    // x(phi) = xa (x0 + 2 sin^2(phi / 2)), also the potential's s^2 / (8 H_ab^2)
    double x0[2], xa[2], ri[2], rp[2], X[2], ha[2], hb[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        ri[u] = A.lin ? A.rmin + (ic[u] + 0.5) * A.dr : exp(A.lnrmin + (ic[u] + 0.5) * A.du);
        rp[u] = A.lin ? A.rmin + (ip[u] + 0.5) * A.dr : exp(A.lnrmin + (ip[u] + 0.5) * A.du);
        ha[u] = H[a * A.nr + ip[u]] / rp[u];
        hb[u] = H[b * A.nr + ic[u]] / ri[u];
        X[u] = A.lin ? log(ri[u] / rp[u]) : (double)(ic[u] - ip[u]) * A.du;
        const ConvRowDh64 d = sg_conv_row64_dh(X[u], ha[u], hb[u]);
        x0[u] = d.two_sxh2;
        xa[u] = d.inv4h2;
    }
    __syncthreads();
#pragma unroll 1
    for (int q = t; q <= N / 2; q += T) {
        double sh, ch, v[2];
        ss_half_angle<N>(q, sh, ch);
        const double two_s2 = 2.0 * sh * sh;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            v[u] = 0.0;
            if (!live[u] || (ic[u] == ip[u] && q == 0)) continue;
            const double x = (x0[u] + two_s2) * xa[u];
            v[u] = A.pot ? sg_E64(x, wq) : sg_D64(x, wq);
        }
        const double2 z = make_double2(v[0], v[1]);
        pl.st(q, z);
        if (q != 0 && q != N / 2) pl.st(N - q, z);
    }
    __syncthreads();
    double2 z[P];
#pragma unroll
    for (int p = 0; p < P; ++p) z[p] = pl.ld(t + T * p);
    __syncthreads();
    fft<N, false>(z, t, pl, TwPow64<N>{t});
#pragma unroll
    for (int p = 0; p < P; ++p) pl.st(t + T * p, z[p]);
    __syncthreads();
    // acc[u][0]: the row; [u][1]: its mirror, or (i = i') the sum of w cr
    double acc[2][2] = {{0.0, 0.0}, {0.0, 0.0}};
    const double b1 = A.pot ? 0.0 : 1.0;
    double c0[2][2];  // K_r = p (c0 S + b1 (1 - cos) S)
    size_t ro[2][2], so[2][2];
    const int ncol = nphi / 2 + 1;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        double sx, ep, em;
        sg_exp_half(X[u], sx, ep, em);
        c0[u][0] = A.pot ? 1.0 : 2.0 * sx * ep;
        c0[u][1] = A.pot ? 1.0 : -2.0 * sx * em;
        ro[u][0] = ((size_t)b * A.nr + ic[u]) * ncol;
        so[u][0] = ((size_t)a * A.nr + ip[u]) * ncol;
        ro[u][1] = ((size_t)a * A.nr + ip[u]) * ncol;
        so[u][1] = ((size_t)b * A.nr + ic[u]) * ncol;
    }
    for (int m = t; m < NC; m += T) {
        const double2 z0 = pl.ld(m), zl = pl.ld(m == 0 ? 1 : m - 1), zh = pl.ld((m + 1) & (N - 1));
        const double wm = (m == 0 || m == nphi / 2) ? 1.0 : 2.0;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            if (!live[u]) continue;
            const double s0 = u ? z0.y : z0.x, sl = u ? zl.y : zl.x, sh = u ? zh.y : zh.x;
            const double B = b1 * (s0 - 0.5 * (sl + sh)), tp = b1 * 0.5 * (sh - sl);
            double cr, cp;
            ssg_mode(lt, st, ro[u][0], so[u][0], m, cr, cp);
            acc[u][0] += wm * ((c0[u][0] * s0 + B) * cr + tp * cp);
            if (m == 1) ext[(g * 2 + u) * 2] = cr + cp;
            if (ic[u] == ip[u]) {
                acc[u][1] += wm * cr;
            } else if (!A.lin) {
                ssg_mode(lt, st, ro[u][1], so[u][1], m, cr, cp);
                acc[u][1] += wm * ((c0[u][1] * s0 + B) * cr + tp * cp);
                if (m == 1) ext[(g * 2 + u) * 2 + 1] = cr + cp;
            }
        }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        double x = acc[e >> 1][e & 1];
#pragma unroll
        for (int o = SUB / 2; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
        if (t % SUB == 0) red[(g * NS + t / SUB) * 4 + e] = x;
    }
    __syncthreads();
    // thread (u, dir) of the group writes the row's partials (part 0 belongs
    // to dL/dh_a at the source ring, part 1 to dL/dh_b at the target ring);
    // k_ssg_finish adds them up
    for (int e = t; e < 4; e += T) {
        const int dir = e & 1;
        const bool second = e >= 2;
        if (!(second ? live[1] : live[0])) continue;
        const int ii = second ? ic[1] : ic[0], jj = second ? ip[1] : ip[0];
        if (dir && (ii == jj || A.lin)) continue;
        double sum = 0.0, own = 0.0;
        for (int w = 0; w < NS; ++w) {
            sum += red[(g * NS + w) * 4 + e];
            if (ii == jj) own += red[(g * NS + w) * 4 + e + 1];
        }
        const double r1 = second ? ri[1] : ri[0], r2 = second ? rp[1] : rp[0];
        const double h1 = second ? ha[1] : ha[0], h2 = second ? hb[1] : hb[0], Xr = second ? X[1] : X[0];
        const int tb = dir ? a : b, ta = dir ? b : a, ti = dir ? jj : ii, tj = dir ? ii : jj;
        const double tr = dir ? r2 : r1, tq = dir ? r1 : r2;    // target and source radius
        const double sa = dir ? h2 : h1, sb = dir ? h1 : h2;    // their h: source, target
        double p1, p2;
        if (A.pot) {
            // d/dh of r'^2 G0(y) / (2 sqrt(pi) H_ab) (the forward's sample):
            // d(G0/H)/dH = (2 y F(y) - G0(y)) / H^2, dH_ab/dh_a = H_a r' / (2 H_ab),
            // dH_ab/dh_b = H_b r_i / (2 H_ab); even in phi (no K_phi part)
            const double Ha = sa * tq, Hb = sb * tr, Hab2 = 0.5 * (Ha * Ha + Hb * Hb), Hab = sqrt(Hab2);
            const double dq = tq * tq / (2.0 * SG_SQRT_PI * Hab2);
            p1 = dq * Ha * tq / (2.0 * Hab);
            p2 = dq * Hb * tr / (2.0 * Hab);
        } else {
            const ConvRowDh64 d = sg_conv_row64_dh(dir ? -Xr : Xr, sa, sb);
            p1 = d.p1;
            p2 = d.p2;
        }
        const double scale = -(A.lin ? A.dr / tq : A.du) * A.dphi / N;
        double v1 = p1 * sum, v2 = p2 * sum;
        if (ii == jj && !A.excl) {
            const size_t o = (size_t)(ta * A.nf + tb) * A.nr + ti, wst = (size_t)A.nf * A.nf * A.nr;
            v1 += dself[o] * own;
            v2 += dself[wst + o] * own;
        }
        if (A.ind) {
            // d/dh_a of r'^2 sqrt(2) K_a(r'/H_a) n_phi / 2, H_a = h_a r':
            // dK_a/dH = pi^{-1/2} r' / (4 H^4) (-3 F(x) - 2 x F'(x)), x = r'^2 / (4 H^2)
            const double Ha = sa * tq, x = tq * tq / (4.0 * Ha * Ha);
            const double dK = (1.0 / SG_SQRT_PI) * tq / (2.0 * Ha * Ha * Ha * Ha) * sg_D64(x, wq);
            v1 += 2.0 * tq * tq * SG_SQRT2 * dK * tq * (0.5 * N) *
                  ext[(g * 2 + (second ? 1 : 0)) * 2 + dir];
        }
        double *o = rowpart + 2 * ((((size_t)tb * A.nf + ta) * A.nr + tj) * A.nrt + ti);
        o[0] = scale * v1;
        o[1] = scale * v2;
    }
}

// The rows of second-order operators: one group of T threads per (b, a, i', i)
// row, for which = 1 (d/dh_a, source) and 2 (d/dh_b, target) the derivative
// samples are transformed as in k_ss_rows and contracted with lam~ and Sigma~
// of the row's mode column.  The samples are the h derivatives of the hat
// weights (k_ss_rows<N, 1>: integrated near the singular point, point value
// plus second moments beyond; both are linear in the kernel, so they apply to
// its derivatives sample by sample).
// N: samples of the rows, as in k_ss_rows; the contraction runs over the modes
// they resolve (m <= N/2; the others' derivatives are below e^{-48} of the
// axisymmetric one).  nphi: the grid's.  SO as in k_ss_rows.
template <int N, int SO>
__global__ void __launch_bounds__(SsRowShape<N>::WGS)
k_ssg_rows(const double *H, const double *dself, SsRowArgs A, SsClass C, int nphi, const float4 *lt,
           const float2 *st, size_t r0, int nrows, double *rowpart)
{
    using S = SsRowShape<N>;
    constexpr int P = S::P, T = S::T, G = S::G, W = LdsPlane<double>::elems(N);
    constexpr int NC = N / 2 + 1;
    __shared__ __attribute__((aligned(16))) double2 lds[W * G];
    __shared__ __attribute__((aligned(16))) double wq[FQuad<double>::TABLE];
    __shared__ double red[S::WGS];
    __shared__ double2 qres[(SO & 1) ? 2 * NC * G : 1];  // SO: the group's integrated samples, both derivatives
    __shared__ int qmax_wg;
    const int g = threadIdx.x / T, t = threadIdx.x % T;
    const LdsPlane<double> pl{lds + W * g};
    const int row = blockIdx.x * G + g;
    int i, ip, a, b;
    const bool valid = ss_row(A, C, (uint32_t)r0 + (row < nrows ? row : 0), b, a, ip, i) && row < nrows;
    if (!__syncthreads_or(valid ? 1 : 0)) return;
    if (!valid) b = a = ip = i = 0;
    sg_fill64(wq, SG_FN_D);
    const bool live = valid && i < A.nr;
    const int ic = i < A.nr ? i : A.nr - 1;
    const double ri = A.lin ? A.rmin + (ic + 0.5) * A.dr : exp(A.lnrmin + (ic + 0.5) * A.du);
    const double rp = A.lin ? A.rmin + (ip + 0.5) * A.dr : exp(A.lnrmin + (ip + 0.5) * A.du);
    const double ha = H[a * A.nr + ip] / rp, hb = H[b * A.nr + ic] / ri;
    const double X = A.lin ? log(ri / rp) : (double)(ic - ip) * A.du;
    const double scale = -(A.lin ? A.dr / rp : A.du) * A.dphi / N;
    const int ncol = nphi / 2 + 1;
    __syncthreads();
    // Both derivatives are sampled in one sweep (one F, F' evaluation per
    // azimuth) and transformed together.  Row d is z_d = K_r,d + i K_phi,d
    // with K_r even and K_phi odd in phi, so its transform Z_d is real; the
    // plane holds z = z_1 + i z_2, whose transform carries Z_1 (d/dh_a) in
    // its real part and Z_2 (d/dh_b) in its imaginary part.
    constexpr int Q = P / 2 + 1;
    // the row and its D_X neighbours
    const ConvRowDh64 d0 = sg_conv_row64_dh(X, ha, hb), dp = sg_conv_row64_dh(X + A.du, ha, hb),
                      dm = sg_conv_row64_dh(X - A.du, ha, hb);
    if constexpr ((SO & 1) != 0) {
        // integrated samples, cooperatively (as in k_ss_rows<N, true>)
        const int Pr = ic - ip;
        const double rn = SG_SS_HAT_NEAR * fmax(A.du, A.dphi), xq = Pr * A.du;
        int qn = -1;
        if (live && xq * xq < rn * rn)
            while (qn < N / 2 && xq * xq + ((qn + 1) * A.dphi) * ((qn + 1) * A.dphi) < rn * rn) ++qn;
        if (threadIdx.x == 0) qmax_wg = -1;
        __syncthreads();
        if (t == 0 && qn >= 0) atomicMax(&qmax_wg, qn);
        __syncthreads();
        const int qm = qmax_wg;
        for (int q = 0; q <= qm; ++q) {
            for (int d = 1; d <= 2; ++d) {
                double wr = 0.0, wp = 0.0;
                if (q <= qn) sg_hat_weight_part<SO == 3>(Pr, q, A.du, A.dphi, ha, hb, d, A.gl, wq, t, T, wr, wp);
                pl.st(t, make_double2(wr, wp));
                __syncthreads();
                if (q <= qn && t == 0) {
                    double sr = 0.0, sp = 0.0;
                    for (int k = 0; k < T; ++k) {
                        const double2 v = pl.ld(k);
                        sr += v.x;
                        sp += v.y;
                    }
                    qres[(g * 2 + (d - 1)) * NC + q] = make_double2(sr, sp);
                }
                __syncthreads();
            }
        }
        // point values of the packed derivative rows (for the neighbours),
        // and the second-order samples in registers: vq at q, vm at N - q
        double2 vq[Q], vm[Q];
        unsigned taylor = 0u;
#pragma unroll
        for (int u = 0; u < Q; ++u) {
            const int q = t + T * u;
            vq[u] = make_double2(0.0, 0.0);
            vm[u] = make_double2(0.0, 0.0);
            if (q > N / 2) continue;
            double sh, ch;
            ss_half_angle<N>(q, sh, ch);
            const double s2 = 2.0 * sh * ch;
            double kr1 = 0.0, kp1 = 0.0, kr2 = 0.0, kp2 = 0.0;
            if (Pr != 0 || q != 0) sg_conv_kernel64_dh(d0, sh, s2, wq, kr1, kp1, kr2, kp2);
            if (q <= qn) {
                const double2 w1 = qres[(g * 2 + 0) * NC + q], w2 = qres[(g * 2 + 1) * NC + q];
                vq[u] = make_double2(w1.x - w2.y, w1.y + w2.x);
                vm[u] = make_double2(w1.x + w2.y, w2.x - w1.y);
            } else {
                // D_X^2 of the packed rows: samples at X +- du
                double a1, b1, c1, e1, a2, b2, c2, e2;
                sg_conv_kernel64_dh(dp, sh, s2, wq, a1, b1, c1, e1);
                sg_conv_kernel64_dh(dm, sh, s2, wq, a2, b2, c2, e2);
                const double dr1 = a1 - 2.0 * kr1 + a2, dp1 = b1 - 2.0 * kp1 + b2;
                const double dr2 = c1 - 2.0 * kr2 + c2, dp2 = e1 - 2.0 * kp2 + e2;
                vq[u] = make_double2(kr1 - kp2 + (dr1 - dp2) / 12.0, kp1 + kr2 + (dp1 + dr2) / 12.0);
                vm[u] = make_double2(kr1 + kp2 + (dr1 + dp2) / 12.0, kr2 - kp1 + (dr2 - dp1) / 12.0);
                taylor |= 1u << u;
            }
            pl.st(q, make_double2(kr1 - kp2, kp1 + kr2));
            if (q != 0 && q != N / 2) pl.st(N - q, make_double2(kr1 + kp2, kr2 - kp1));
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < Q; ++u) {
            const int q = t + T * u;
            if (q > N / 2 || !((taylor >> u) & 1u)) continue;
            // D_phi^2 at q and at the mirror N - q (the plane holds the
            // packed rows on the whole circle)
            const double2 z0 = pl.ld(q), zl = pl.ld((q + N - 1) & (N - 1)), zh = pl.ld((q + 1) & (N - 1));
            vq[u].x += (zl.x - 2.0 * z0.x + zh.x) / 12.0;
            vq[u].y += (zl.y - 2.0 * z0.y + zh.y) / 12.0;
            if (q != 0 && q != N / 2) {
                const int qm2 = N - q;
                const double2 y0 = pl.ld(qm2), yl = pl.ld(qm2 - 1), yh = pl.ld((qm2 + 1) & (N - 1));
                vm[u].x += (yl.x - 2.0 * y0.x + yh.x) / 12.0;
                vm[u].y += (yl.y - 2.0 * y0.y + yh.y) / 12.0;
            }
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < Q; ++u) {
            const int q = t + T * u;
            if (q > N / 2) continue;
            pl.st(q, vq[u]);
            if (q != 0 && q != N / 2) pl.st(N - q, vm[u]);
        }
    } else {
#pragma unroll
    for (int u = 0; u < Q; ++u) {
        const int q = t + T * u;
        if (q > N / 2) break;
        double kr1 = 0.0, kp1 = 0.0, kr2 = 0.0, kp2 = 0.0;
        // K + (D_X^2 K + D_phi^2 K)/12 of both derivatives
#pragma unroll 1
        for (int k = 0; k < 5; ++k) {
            const double ph = 2.0 * q / N + (k == 3 ? A.dphi : k == 4 ? -A.dphi : 0.0) / SG_PI;
            double sh, ch, a1, b1, a2, b2;
            sincospi(0.5 * ph, &sh, &ch);
            sg_conv_kernel64_dh(k == 1 ? dp : k == 2 ? dm : d0, sh, 2.0 * sh * ch, wq, a1, b1, a2, b2);
            const double w = k == 0 ? 2.0 / 3.0 : 1.0 / 12.0;
            kr1 += w * a1;
            kp1 += w * b1;
            kr2 += w * a2;
            kp2 += w * b2;
        }
        pl.st(q, make_double2(kr1 - kp2, kp1 + kr2));
        if (q != 0 && q != N / 2) pl.st(N - q, make_double2(kr1 + kp2, kr2 - kp1));
    }
    }
    __syncthreads();
    double2 z[P];
#pragma unroll
    for (int p = 0; p < P; ++p) z[p] = pl.ld(t + T * p);
    __syncthreads();
    fft<N, false>(z, t, pl, TwPow64<N>{t});
#pragma unroll
    for (int p = 0; p < P; ++p) pl.st(t + T * p, z[p]);
    __syncthreads();
    double dind = 0.0;
    if (A.ind) {
        // d/dh_a of r'^2 sqrt(2) K_a(r'/H_a) n_phi / 2, H_a = h_a r':
        // dK_a/dH = pi^{-1/2} r' / (4 H^4) (-3 F(x) - 2 x F'(x)), x = r'^2 / (4 H^2)
        const double Ha = ha * rp, x = rp * rp / (4.0 * Ha * Ha);
        const double dK = (1.0 / SG_SQRT_PI) * rp / (2.0 * Ha * Ha * Ha * Ha) * sg_D64(x, wq);
        dind = rp * rp * SG_SQRT2 * dK * rp * (0.5 * N);
    }
    double part[2] = {0.0, 0.0};
    if (live) {
        for (int m = t; m < NC; m += T) {
            const double2 zm = pl.ld(m), zn = pl.ld((N - m) & (N - 1));
            double cr, cp;
            ssg_mode(lt, st, ((size_t)b * A.nr + ic) * ncol, ((size_t)a * A.nr + ip) * ncol, m, cr, cp);
            const double wm = ((m == 0 || m == nphi / 2) ? 1.0 : 2.0) * scale;
            double tr = 0.5 * (zm.x + zn.x), tp = 0.5 * (zn.x - zm.x);
            if (m == 1) {
                tr += dind;
                tp += dind;
            }
            part[0] += wm * (tr * cr + tp * cp);
            part[1] += wm * (0.5 * (zm.y + zn.y) * cr + 0.5 * (zn.y - zm.y) * cp);
        }
    }
    __syncthreads();
    // per-group sums, stored per row (part 0 belongs to dL/dh_a at the source
    // ring, part 1 to dL/dh_b at the target ring); k_ssg_finish adds them up
    for (int d = 0; d < 2; ++d) {
        red[threadIdx.x] = part[d];
        __syncthreads();
        for (int o = T / 2; o > 0; o >>= 1) {
            if (t < o) red[threadIdx.x] += red[threadIdx.x + o];
            __syncthreads();
        }
        if (t == 0 && live) rowpart[2 * ((((size_t)b * A.nf + a) * A.nr + ip) * A.nrt + i) + d] = red[threadIdx.x];
        __syncthreads();
    }
}

// dL/dH_f(r_k) = (1/r_k) dL/dh_f(r_k): the row partials that touch ring k of
// group f, in a fixed order (so the result is the same on every call).
// Row R = ((b nf + a) nr + i') nrt + i; ring k of group f is the source ring
// of rows (b, f, k, i) and the target ring of rows (f, a, i', k).
__global__ void __launch_bounds__(256) k_ssg_finish(const double *rowpart, SsRowArgs A, double *dH)
{
    __shared__ double red[256];
    const int f = blockIdx.x / A.nr, k = blockIdx.x % A.nr;
    const int n = A.nf * A.nr;
    double s = 0.0;
    for (int j = threadIdx.x; j < n; j += 256) {
        const int o = j / A.nr, x = j % A.nr;
        s += rowpart[2 * ((((size_t)o * A.nf + f) * A.nr + k) * A.nrt + x)];
        s += rowpart[2 * ((((size_t)f * A.nf + o) * A.nr + x) * A.nrt + k) + 1];
    }
    red[threadIdx.x] = s;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const double r = A.lin ? A.rmin + (k + 0.5) * A.dr : exp(A.lnrmin + (k + 0.5) * A.du);
        dH[blockIdx.x] = red[0] / r;
    }
}

struct SsGradWs {
    size_t lt, st, dself, rowpart, total;
};

static SsGradWs ssg_ws(int nr, int nphi, int nf)
{
    const size_t fs = sg_blk_field_elems(nphi, nr);
    const size_t rows = (size_t)nf * nf * nr * ((nr + 1) & ~1);
    SsGradWs w;
    w.lt = 0;
    w.st = sg_align256(sizeof(float2) * fs * 2 * nf);
    w.dself = w.st + sg_align256(sizeof(float2) * fs * nf);
    w.rowpart = w.dself + sg_align256(sizeof(double) * 2 * nf * nf * nr);
    w.total = w.rowpart + sg_align256(sizeof(double) * 2 * rows);
    return w;
}

size_t sg_ss_grad_ws_bytes(int nr, int nphi, int nf) { return ssg_ws(nr, nphi, nf).total; }

template <int N>
static void launch_ssg_phi(const SsRowArgs &A, const float *lam_r, const float *lam_p, const float *sigma,
                           const float2 *tw, float4 *lt, float2 *st, hipStream_t s)
{
    using S = SsRowShape<N>;
    const int jobs = A.nf * A.nr + A.nf * ((A.nr + 1) / 2);
    hipLaunchKernelGGL(k_ssg_phi<N>, dim3((jobs + S::G - 1) / S::G), dim3(S::WGS), 0, s, lam_r, lam_p, sigma, tw, lt,
                       st, A.nr, A.nf);
}

template <int N>
static void launch_ssg_rows(const double *H, const double *dself, const SsRowArgs &A, const SsPart &P, int nphi,
                            const float4 *lt, const float2 *st, double *rowpart, hipStream_t s)
{
    using S = SsRowShape<N>;
    SsClass C = P.C;
    if (P.kind == 0) {
        if (!C.on) {  // all ring pairs as one class
            C.on = 1;
            C.nt = (A.nr + SG_SS_TI - 1) / SG_SS_TI;
            C.K1 = 0;
            C.K2 = A.nr;
            C.nk = 2 * C.K2 - 1;
            C.x1 = 0.0;
            C.x2 = INFINITY;
        }
        if (!A.lin) C.half = 1;  // offsets k >= 0, the mirrors along
        if (C.half) C.nk = C.K2 - C.K1;
    }
    const size_t rows = C.on ? ss_class_rows(A, C) : (size_t)A.nf * A.nf * A.nr * A.nrt;
    const size_t chunk = (size_t)1 << 22;
    for (size_t r0 = 0; r0 < rows; r0 += chunk) {
        const int n = (int)std::min(chunk, rows - r0);
        const dim3 one((n + S::G - 1) / S::G), two((n / 2 + S::G - 1) / S::G);
        if (P.kind == 1 && sg_hat_long(A.du, A.dphi))
            hipLaunchKernelGGL((k_ssg_rows<N, 3>), one, dim3(S::WGS), 0, s, H, dself, A, C, nphi, lt, st, r0, n,
                               rowpart);
        else if (P.kind == 1)
            hipLaunchKernelGGL((k_ssg_rows<N, 1>), one, dim3(S::WGS), 0, s, H, dself, A, C, nphi, lt, st, r0, n,
                               rowpart);
        else if (P.kind == 2)
            hipLaunchKernelGGL((k_ssg_rows<N, 2>), one, dim3(S::WGS), 0, s, H, dself, A, C, nphi, lt, st, r0, n,
                               rowpart);
        else
            hipLaunchKernelGGL(k_ssg_pairs<N>, two, dim3(S::WGS), 0, s, H, dself, A, C, nphi, lt, st, r0, n, rowpart);
    }
}

sg_status sg_ss_grad_run(const sg_disc &d0, const double *d_H, const float *lam_r, const float *lam_p, double *dH,
                         void *d_ws, hipStream_t s)
{
    // species discs: the derivative of the group disc at the group sums
    // (placed after the gradient's own workspace)
    sg_disc d = d0;
    if (d0.n_species) {
        float *gsig = (float *)((char *)d_ws + sg_ss_grad_ws_bytes(d0.grid.n_r, d0.grid.n_phi, d0.fluids.n_fluids));
        const sg_status st = sg_species_group_sums(d0, gsig, s);
        if (st != SG_OK) return st;
        d.n_species = 0;
        d.sigma = gsig;
    }
    const sg_grid *grid = &d.grid;
    const int nr = grid->n_r, nphi = grid->n_phi, nf = d.fluids.n_fluids;
    const uint32_t flags = d.flags;
    const bool lin = (flags & SG_LINEAR_R) != 0;
    const SsLayout L = sg_ss_layout(nr, nphi, nf, sg_ss_du(*grid, flags), (flags & SG_SS_FULL) != 0);
    const float2 *tw = (const float2 *)((const char *)d.table + L.off_tw_phi);
    const SsGradWs W = ssg_ws(nr, nphi, nf);
    char *ws = (char *)d_ws;
    float4 *lt = (float4 *)(ws + W.lt);
    float2 *st = (float2 *)(ws + W.st);
    double *dself = (double *)(ws + W.dself), *rowpart = (double *)(ws + W.rowpart);
    const double dphi = 2.0 * SG_PI / nphi;
    SsRowArgs A;
    A.nr = nr;
    A.nrt = L.nrt;
    A.nf = nf;
    A.excl = (flags & SG_SELF_CELL_EXCLUDE) ? 1 : 0;
    A.ind = (flags & SG_INDIRECT) ? 1 : 0;
    A.pot = (flags & SG_POTENTIAL) ? 1 : 0;
    A.lin = lin ? 1 : 0;
    A.lnrmin = log(grid->r_min);
    A.du = log(grid->r_max / grid->r_min) / nr;
    A.dphi = dphi;
    A.rmin = grid->r_min;
    A.dr = (grid->r_max - grid->r_min) / nr;
    A.second = (flags & SG_SECOND_ORDER) ? 1 : 0;
    sg_gl_nodes(A.gl, A.du / dphi);
    if (!A.excl && !A.second) {  // second order: the own cell is one of the integrated samples
        GLNodes gl;
        sg_gl_nodes(gl, lin ? sg_lin_aspect(*grid, dphi) : A.du / dphi);
        for (int which = 1; which <= 2; ++which) {
            double *out = dself + (size_t)(which - 1) * nf * nf * nr;
            if (lin) {
                hipLaunchKernelGGL(k_ss_self_lin, dim3(nf * nf * nr), dim3(256), 0, s, d_H, nf, nr, 1, grid->r_min,
                                   A.dr, dphi, A.pot, which, out, gl);
            } else if (A.pot) {
                sg_pot_cells<double>(d_H, nullptr, nf, nr, 1, A.lnrmin, A.du, dphi, 0, out, which, s);
                SG_HIP(hipGetLastError());
                // as the forward's own-cell sample: -I / (du dphi)
                hipLaunchKernelGGL(k_ss_scale, dim3((nf * nf * nr + 255) / 256), dim3(256), 0, s, out, nf * nf * nr,
                                   -1.0 / (A.du * dphi));
            } else {
                hipLaunchKernelGGL(k_self_cell_ring, dim3(nf * nf * nr), dim3(256), 0, s, d_H, nf, nr, A.lnrmin,
                                   A.du, dphi, which, out, gl);
            }
            SG_HIP(hipGetLastError());
        }
    }
#define SG_SIZES(F) F(4) F(8) F(16) F(32) F(64) F(128) F(256) F(512) F(1024) F(2048)
    switch (nphi) {
#define SG_PHI(N) \
    case N: launch_ssg_phi<N>(A, lam_r, lam_p, d.sigma, tw, lt, st, s); break;
        SG_SIZES(SG_PHI)
#undef SG_PHI
    default: return SG_ERR_UNSUPPORTED;
    }
    for (const SsPart &P : ss_parts(A, nphi, (flags & SG_SS_FULL) != 0, SG_SS_ALIAS_GRAD)) {
        switch (P.M) {
#define SG_ROWS(N) \
    case N: launch_ssg_rows<N>(d_H, dself, A, P, nphi, lt, st, rowpart, s); break;
            SG_SIZES(SG_ROWS)
#undef SG_ROWS
        }
    }
#undef SG_SIZES
    SG_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_ssg_finish, dim3(nf * nr), dim3(256), 0, s, rowpart, A, dH);
    SG_HIP(hipGetLastError());
    return SG_OK;
}
