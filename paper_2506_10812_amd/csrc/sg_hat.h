// sg_hat.h -- quadrature of the second-order (hat-weighted) kernel weights,
// shared by the FFT path's table build and the semi-spectral operator rows.
#pragma once
#include "sg_kfn.h"
#include "sg_table.h"

// SG_SECOND_ORDER: the sources are the piecewise-bilinear interpolant of the
// cell values on the (u, phi) grid (tensor-product hat functions Lambda
// centred on the cell centres, periodic in phi), integrated exactly against
// the kernel, so the table holds, in place of the point samples and the
// own-cell average,
//   W_c(P, Q) = int int Lambda(s) Lambda(t) K_c((P + s) du, (Q + t) dphi) ds dt
// over s, t in [-1, 1] (Lambda(x) = 1 - |x|).  The support splits into four
// unit squares on which the weight is bilinear.  A square whose corner is
// the kernel's singular point (s, t) = (-P, -Q) (|P|, |Q| <= 1) is done in
// polar coordinates about that corner (the Duffy split and geometric panels
// of the self-cell rule); at (P, Q) = (0, 0) the four squares are folded
// into one with K_r symmetrised in X (the 1/rho part of K_r is odd in X and
// cancels only between the halves; K_phi, odd in phi, gives 0).  Elsewhere
// tensor Gauss-Legendre rules of 6 x 6 points on sub-squares small against
// their distance to the singular point (at most a third of it; where a long
// side starts beside the singular point, pieces that grow with the distance:
// sg_hat_long_node).
static __device__ __constant__ double sg_gl6_x[6] = {0.0337652428984239860, 0.1693953067668677431,
                                                     0.3806904069584015457, 0.6193095930415984543,
                                                     0.8306046932331322569, 0.9662347571015760140};
static __device__ __constant__ double sg_gl6_w[6] = {0.0856622461895851725, 0.1803807865240693038,
                                                     0.2339569672863455237, 0.2339569672863455237,
                                                     0.1803807865240693038, 0.0856622461895851725};

__device__ inline double sg_hat(double x) { return fmax(0.0, 1.0 - fabs(x)); }

// A side of length len that starts beside the singular point, at the distance d
// across: pieces uniform in v, the distance along it being d sinh v.  The
// kernel's singularities lie at v = +-i pi/2, so pieces of 1/2 in v take 6 points
// to 1e-13, where uniform ones of a third of the distance would number 3 len / d.
// (Held at 32 of those, fields on cells 276 and 1103 times longer than wide were
// 2e-5 and 4e-4 off.)  From the place u in [0, 1] in v: the place along the side
// from its start, in units of len, the weight's factor in w.
#define SG_HAT_PIECES 32
__device__ inline double sg_hat_long_node(double len, double d, double u, double &w)
{
    const double q = d / len, V = asinh(len / d), e = sinh(u * V);
    w *= q * V * sqrt(1.0 + e * e);
    return q * e;
}

// Tensor Gauss-Legendre over pieces k in [k0, k1) (step dk) of the unit square
// [ds, ds + 1] x [dt, dt + 1] of entry (P, Q), cut into |ms| x |mt| sub-squares;
// a negative count is that of a long side's pieces (sg_hat_split).  LONG: such
// sides come up (sg_hat_long).  The semi-spectral rows, which hold the rule next
// to a transform, have a kernel for either: the node of a long side, inlined for
// all, took them from 3.0 to 3.7 ms (200 x 256).
template <bool LONG>
__device__ inline void sg_hat_square(int P, int Q, int ds, int dt, int ms, int mt, int k0, int k1, int dk,
                                     double du, double dphi, double ha, double hb, int which, const double *wq,
                                     double &wr, double &wp)
{
    const bool ls = LONG && ms < 0, lt = LONG && mt < 0;  // not both: each has the other's distance
    if constexpr (LONG) {
        ms = abs(ms);
        mt = abs(mt);
    }
    for (int k = k0; k < k1; k += dk) {
        const int piece = k / 36, node = k % 36;
        const int is = piece % ms, it = piece / ms;
        const int a = node % 6, b = node / 6;
        double s = ds + (is + sg_gl6_x[a]) / ms, t = dt + (it + sg_gl6_x[b]) / mt;
        double w = sg_gl6_w[a] * sg_gl6_w[b] / (ms * mt);
        if (LONG && (ls || lt)) {
            // the distance across, and the end (-P or -Q) the side starts from
            if (ls) {
                const double u = sg_hat_long_node(du, (Q + dt >= 0 ? Q + dt : -(Q + dt + 1)) * dphi, s - ds, w);
                s = ds == -P ? ds + u : ds + 1 - u;
            } else {
                const double u = sg_hat_long_node(dphi, (P + ds >= 0 ? P + ds : -(P + ds + 1)) * du, t - dt, w);
                t = dt == -Q ? dt + u : dt + 1 - u;
            }
        }
        w = w * sg_hat(s) * sg_hat(t);
        const double X = (P + s) * du, ph = (Q + t) * dphi;
        double kr, kp;
        sg_conv_kernel64(X, sin(0.5 * ph), sin(ph), ha, hb, which, wq, kr, kp);
        wr += w * kr;
        wp += w * kp;
    }
}

// Whether cells of these sides have squares with long sides.
__host__ __device__ inline bool sg_hat_long(double du, double dphi)
{
    return 3.0 * fmax(du, dphi) > SG_HAT_PIECES * fmin(du, dphi);
}

// Sub-square count per side: pieces at most a third of their distance to the
// singular point (physical units); more than 32 only where the side starts
// beside it, which then counts its pieces in v, negative.
template <bool LONG>
__device__ inline void sg_hat_split(int P, int Q, int ds, int dt, double du, double dphi, int &ms, int &mt)
{
    const double x0 = (P + ds) * du, x1 = x0 + du, y0 = (Q + dt) * dphi, y1 = y0 + dphi;
    const double dx = x0 > 0.0 ? x0 : (x1 < 0.0 ? -x1 : 0.0);
    const double dy = y0 > 0.0 ? y0 : (y1 < 0.0 ? -y1 : 0.0);
    const double d = sqrt(dx * dx + dy * dy);
    const double ws = ceil(3.0 * du / d), wt = ceil(3.0 * dphi / d);
    ms = max(1, (int)ws);
    mt = max(1, (int)wt);
    if (LONG && ws > SG_HAT_PIECES) ms = -(int)ceil(2.0 * asinh(du / d));
    if (LONG && wt > SG_HAT_PIECES) mt = -(int)ceil(2.0 * asinh(dphi / d));
}

__device__ inline bool sg_hat_singular(int P, int Q, int ds, int dt)
{
    return (-P == ds || -P == ds + 1) && (-Q == dt || -Q == dt + 1);
}

// Polar rule on the unit square [ds, ds + 1] x [dt, dt + 1] whose corner is
// the singular point: (X, phi) = (sx du x, sy dphi y) with (x, y) in [0, 1]^2
// measured from the corner, cut along its diagonal, each triangle mapped to
// the unit square with the corner collapsed (x = xi, y = xi eta and
// x = xi eta, y = xi; Jacobian xi).  sym: K_r symmetrised in X (entry (0, 0)).
// Nodes k0, k0 + dk, ... of the rule (a block's threads, or one thread).
__device__ inline void sg_hat_corner(int P, int Q, int sx, int sy, bool sym, double du, double dphi, double ha,
                                     double hb, int which, const GLNodes &gl, const double *wq, int k0, int dk,
                                     double &wr, double &wp)
{
    const int nx = sg_own_nx(du, dphi, fmin(ha, hb)), n = nx * gl.ne;
    const OwnEta e0(du, dphi), e1(dphi, du);
    for (int idx = k0; idx < n; idx += dk) {
        double xi, s, wn;
        sg_own_node(gl, nx, idx, xi, s, wn);
        for (int tri = 0; tri < 2; ++tri) {
            double wgt = wn;
            const double eta = (tri == 0 ? e0 : e1).at(s, wgt);
            const double x = tri == 0 ? xi : xi * eta, y = tri == 0 ? xi * eta : xi;
            const double X = sx * x * du, ph = sy * y * dphi;
            // hats from the corner: 1 - x at a corner s = 0, x at s = +-1
            // (not 1 - |-1 + x|, which loses the digits of a small x)
            const double w = wgt * (P == 0 ? 1.0 - x : x) * (Q == 0 ? 1.0 - y : y);
            if (sym) {
                wr += w * sg_sym_kr64(X, ph, ha, hb, which, wq);
            } else {
                double kr, kp;
                sg_conv_kernel64(X, sin(0.5 * ph), sin(ph), ha, hb, which, wq, kr, kp);
                wr += w * kr;
                wp += w * kp;
            }
        }
    }
}

// Part of W_c(P, Q) (or an h derivative, which): the quadrature nodes
// k0, k0 + dk, ... of every piece (the polar rules at the singular corner for
// |P|, |Q| <= 1, split tensor squares elsewhere, as the table build's kernels
// apply them); the sum of the parts over k0 = 0 .. dk - 1 is the weight.
template <bool LONG>
__device__ inline void sg_hat_weight_part(int P, int Q, double du, double dphi, double ha, double hb, int which,
                                          const GLNodes &gl, const double *wq, int k0, int dk, double &wr,
                                          double &wp)
{
    wr = 0.0;
    wp = 0.0;
    if (P == 0 && Q == 0) {
        double r = 0.0, t = 0.0;
        sg_hat_corner(0, 0, 1, 1, true, du, dphi, ha, hb, which, gl, wq, k0, dk, r, t);
        wr = 4.0 * r;
        return;
    }
    const bool near = abs(P) <= 1 && abs(Q) <= 1;
    for (int ds = -1; ds <= 0; ++ds)
        for (int dt = -1; dt <= 0; ++dt) {
            if (near && sg_hat_singular(P, Q, ds, dt)) {
                const int sx = (ds == -P) ? 1 : -1, sy = (dt == -Q) ? 1 : -1;
                sg_hat_corner(P, Q, sx, sy, false, du, dphi, ha, hb, which, gl, wq, k0, dk, wr, wp);
            } else {
                int ms, mt;
                sg_hat_split<LONG>(P, Q, ds, dt, du, dphi, ms, mt);
                sg_hat_square<LONG>(P, Q, ds, dt, ms, mt, k0, 36 * abs(ms * mt), dk, du, dphi, ha, hb, which, wq, wr, wp);
            }
        }
}
