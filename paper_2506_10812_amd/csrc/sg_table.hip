// sg_table.hip -- one-off, double-precision construction of the kernel
// spectra for the log-polar FFT path (sg_kernel_table), the self-cell
// quadrature, and device evaluation of F for tests.
//
// App. C: with H_f = h_f r the radial and azimuthal fields are convolutions
// in (u = ln r, phi) with offset-only kernels K_r(X, phi), K_phi(X, phi);
// Sect. 5.2: zero padding of the radial axis to 2 n_r makes the periodic
// convolution equal the aperiodic one, and the kernel is computed once.
// Steps (all double precision):
//   1. rows X = p du (p in (-n_r, n_r), stored at p mod 2 n_r; row n_r is
//      zero): samples K_r + i K_phi at phi = q dphi, q <= n_phi/2, mirrored
//      (K_r even, K_phi odd), and their phi transform, which is real: T_r(m)
//      and t_phi(m), K_phi's being i t_phi.  Two rows share one transform, and
//      a row takes only as many azimuths as it resolves (its modes fall off
//      as e^{-m|X|}; see SG_SS_ALIAS in sg_semispec.h).  SG_SECOND_ORDER:
//      every sample is the hat-weighted integral of the kernel instead;
//   2. u transform (length 2 n_r) of each column m of T_r + i t_phi (both
//      real), split into K_r and K_phi; the own-cell average (offset (0,0), a
//      flat spectrum in phi) joins T_r at p = 0 here; keep k_u <= n_r (K_r is
//      Hermitian and K_phi anti-Hermitian in k_u because K_r is even and K_phi
//      odd in phi), scale by -du dphi/(2 n_r n_phi), round to float.
// Four launches for up to SG_TAB_ITEMS pairs: own-cell integrals and twiddles
// (9 to 11 us), rows (16 us), columns (35 us), header (5 us) on the two-fluid
// 1024 x 2048 disc, bound by the columns' FP64 transforms; one sampling, one phi
// and two u launches per pair on the full grid took 700 us.
#include <algorithm>
#include <vector>

#include "sg_fft.h"
#include "sg_kfn.h"
#include "sg_semispec.h"
#include "sg_table.h"
#include "sg_hat.h"

// ------------------------------------------------------------------ twiddles
__global__ void k_twiddles(float2 *tw_phi, int nphi)
{
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < nphi) {
        double s, c;
        sincospi(-2.0 * i / nphi, &s, &c);
        tw_phi[i] = make_float2((float)c, (float)s);
    }
}

// --------------------------------------------------------------- self cell
// Kbar = (1/(du dphi)) PV-int over the own cell of K_r.  By symmetry
// (K_r even in phi; its 1/rho singularity odd in X) it is (1/(a b)) times the
// integral of S = (K_r(X,phi) + K_r(-X,phi))/2 over [0,a]x[0,b], a = du/2,
// b = dphi/2.  The quarter cell is cut along its diagonal; each triangle is
// mapped to the unit square with the singular corner collapsed
// (X = a xi, phi = b xi eta and X = a xi eta, phi = b xi; Jacobian a b xi),
// which turns the direction-dependent limit at the corner into a smooth
// integrand.  The rules in xi and eta are those of sg_own_node.
//
// An OwnPt holds what one node contributes independently of the scale
// heights: with h^2(X) = h0 cosh X + g sinh X, h0 = (h_a^2 + h_b^2)/2,
// g = (h_b^2 - h_a^2)/2, and x = c / (4 h^2(X)),
//   S w = gp F(x) h^-3 |_X + gm F(x) h^-3 |_-X   (1/(8 sqrt(pi)) left out),
// gp, gm = (w/2) e^{-+3X/2} (e^{+-X} - cos phi); gs = gp + gm without their
// cancellation, for h_a = h_b, where both sides share one F.  The pair
// (b, a) swaps the two F of (a, b), so each unordered pair costs two F.
struct OwnPt {
    double c, ch, sh, gp, gm, gs;
};

__device__ inline OwnPt own_pt(double X, double phi, double w)
{
    const double s = sinh(0.5 * X), co = sqrt(1.0 + s * s), sp = sin(0.5 * phi);
    const double ep = co + s, em = co - s;  // e^{X/2}, e^{-X/2}
    const double p2 = 2.0 * sp * sp;        // 1 - cos phi
    OwnPt q;
    q.c = 2.0 * s * s + p2;
    q.ch = 1.0 + 2.0 * s * s;
    q.sh = 2.0 * s * co;
    q.gp = 0.5 * w * (2.0 * s * em * em + p2 * em * em * em);
    q.gm = 0.5 * w * (-2.0 * s * ep * ep + p2 * ep * ep * ep);
    q.gs = 0.5 * w * (-4.0 * s * q.sh + p2 * (ep * ep * ep + em * em * em));
    return q;
}

// Node of triangle tri (0: X = a xi, phi = b xi eta; 1: X = a xi eta, phi = b xi).
__device__ inline OwnPt own_tri_pt(double a, double b, const OwnEta &e, int tri, double xi, double s, double w)
{
    const double eta = e.at(s, w);
    return tri == 0 ? own_pt(a * xi, b * xi * eta, w) : own_pt(a * xi * eta, b * xi, w);
}

// F(x) h^-3, x = c / (4 h^2)
__device__ inline double own_val(double c, double h2, const double *wq)
{
    const double rs = rsqrt(h2), r2 = rs * rs;
    return sg_F64(0.25 * c * r2, wq) * (r2 * rs);
}

// D(x) h^-5
__device__ inline double own_dval(double c, double h2, const double *wq)
{
    const double rs = rsqrt(h2), r2 = rs * rs;
    return sg_D64(0.25 * c * r2, wq) * (r2 * r2 * rs);
}

// One node of the h derivative (which = 1: h_a, 2: h_b) of one pair:
// dK/dh = dK/d(h^2) d(h^2)/dh, d(h^2(X))/dh_a = h_a e^{-X}, /dh_b = h_b e^X.
__device__ inline double own_dnode(const OwnPt &q, double ha, double hb, int which, const double *wq)
{
    const double h0 = 0.5 * (ha * ha + hb * hb), g = 0.5 * (hb * hb - ha * ha);
    const double eX = q.ch + q.sh, emX = q.ch - q.sh;
    const double vp = own_dval(q.c, h0 * q.ch + g * q.sh, wq), vm = own_dval(q.c, h0 * q.ch - g * q.sh, wq);
    return which == 1 ? ha * (q.gp * vp * emX + q.gm * vm * eX) : hb * (q.gp * vp * eX + q.gm * vm * emX);
}

__device__ inline double block_sum256(double v, double *red)
{
    red[threadIdx.x] = v;
    __syncthreads();
    for (int s = blockDim.x / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    return red[0];
}

#define SG_OWN_SCALE (1.0 / (8.0 * SG_SQRT_PI))

// Nodes k0, k0 + dk, ... of one item (pair h_a, h_b; which as above).
__device__ inline double self_cell_partial(double ha, double hb, int which, double a, double b,
                                           const GLNodes &gl, const double *wq, int k0, int dk)
{
    const int nx = sg_own_nx(a, b, fmin(ha, hb)), n = nx * gl.ne;
    const double h0 = 0.5 * (ha * ha + hb * hb), g = 0.5 * (hb * hb - ha * ha);
    const OwnEta e0(a, b), e1(b, a);
    double acc = 0.0;
#pragma unroll 1
    for (int idx = k0; idx < 2 * n; idx += dk) {
        double xi, s, w;
        const int tri = idx >= n ? 1 : 0;
        sg_own_node(gl, nx, idx - tri * n, xi, s, w);
        {
            const OwnPt q = own_tri_pt(a, b, tri == 0 ? e0 : e1, tri, xi, s, w);
            if (which)
                acc += own_dnode(q, ha, hb, which, wq);
            else if (g == 0.0)
                acc += q.gs * own_val(q.c, h0 * q.ch, wq);
            else
                acc += q.gp * own_val(q.c, h0 * q.ch + g * q.sh, wq) + q.gm * own_val(q.c, h0 * q.ch - g * q.sh, wq);
        }
    }
    return acc * SG_OWN_SCALE;
}

__global__ void __launch_bounds__(256) k_self_cell(SelfItems items, double *out, double du, double dphi, GLNodes gl)
{
    __shared__ __attribute__((aligned(16))) double wq[FQuad<double>::TABLE];
    __shared__ double red[256];
    const int it = blockIdx.x;
    sg_fill64(wq, items.which[it] ? SG_FN_D : SG_FN_F);
    __syncthreads();
    const double acc = self_cell_partial(items.ha[it], items.hb[it], items.which[it], 0.5 * du,
                                         0.5 * dphi, gl, wq, threadIdx.x, 256);
    const double tot = block_sum256(acc, red);
    if (threadIdx.x == 0) out[it] = tot;
}

// Sum of each of the n per-thread values over the block, value k to out(k);
// red: one double per wave and value.
template <int n, typename Out> __device__ inline void own_block_sums(double (&v)[n], double *red, Out out)
{
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < n; ++k) {
        double x = v[k];
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
        if (lane == 0) red[k * 4 + wv] = x;
    }
    __syncthreads();
    if ((int)threadIdx.x < n) {
        const double *r = red + 4 * threadIdx.x;
        out((int)threadIdx.x, (r[0] + r[1]) + (r[2] + r[3]));
    }
    __syncthreads();
}

// Per-cell variant (the direct path with general H, and per ring with nphi =
// 1): h_f = H_f[i]/r_i from the caller's arrays, all pairs of CPB cells per
// block.  FP64 VALU bound: a node's geometry (a sinh, a sine, two square
// roots) depends on the grid only and is formed once for the CPB cells, whose
// heights are wave-uniform; the two-fluid case takes 4 F per node and
// triangle for its four pairs.  Two fluids, 101 x 250 cells: 0.80 ms (1.43 with
// a Chebyshev series for F), against 30.9 ms with 112 x 48 nodes, one (cell,
// pair) per block and the kernel evaluated whole at +-X.
template <typename T, int NF, int CPB>
__global__ void __launch_bounds__(256)
k_self_cells(const T *H, int64_t N, int nphi, double lnrmin, double du, double dphi, double *out, GLNodes gl)
{
    __shared__ __attribute__((aligned(16))) double wq[FQuad<double>::TABLE];
    __shared__ double red[4 * NF * NF * CPB];
    sg_fill64(wq, SG_FN_F);
    __syncthreads();
    const int64_t c0 = (int64_t)blockIdx.x * CPB;
    double h2[CPB][NF], hm = INFINITY;  // h_f^2 of each cell (past the last: the last cell's)
#pragma unroll
    for (int c = 0; c < CPB; ++c) {
        const int64_t cell = c0 + c < N ? c0 + c : N - 1;
        const double r = exp(lnrmin + ((int)(cell / nphi) + 0.5) * du);
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            const double h = (double)H[f * N + cell] / r;
            h2[c][f] = h * h;
            hm = fmin(hm, h);
        }
    }
    const double a = 0.5 * du, b = 0.5 * dphi;
    const int nx = sg_own_nx(a, b, hm), n = nx * gl.ne;
    double acc[CPB * NF * NF];
#pragma unroll
    for (int k = 0; k < CPB * NF * NF; ++k) acc[k] = 0.0;
    const OwnEta e0(a, b), e1(b, a);
    for (int idx = threadIdx.x; idx < n; idx += 256) {
        double xi, s, w;
        sg_own_node(gl, nx, idx, xi, s, w);
#pragma unroll 1
        for (int tri = 0; tri < 2; ++tri) {
            const OwnPt q = own_tri_pt(a, b, tri == 0 ? e0 : e1, tri, xi, s, w);
#pragma unroll
            for (int c = 0; c < CPB; ++c)
#pragma unroll
                for (int fa = 0; fa < NF; ++fa) {
                    acc[(c * NF + fa) * NF + fa] += q.gs * own_val(q.c, h2[c][fa] * q.ch, wq);
#pragma unroll
                    for (int fb = fa + 1; fb < NF; ++fb) {
                        const double h0 = 0.5 * (h2[c][fa] + h2[c][fb]), g = 0.5 * (h2[c][fb] - h2[c][fa]);
                        const double vp = own_val(q.c, h0 * q.ch + g * q.sh, wq);
                        const double vm = own_val(q.c, h0 * q.ch - g * q.sh, wq);
                        acc[(c * NF + fa) * NF + fb] += q.gp * vp + q.gm * vm;
                        acc[(c * NF + fb) * NF + fa] += q.gp * vm + q.gm * vp;
                    }
                }
        }
    }
    own_block_sums(acc, red, [&](int k, double v) {
        const int c = k / (NF * NF), pair = k % (NF * NF);
        if (c0 + c < N) out[(int64_t)pair * N + c0 + c] = v * SG_OWN_SCALE;
    });
}

// Cells per block: as many as keep the accumulators (one per cell and pair)
// in registers, but fewer where that would leave the GPU idle.
template <typename T>
void sg_self_cells(const T *H, int nf, int nr, int nphi, double lnrmin, double du, double dphi, double *out,
                   hipStream_t s)
{
    const int64_t N = (int64_t)nr * nphi;
    GLNodes gl;
    sg_gl_nodes(gl, du / dphi);
#define SG_OWN(NF, CPB)                                                                                     \
    hipLaunchKernelGGL((k_self_cells<T, NF, CPB>), dim3((unsigned)((N + CPB - 1) / CPB)), dim3(256), 0, s, H, N, \
                       nphi, lnrmin, du, dphi, out, gl)
    const bool many = N >= 4096;
    switch (nf) {
    case 1:
        if (many) SG_OWN(1, 8);
        else SG_OWN(1, 1);
        break;
    case 2:
        if (many) SG_OWN(2, 2);
        else SG_OWN(2, 1);
        break;
    case 3: SG_OWN(3, 1); break;
    default: SG_OWN(4, 1); break;
    }
#undef SG_OWN
}
template void sg_self_cells<float>(const float *, int, int, int, double, double, double, double *, hipStream_t);
template void sg_self_cells<double>(const double *, int, int, int, double, double, double, double *, hipStream_t);

// Per-ring variant with a derivative selector for the semi-spectral
// gradient: item = (pair, ring), h = H[f][ring] / r; which = 1: dKbar/dh_a,
// 2: dKbar/dh_b.
__global__ void __launch_bounds__(256)
k_self_cell_ring(const double *H, int nf, int nr, double lnrmin, double du, double dphi, int which,
                                 double *out, GLNodes gl)
{
    __shared__ __attribute__((aligned(16))) double wq[FQuad<double>::TABLE];
    __shared__ double red[256];
    sg_fill64(wq, which ? SG_FN_D : SG_FN_F);
    __syncthreads();
    const int item = blockIdx.x;
    if (item >= nf * nf * nr) return;
    const int pair = item / nr, ir = item % nr;
    const int fa = pair / nf, fb = pair % nf;
    const double r = exp(lnrmin + (ir + 0.5) * du);
    const double acc = self_cell_partial(H[fa * nr + ir] / r, H[fb * nr + ir] / r, which, 0.5 * du, 0.5 * dphi, gl, wq,
                                         threadIdx.x, 256);
    const double tot = block_sum256(acc, red);
    if (threadIdx.x == 0) out[item] = tot;
}

// Own-cell integral of the potential kernel (reading: the paper does not
// treat k = i): int P_ab(|x_i - x'|) dA' over the cell, x' = r e^X (cos phi,
// sin phi) relative to the centre direction, |x_i - x'|^2 = r^2 e^X
// (4 sinh^2(X/2) + 4 sin^2(phi/2)), dA' = r^2 e^{2X} dX dphi; even in phi,
// so 2 x (X >= 0 and X <= 0 halves) over [0,a]x[0,b] with the same Duffy
// rule as the force self term (the singularity is logarithmic).
// which = 0: P; which = 1: dP/dH_ab (H_ab the r.m.s. height: with
// G0 = e^y K0(y), dG0/dy = -F(y), so dP/dH = -E(y) / (2 sqrt(pi) H^2), E(y) =
// 2 y F(y) - G0(y); like P, logarithmic at s -> 0).
//
// One block per CPB cells and unordered pair (P_ab = P_ba), or rows when
// per_row (H_f = h_f r: depends on the row only); a node's geometry is shared
// by the CPB cells (96 x 200 cells in double: 0.26 ms, against 5.0 ms with
// 112 x 48 nodes and one cell per block).  which = 1, 2 of the item: the integral's derivative with
// respect to h_a = H_a / r, h_b = H_b / r (dH_ab/dh_a = H_a r / (2 H_ab),
// likewise for b) instead.
template <typename T, int CPB, bool DER>
__global__ void __launch_bounds__(256)
k_pot_cells(const T *H, const double *h, int nf, int64_t per, int nphi, double lnrmin, double du, double dphi,
            int per_row, double *out, GLNodes gl, int which)
{
    __shared__ __attribute__((aligned(16))) double wq[FQuad<double>::TABLE];
    __shared__ double red[4 * CPB];
    sg_fill64(wq, DER ? SG_FN_E : SG_FN_G0);
    __syncthreads();
    int fa = 0, fb = blockIdx.y;  // unordered pair blockIdx.y of (0,0), (0,1), ..., (1,1), ...
    while (fb >= nf - fa) {
        fb -= nf - fa;
        ++fa;
    }
    fb += fa;
    const int64_t c0 = (int64_t)blockIdx.x * CPB;
    double r2H[CPB], hm = INFINITY;  // r^2 / (4 H_ab^2) of each cell
    auto heights = [&](int64_t c, double &r, double &Ha, double &Hb) {
        r = exp(lnrmin + ((per_row ? (int)c : (int)(c / nphi)) + 0.5) * du);
        Ha = per_row ? h[fa] * r : (double)H[fa * per + c];
        Hb = per_row ? h[fb] * r : (double)H[fb * per + c];
    };
#pragma unroll
    for (int c = 0; c < CPB; ++c) {
        double r, Ha, Hb;
        heights(c0 + c < per ? c0 + c : per - 1, r, Ha, Hb);
        const double Hab2 = 0.5 * (Ha * Ha + Hb * Hb);
        r2H[c] = r * r / (4.0 * Hab2);
        hm = fmin(hm, sqrt(Hab2) / r);
    }
    const double a = 0.5 * du, b = 0.5 * dphi;
    const int nx = sg_own_nx(a, b, hm), n = nx * gl.ne;
    double acc[CPB];
#pragma unroll
    for (int c = 0; c < CPB; ++c) acc[c] = 0.0;
    const OwnEta e0(a, b), e1(b, a);
    for (int idx = threadIdx.x; idx < n; idx += 256) {
        double xi, sn, w;
        sg_own_node(gl, nx, idx, xi, sn, w);
#pragma unroll 1
        for (int k = 0; k < 4; ++k) {
            double wk = w;
            const double eta = (k & 2 ? e1 : e0).at(sn, wk);
            const double X = (k & 1 ? -a : a) * (k & 2 ? xi * eta : xi), phi = k & 2 ? b * xi : b * xi * eta;
            const double s = sinh(0.5 * X), sp = sin(0.5 * phi), ex = sqrt(1.0 + s * s) + s;
            const double eX = ex * ex, cy = eX * (2.0 * s * s + 2.0 * sp * sp), we = wk * eX * eX;
#pragma unroll
            for (int c = 0; c < CPB; ++c) {
                const double y = cy * r2H[c];
                acc[c] += we * (DER ? sg_E64(y, wq) : sg_G0_64(y, wq));
            }
        }
    }
    own_block_sums(acc, red, [&](int c, double v) {
        if (c0 + c >= per) return;
        double r, Ha, Hb;
        heights(c0 + c, r, Ha, Hb);
        const double Hab = sqrt(0.5 * (Ha * Ha + Hb * Hb));
        v *= -2.0 * a * b * r * r / (2.0 * SG_SQRT_PI * Hab);
        const int64_t ab = (int64_t)(fa * nf + fb) * per + c0 + c, ba = (int64_t)(fb * nf + fa) * per + c0 + c;
        if constexpr (DER) {
            v *= r / (2.0 * Hab * Hab);
            out[ab] = v * (which == 1 ? Ha : Hb);
            out[ba] = v * (which == 1 ? Hb : Ha);
        } else {
            out[ab] = v;
            out[ba] = v;
        }
    });
}

template <typename T>
void sg_pot_cells(const T *H, const double *h, int nf, int nr, int nphi, double lnrmin, double du, double dphi,
                  int per_row, double *out, int which, hipStream_t s)
{
    const int64_t per = per_row ? nr : (int64_t)nr * nphi;
    GLNodes gl;
    sg_gl_nodes(gl, du / dphi);
    const unsigned pairs = (unsigned)(nf * (nf + 1) / 2);
#define SG_POT(CPB, DER)                                                                                         \
    hipLaunchKernelGGL((k_pot_cells<T, CPB, DER>), dim3((unsigned)((per + CPB - 1) / CPB), pairs), dim3(256), 0, s, \
                       H, h, nf, per, nphi, lnrmin, du, dphi, per_row, out, gl, which)
    if (which)
        SG_POT(1, true);
    else if (per >= 4096)
        SG_POT(8, false);
    else
        SG_POT(1, false);
#undef SG_POT
}
template void sg_pot_cells<float>(const float *, const double *, int, int, int, double, double, double, int, double *,
                                  int, hipStream_t);
template void sg_pot_cells<double>(const double *, const double *, int, int, int, double, double, double, int,
                                   double *, int, hipStream_t);

__global__ void k_fill_f64(double *p, int64_t n, double v)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

// ------------------------------------------- second-order (hat) weights
// (the rules themselves are in sg_hat.h)
// One thread per entry of the wrapped offset grid: entries with
// |P| >= 2 or |Q| >= 2 (no singular square); row n_r (offset +-n_r) is zero.
// which: 0 the weights, 1 and 2 their derivatives in h_a and h_b (the
// kernel's derivatives integrated with the same rules).
__global__ void __launch_bounds__(256) k_sample_hat_far(double2 *A, int nr, int nphi, double du, double ha, double hb, int which)
{
    __shared__ __attribute__((aligned(16))) double wq[FQuad<double>::TABLE];
    sg_fill64(wq, which ? SG_FN_D : SG_FN_F);
    __syncthreads();
    const int p = blockIdx.y;
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= nphi) return;
    const int P = p < nr ? p : p - 2 * nr, Q = 2 * q <= nphi ? q : q - nphi;
    if (p == nr) {
        A[(size_t)p * nphi + q] = make_double2(0.0, 0.0);
        return;
    }
    if (abs(P) <= 1 && abs(Q) <= 1) return;  // k_sample_hat_near
    const double dphi = 2.0 * SG_PI / nphi;
    double wr = 0.0, wp = 0.0;
    for (int ds = -1; ds <= 0; ++ds)
        for (int dt = -1; dt <= 0; ++dt) {
            int ms, mt;
            sg_hat_split<true>(P, Q, ds, dt, du, dphi, ms, mt);
            sg_hat_square<true>(P, Q, ds, dt, ms, mt, 0, 36 * abs(ms * mt), 1, du, dphi, ha, hb, which, wq, wr, wp);
        }
    A[(size_t)p * nphi + q] = make_double2(wr, wp);
}

// One 256-thread block per entry with |P|, |Q| <= 1 (nine entries).
__global__ void __launch_bounds__(256) k_sample_hat_near(double2 *A, int nr, int nphi, double du, double ha,
                                                          double hb, int which, GLNodes gl)
{
    __shared__ __attribute__((aligned(16))) double wq[FQuad<double>::TABLE];
    __shared__ double red[256];
    sg_fill64(wq, which ? SG_FN_D : SG_FN_F);
    __syncthreads();
    const int P = (int)(blockIdx.x % 3) - 1, Q = (int)(blockIdx.x / 3) - 1;
    const double dphi = 2.0 * SG_PI / nphi;
    double wr = 0.0, wp = 0.0;
    if (P == 0 && Q == 0) {
        // four squares with the singular corner; folded: 2 x 2 x [0,1]^2 with
        // K_r symmetrised in X and even in phi (K_phi contributes 0)
        double r = 0.0, t = 0.0;
        sg_hat_corner(0, 0, 1, 1, true, du, dphi, ha, hb, which, gl, wq, threadIdx.x, blockDim.x, r, t);
        wr = 4.0 * r;
    } else {
        for (int ds = -1; ds <= 0; ++ds)
            for (int dt = -1; dt <= 0; ++dt) {
                if (sg_hat_singular(P, Q, ds, dt)) {
                    // orientation of the square seen from the corner (-P, -Q)
                    const int sx = (ds == -P) ? 1 : -1, sy = (dt == -Q) ? 1 : -1;
                    sg_hat_corner(P, Q, sx, sy, false, du, dphi, ha, hb, which, gl, wq, threadIdx.x, blockDim.x,
                                  wr, wp);
                } else {
                    int ms, mt;
                    sg_hat_split<true>(P, Q, ds, dt, du, dphi, ms, mt);
                    sg_hat_square<true>(P, Q, ds, dt, ms, mt, threadIdx.x, 36 * abs(ms * mt), blockDim.x, du, dphi, ha, hb,
                                  which, wq, wr, wp);
                }
            }
    }
    const double tr = block_sum256(wr, red);
    __syncthreads();
    const double tp = block_sum256(wp, red);
    if (threadIdx.x == 0) {
        const int p = P < 0 ? P + 2 * nr : P, q = Q < 0 ? Q + nphi : Q;
        A[(size_t)p * nphi + q] = make_double2(tr, tp);
    }
}

// The own-cell value of a second-order table is W_r(0, 0).
__global__ void k_copy_w00(const double2 *A, double *out)
{
    out[0] = A[0].x;
    for (int k = 1; k < SG_SELF_PARTS; ++k) out[k] = 0.0;
}

// ------------------------------------------------------------ build kernels
// One table item: the kernel of a pair (which = 0) or its derivative in h_a or
// h_b (which = 1, 2), where its spectra go and their strides.
struct TabItem {
    double ha, hb;
    float2 *dst;         // [m][...] first column, component r
    uint32_t cs, comp;   // float2 per column; from component r to phi
    int which;
};
#define SG_TAB_ITEMS 8   // items per launch
struct TabArgs {
    int nr, nphi, nit;
    double du, dphi, scale;
    int ncls, M[5], K1[5], K2[5], blk0[6];  // row classes (as SsClass on the log grid)
    const double *self;  // [item][SG_SELF_PARTS], null: no own-cell term to add
    double2 *B;          // [item][n_phi/2 columns in tiles of 4][2 n_r]
    const double2 *A;    // second order: samples [2 n_r][n_phi] of the one item
    TabItem it[SG_TAB_ITEMS];
};

// B: column m < n_phi/2, offset row p.  Column 0 holds (T_r(0), T_r(n_phi/2)):
// t_phi is zero in both.  Tiles of 4 columns make 64 contiguous bytes per row.
__device__ __host__ inline size_t tab_index(int m, int p, int nu) { return ((size_t)(m >> 2) * nu + p) * 4 + (m & 3); }
static size_t tab_item_elems(int nr, int nphi) { return (size_t)((nphi / 2 + 3) / 4 * 4) * 2 * nr; }

// SG_SELF_PARTS blocks per own-cell item (the nodes are few: one or two per
// thread) and, beyond them, the float twiddle tables.
__global__ void __launch_bounds__(256)
k_tab_pre(SelfItems items, int nself, double *out, double du, double dphi, GLNodes gl, float2 *tw_u, int nu,
          float2 *tw_phi, int nphi)
{
    __shared__ __attribute__((aligned(16))) double wq[FQuad<double>::TABLE];
    __shared__ double red[256];
    const int nb = nself * SG_SELF_PARTS;
    if ((int)blockIdx.x < nb) {
        const int it = blockIdx.x / SG_SELF_PARTS, part = blockIdx.x % SG_SELF_PARTS;
        sg_fill64(wq, items.which[it] ? SG_FN_D : SG_FN_F);
        __syncthreads();
        const double acc = self_cell_partial(items.ha[it], items.hb[it], items.which[it], 0.5 * du, 0.5 * dphi, gl, wq,
                                             part * 256 + threadIdx.x, SG_SELF_PARTS * 256);
        const double tot = block_sum256(acc, red);
        if (threadIdx.x == 0) out[blockIdx.x] = tot;
        return;
    }
    const int i = (blockIdx.x - nb) * 256 + threadIdx.x;
    const double2 *tw = (const double2 *)sg_tw64;
    if (i < nu) {
        const double2 v = tw[i * (SG_TW64_N / nu)];
        tw_u[i] = make_float2((float)v.x, (float)-v.y);
    }
    if (i < nphi) {
        const double2 v = tw[i * (SG_TW64_N / nphi)];
        tw_phi[i] = make_float2((float)v.x, (float)-v.y);
    }
}

// Rows of one class (M samples), block blk of the class: G groups of T threads,
// two rows per group (z_A + i z_B, as in k_ss_rows).
template <int M, int N>
__device__ inline void tab_rows_body(const TabArgs &A, int cls, int blk, double2 *lds, const double *wq)
{
    using Sh = FftShape<M>;
    constexpr int P = Sh::P, T = Sh::T, G = 256 / T, W = LdsPlane<double>::elems(M);
    const int g = threadIdx.x / T, t = threadIdx.x % T;
    const LdsPlane<double> pl{lds + W * g};
    const TabItem &it = A.it[blockIdx.y];
    const int nr = A.nr, K1 = A.K1[cls], K2 = A.K2[cls];
    const int nk = K1 == 0 ? 2 * K2 - 1 : 2 * (K2 - K1);
    int off[2];
    bool live[2];
    ConvRow64 cr[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int q = 2 * (blk * G + g) + u;
        live[u] = q < nk;
        off[u] = !live[u] ? 0 : K1 == 0 ? q - (K2 - 1) : q < K2 - K1 ? K1 + q : -(K1 + q - (K2 - K1));
        cr[u] = sg_conv_row64(off[u] * A.du, it.ha, it.hb, it.which);
    }
#pragma unroll 1
    for (int q = t; q <= M / 2; q += T) {
        double kr[2], kp[2];
        if (A.A) {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const double2 v = A.A[(size_t)(off[u] < 0 ? off[u] + 2 * nr : off[u]) * N + q];
                kr[u] = live[u] ? v.x : 0.0;
                kp[u] = live[u] ? v.y : 0.0;
            }
        } else {
            const double2 v = ((const double2 *)sg_tw64)[q * (SG_TW64_N / (2 * M))];  // half the azimuth
            const double two_s2 = 2.0 * v.y * v.y, sphi = 2.0 * v.y * v.x;
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const bool none = !live[u] || (off[u] == 0 && q == 0);  // the own cell is added later
                const double x = none ? 1.0 : (cr[u].two_sxh2 + two_s2) * cr[u].inv4h2;
                const double p = none ? 0.0 : (it.which ? sg_D64(x, wq) : sg_F64(x, wq)) * cr[u].pref;
                kr[u] = p * (cr[u].em1 + two_s2);
                kp[u] = p * sphi;
            }
        }
        pl.st(q, make_double2(kr[0] - kp[1], kp[0] + kr[1]));
        if (q != 0 && q != M / 2) pl.st(M - q, make_double2(kr[0] + kp[1], kr[1] - kp[0]));
    }
    __syncthreads();
    double2 z[P];
#pragma unroll
    for (int p = 0; p < P; ++p) z[p] = pl.ld(t + T * p);
    __syncthreads();
    fft<M, false>(z, t, pl, TwPow64<M>{t});
#pragma unroll
    for (int p = 0; p < P; ++p) pl.st(t + T * p, z[p]);
    __syncthreads();
    constexpr double f = 0.5 * (N / M);
    double2 *B = A.B + blockIdx.y * (size_t)((N / 2 + 3) / 4 * 4) * 2 * nr;
    for (int m = t; m < (M == N ? N / 2 : M / 2 + 1); m += T) {
        const double2 zm = pl.ld(m), zn = pl.ld((M - m) & (M - 1));
        double2 v[2] = {make_double2(f * (zm.x + zn.x), f * (zn.x - zm.x)),
                        make_double2(f * (zm.y + zn.y), f * (zn.y - zm.y))};
        if (m == 0) {
            v[0].y = v[1].y = 0.0;
            if (M == N) {
                const double2 zh = pl.ld(M / 2);
                v[0].y = zh.x;
                v[1].y = zh.y;
            }
        }
#pragma unroll
        for (int u = 0; u < 2; ++u)
            if (live[u]) B[tab_index(m, off[u] < 0 ? off[u] + 2 * nr : off[u], 2 * nr)] = v[u];
    }
}

template <int M, int N>
__device__ inline void tab_rows_dispatch(const TabArgs &A, int cls, int blk, double2 *lds, const double *wq)
{
    if (A.M[cls] == M) {
        tab_rows_body<M, N>(A, cls, blk, lds, wq);
        return;
    }
    if constexpr (M > SG_SS_MIN_M && M > 4) tab_rows_dispatch<M / 2, N>(A, cls, blk, lds, wq);
}

// Step 1, all items of a launch (blockIdx.y) and all row classes (blockIdx.x).
template <int N>
__global__ void __launch_bounds__(256) k_tab_rows(TabArgs A)
{
    // the largest plane set over the classes: 256/T planes of M points
    constexpr int E = LdsPlane<double>::elems(N) * (256 / FftShape<N>::T);
    constexpr int E2 = N > SG_SS_MIN_M ? LdsPlane<double>::elems(SG_SS_MIN_M) * (256 / FftShape<SG_SS_MIN_M>::T) : 0;
    __shared__ __attribute__((aligned(16))) double2 lds[E > E2 ? E : E2];
    __shared__ __attribute__((aligned(16))) double wq[FQuad<double>::TABLE];
    if (!A.A) sg_fill64(wq, A.it[blockIdx.y].which ? SG_FN_D : SG_FN_F);
    __syncthreads();
    int cls = 0;
    while (cls + 1 < A.ncls && (int)blockIdx.x >= A.blk0[cls + 1]) ++cls;
    tab_rows_dispatch<N, N>(A, cls, blockIdx.x - A.blk0[cls], lds, wq);
}

// Step 2: column m of item blockIdx.y (column 0: the two real columns 0 and
// n_phi/2 together).  Rows beyond those that resolve mode m are zero and not
// read.  out: spectra at k <= n_r, scaled and rounded; for the kernel itself
// (which = 0) also the pair column of the FFT pass that transforms the two real
// columns as one, (K0 + KN)/2 in the K_r place and (K0 - KN)/2 in the K_phi place.
template <int NU>
__global__ void __launch_bounds__((FftShape<NU>::T > 256 ? FftShape<NU>::T : 256)) k_tab_u(TabArgs A)
{
    using Sh = FftShape<NU>;
    constexpr int P = Sh::P, T = Sh::T, H = NU / 2;
    constexpr int WGS = T > 256 ? T : 256, G = WGS / T, W = LdsPlane<double>::elems(NU);
    __shared__ __attribute__((aligned(16))) double2 lds[W * G];
    const int g = threadIdx.x / T, t = threadIdx.x % T;
    const LdsPlane<double> pl{lds + W * g};
    const int nc = A.nphi / 2, job = sg_xcd_remap(blockIdx.x, 4 / G > 0 ? 4 / G : 1) * G + g;
    const bool valid = job < nc;
    const int m = valid ? job : 0;
    const TabItem &it = A.it[blockIdx.y];
    const double2 *B = A.B + blockIdx.y * (size_t)((nc + 3) / 4 * 4) * NU;
    int kmax = 0;  // rows |k| < kmax resolve mode m (column 0 holds mode n_phi/2 too: its rows are zeros there)
    for (int c = 0; c < A.ncls; ++c)
        if (A.M[c] / 2 >= m) kmax = max(kmax, A.K2[c]);
    double2 v[P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const int r = t + T * p, k = r < H ? r : r - NU;
        v[p] = make_double2(0.0, 0.0);
        if (abs(k) < kmax) v[p] = B[tab_index(m, r, NU)];
    }
    if (t == 0 && A.self) {
        double s = 0.0;
        for (int q = 0; q < SG_SELF_PARTS; ++q) s += A.self[blockIdx.y * SG_SELF_PARTS + q];
        v[0].x += s;
        if (m == 0) v[0].y += s;
    }
    fft<NU, false>(v, t, pl, TwPow64<NU>{t});
#pragma unroll
    for (int p = 0; p < P; ++p) pl.st(t + T * p, v[p]);
    __syncthreads();
    if (!valid) return;
    const double sc = 0.5 * A.scale;
    float2 *o = it.dst + (size_t)m * it.cs;
    float2 *on = it.dst + (size_t)nc * it.cs, *oq = on + it.cs;  // columns n_phi/2 and the pair column
    for (int k = t; k <= H; k += T) {
        const double2 a = pl.ld(k), b = pl.ld((NU - k) & (NU - 1));
        // (W + conj W')/2 and (W - conj W')/2
        const float2 e = make_float2((float)(sc * (a.x + b.x)), (float)(sc * (a.y - b.y)));
        const float2 d = make_float2((float)(sc * (a.x - b.x)), (float)(sc * (a.y + b.y)));
        o[k] = e;
        if (m > 0) {
            o[it.comp + k] = d;  // i times the transform of t_phi
            continue;
        }
        const float2 n = make_float2(d.y, -d.x), zero = make_float2(0.f, 0.f);  // d / i
        o[it.comp + k] = zero;
        on[k] = n;
        on[it.comp + k] = zero;
        if (it.which == 0) {
            oq[k] = make_float2(0.5f * (e.x + n.x), 0.5f * (e.y + n.y));
            oq[it.comp + k] = make_float2(0.5f * (e.x - n.x), 0.5f * (e.y - n.y));
        }
    }
}

// Header, including the indirect-term coefficient of each source fluid: with
// H_a = h_a r the star's kernel has d = 1/h_a at every cell, so
//   sqrt(2) K_a A_k = sqrt(2) pi^{-1/2} h_a^{-3} / 4 F(1 / (4 h_a^2)) du dphi
// (times Sigma_a[k] e^{i phi_k} in the sum), the same for all cells.
__global__ void __launch_bounds__(256)
k_header(sg_table_header *hd, sg_table_header proto, const double *selfbuf, int npair, int with_dh)
{
    // the block fills the coefficient table; one wave adds up the header's values
    __shared__ __attribute__((aligned(16))) double w[FQuad<double>::TABLE];
    sg_fill64(w, SG_FN_F);
    __syncthreads();
    const int k = threadIdx.x;
    if (k >= 64) return;
    const double du = log(proto.r_max / proto.r_min) / proto.n_r;
    const double dphi = 2.0 * SG_PI / proto.n_phi;
    auto self = [&](int it) {
        double s = 0.0;
        for (int q = 0; q < SG_SELF_PARTS; ++q) s += selfbuf[it * SG_SELF_PARTS + q];
        return s;
    };
    if (k == 0) {  // all but the values that follow
        hd->magic = proto.magic;
        hd->version = proto.version;
        hd->n_r = proto.n_r;
        hd->n_phi = proto.n_phi;
        hd->n_fluids = proto.n_fluids;
        hd->flags = proto.flags;
        hd->r_min = proto.r_min;
        hd->r_max = proto.r_max;
        hd->total_bytes = proto.total_bytes;
    }
    if (k < 4) {
        hd->h[k] = proto.h[k];
        const double ha = k < proto.n_fluids ? proto.h[k] : 1.0;
        const double c = SG_SQRT2 / SG_SQRT_PI / (4.0 * ha * ha * ha) * sg_F64(0.25 / (ha * ha), w) * du * dphi;
        hd->ind_coef[k] = k < proto.n_fluids ? c : 0.0;
    }
    if (k < 16) {
        const bool in = k < npair;
        hd->self_r[k] = in ? self(k) : 0.0;
        hd->dself_r[k][0] = in && with_dh ? self(npair + 2 * k) : 0.0;
        hd->dself_r[k][1] = in && with_dh ? self(npair + 2 * k + 1) : 0.0;
    }
}

// ------------------------------------------------------------- F for tests
template <typename T>
__global__ void k_eval_F(const T *x, T *F, T *dF, int64_t n)
{
    __shared__ __attribute__((aligned(16))) T wq[FQuad<T>::TABLE];
    __shared__ __attribute__((aligned(16))) T wd[sizeof(T) == 8 ? FQuad<T>::TABLE : 2];
    if constexpr (sizeof(T) == 8) {
        sg_fill64(wq, SG_FN_F);
        sg_fill64(wd, SG_FN_D);
    } else {
        sg_fill_v(wq, SG_FN_V);
    }
    __syncthreads();
    int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    if constexpr (sizeof(T) == 8) {
        const double f = sg_F64(x[i], wq);
        F[i] = f;
        if (dF) dF[i] = -(sg_D64(x[i], wd) + 1.5 * f) / x[i];
    } else {
        F[i] = sg_F32(x[i], wq);
        if (dF) dF[i] = 0.0f;
    }
}

template <typename T>
__global__ void k_eval_G0(const T *x, T *G, int64_t n)
{
    __shared__ __attribute__((aligned(16))) T wq[FQuad<T>::TABLE];
    if constexpr (sizeof(T) == 8) sg_fill64(wq, SG_FN_G0);
    else sg_fill_v(wq, SG_FN_VG);
    __syncthreads();
    int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    if constexpr (sizeof(T) == 8) G[i] = sg_G0_64(x[i], wq);
    else G[i] = sg_G0_32(x[i], wq);
}

// ------------------------------------------------------------------- host
// Gauss-Legendre nodes and weights on [0,1] (Newton iteration on the
// Legendre three-term recurrence).
static void gl_rule(int n, double *x, double *w)
{
    for (int i = 0; i < n; ++i) {
        double z = cos(SG_PI * (i + 0.75) / (n + 0.5)), p1 = 0, dp = 1;
        for (int it = 0; it < 100; ++it) {
            double p0 = 1.0;
            p1 = z;
            for (int k = 2; k <= n; ++k) {
                double p2 = ((2.0 * k - 1.0) * z * p1 - (k - 1.0) * p0) / k;
                p0 = p1;
                p1 = p2;
            }
            dp = n * (z * p1 - p0) / (z * z - 1.0);
            double dz = p1 / dp;
            z -= dz;
            if (fabs(dz) < 1e-16) break;
        }
        double p0 = 1.0;
        p1 = z;
        for (int k = 2; k <= n; ++k) {
            double p2 = ((2.0 * k - 1.0) * z * p1 - (k - 1.0) * p0) / k;
            p0 = p1;
            p1 = p2;
        }
        dp = n * (z * p1 - p0) / (z * z - 1.0);
        x[i] = 0.5 * (1.0 - z);
        w[i] = 1.0 / ((1.0 - z * z) * dp * dp);
    }
}

namespace {
struct GLCache {  // eta orders 16 and 24 (OwnEta), the same xi rules in each
    GLNodes g[2];
    GLCache()
    {
        const int order[2] = {16, SG_GL_N};
        for (int k = 0; k < 2; ++k) {
            g[k] = GLNodes{};
            g[k].ne = order[k];
            gl_rule(order[k], g[k].x, g[k].w);
            gl_rule(SG_GLX_N, g[k].xr, g[k].wr);
            gl_rule(SG_GLT_N, g[k].tx, g[k].tw);
            for (int i = 0; i < SG_GLT_N; ++i) {
                const double t = g[k].tx[i];
                g[k].tx[i] = t * t * t * t;
                g[k].tw[i] *= 4.0 * t * t * t;
            }
        }
    }
};
}  // namespace

void sg_gl_nodes(GLNodes &gl, double aspect)
{
    static const GLCache cache;  // built once, by the first caller
    gl = cache.g[aspect <= 8.0 && aspect >= 0.125 ? 0 : 1];
}

static bool launch_tab_rows(const TabArgs &A, hipStream_t s)
{
    const dim3 grid((unsigned)A.blk0[A.ncls], (unsigned)A.nit);
    switch (A.nphi) {
#define SG_ROWS(N) \
    case N: hipLaunchKernelGGL(k_tab_rows<N>, grid, dim3(256), 0, s, A); return true;
        SG_ROWS(4) SG_ROWS(8) SG_ROWS(16) SG_ROWS(32) SG_ROWS(64) SG_ROWS(128) SG_ROWS(256) SG_ROWS(512)
        SG_ROWS(1024) SG_ROWS(2048)
#undef SG_ROWS
    }
    return false;
}

template <int NU> static void launch_tab_u(const TabArgs &A, hipStream_t s)
{
    constexpr int T = FftShape<NU>::T, WGS = T > 256 ? T : 256, G = WGS / T, K = 4 / G > 0 ? 4 / G : 1;
    const int nwg = (A.nphi / 2 + G - 1) / G;  // whole XCD clusters of 8 K
    hipLaunchKernelGGL(k_tab_u<NU>, dim3((unsigned)((nwg + 8 * K - 1) / (8 * K) * (8 * K)), (unsigned)A.nit), dim3(WGS),
                       0, s, A);
}

static bool dispatch_tab_u(const TabArgs &A, hipStream_t s)
{
    switch (2 * A.nr) {
#define SG_COLS(N) \
    case N: launch_tab_u<N>(A, s); return true;
        SG_COLS(4) SG_COLS(8) SG_COLS(16) SG_COLS(32) SG_COLS(64) SG_COLS(128) SG_COLS(256) SG_COLS(512)
        SG_COLS(1024) SG_COLS(2048) SG_COLS(4096)
#undef SG_COLS
    }
    return false;
}

// Own-cell parts, then the intermediate columns (with SG_SECOND_ORDER the
// samples before them).
static size_t tab_self_bytes() { return sg_align256(sizeof(double) * SG_SELF_MAX * SG_SELF_PARTS); }

size_t sg_table_ws_bytes(int nr, int nphi)
{
    const size_t A = sizeof(double2) * 2 * (size_t)nr * nphi;
    const size_t B = sizeof(double2) * 2 * (size_t)(nphi / 2 + 1) * 2 * nr;
    const size_t item = sizeof(double2) * tab_item_elems(nr, nphi);
    return sg_align256(A) + sg_align256(B > item ? B : item) + tab_self_bytes();
}

// Row classes of the grid: M azimuths for the offsets K1 <= |k| < K2 with
// M |k| du >= SG_SS_ALIAS; one class of all rows where that saves nothing (and
// with second-order samples, which exist on the full grid).
static void tab_classes(TabArgs &A, bool second)
{
    A.ncls = 0;
    A.blk0[0] = 0;
    for (int M = A.nphi;; M /= 2) {
        const bool last = second || M / 2 < SG_SS_MIN_M;
        const int K1 = M == A.nphi ? 0 : (int)fmin(ceil(SG_SS_ALIAS / M / A.du), (double)A.nr);
        const int K2 = last ? A.nr : (int)fmin(ceil(SG_SS_ALIAS / (M / 2) / A.du), (double)A.nr);
        if (K1 < K2) {
            const int c = A.ncls++;
            const int nk = K1 == 0 ? 2 * K2 - 1 : 2 * (K2 - K1), T = M >= 8 ? M / 8 : 1, G = 256 / T;
            A.M[c] = M;
            A.K1[c] = K1;
            A.K2[c] = K2;
            A.blk0[c + 1] = A.blk0[c] + ((nk + 1) / 2 + G - 1) / G;
        }
        if (last) break;
    }
}

sg_status sg_table_build(const sg_grid *grid, const sg_fluids *fl, uint32_t flags, void *d_table,
                         void *d_ws, hipStream_t s)
{
    const int nr = grid->n_r, nphi = grid->n_phi, nf = fl->n_fluids;
    const TableLayout L = sg_table_layout(nr, nphi, nf, flags);
    const double du = log(grid->r_max / grid->r_min) / nr;
    const double dphi = 2.0 * SG_PI / nphi;
    char *tb = (char *)d_table;
    char *ws = (char *)d_ws;
    double *selfbuf = (double *)ws;
    double2 *A0 = (double2 *)(ws + tab_self_bytes());
    const size_t bytes = sg_table_ws_bytes(nr, nphi) - tab_self_bytes();
    const bool with_dh = (flags & SG_WITH_DH) != 0;
    const bool excl = (flags & SG_SELF_CELL_EXCLUDE) != 0;
    const bool second = (flags & SG_SECOND_ORDER) != 0;  // no own-cell switch

    // items: [pair] for which = 0, then [pair][d] for the derivatives
    float2 *spec = (float2 *)(tb + L.off_spec);
    float2 *dspec = (float2 *)(tb + L.off_dspec);
    SelfItems items{};
    std::vector<TabItem> its;
    for (int w = 0; w < (with_dh ? 2 : 1); ++w)
        for (int a = 0; a < nf; ++a)
            for (int b = 0; b < nf; ++b)
                for (int d = 0; d < (w ? 2 : 1); ++d) {
                    const int pair = a * nf + b, n = (int)its.size();
                    TabItem it;
                    it.ha = fl->h[a];
                    it.hb = fl->h[b];
                    it.which = w ? 1 + d : 0;
                    it.comp = (uint32_t)L.kk;
                    it.cs = (uint32_t)(L.npair * (w ? 4 : 2) * L.kk);                  // dspec: [m][pair][d][c][k]
                    it.dst = w ? dspec + (size_t)(pair * 2 + d) * 2 * L.kk : spec + (size_t)pair * 2 * L.kk;
                    its.push_back(it);
                    items.ha[n] = it.ha;
                    items.hb[n] = it.hb;
                    items.which[n] = it.which;
                }
    const int nit = (int)its.size();
    const bool own = !excl && !second;  // second order: W_r(0, 0) is copied in per item below
    GLNodes gl;
    sg_gl_nodes(gl, du / dphi);
    if (excl) {
        hipLaunchKernelGGL(k_fill_f64, dim3(4), dim3(256), 0, s, selfbuf, (int64_t)nit * SG_SELF_PARTS, 0.0);
        SG_HIP(hipGetLastError());
    }
    {
        const int n = 2 * nr > nphi ? 2 * nr : nphi, nself = own ? nit : 0;
        hipLaunchKernelGGL(k_tab_pre, dim3((unsigned)(nself * SG_SELF_PARTS + (n + 255) / 256)), dim3(256), 0, s, items,
                           nself, selfbuf, du, dphi, gl, (float2 *)(tb + L.off_tw_u), 2 * nr,
                           (float2 *)(tb + L.off_tw_phi), nphi);
        SG_HIP(hipGetLastError());
    }
    TabArgs T{};
    T.nr = nr;
    T.nphi = nphi;
    T.du = du;
    T.dphi = dphi;
    T.scale = -du * dphi / (2.0 * nr * (double)nphi);
    tab_classes(T, second);
    const size_t item = sizeof(double2) * tab_item_elems(nr, nphi);
    T.B = second ? (double2 *)((char *)A0 + sg_align256(sizeof(double2) * 2 * (size_t)nr * nphi)) : A0;
    const int batch = second ? 1 : std::max(1, (int)std::min<size_t>(SG_TAB_ITEMS, bytes / item));
    for (int i0 = 0; i0 < nit; i0 += batch) {
        T.nit = std::min(batch, nit - i0);
        for (int i = 0; i < T.nit; ++i) T.it[i] = its[i0 + i];
        T.self = own ? selfbuf + (size_t)i0 * SG_SELF_PARTS : nullptr;
        if (second) {
            const TabItem &it = its[i0];
            T.A = A0;
            hipLaunchKernelGGL(k_sample_hat_far, dim3((nphi + 255) / 256, 2 * nr), dim3(256), 0, s, A0, nr, nphi, du,
                               it.ha, it.hb, it.which);
            hipLaunchKernelGGL(k_sample_hat_near, dim3(9), dim3(256), 0, s, A0, nr, nphi, du, it.ha, it.hb, it.which,
                               gl);
            // the header's own-cell value of this pair (or its derivative): W_r(0, 0)
            hipLaunchKernelGGL(k_copy_w00, dim3(1), dim3(1), 0, s, (const double2 *)A0, selfbuf + (size_t)i0 * SG_SELF_PARTS);
            SG_HIP(hipGetLastError());
        }
        if (!launch_tab_rows(T, s)) return SG_ERR_UNSUPPORTED;
        SG_HIP(hipGetLastError());
        if (!dispatch_tab_u(T, s)) return SG_ERR_UNSUPPORTED;
        SG_HIP(hipGetLastError());
    }
    sg_table_header proto{};
    proto.magic = SG_TABLE_MAGIC;
    proto.version = 1;
    proto.n_r = nr;
    proto.n_phi = nphi;
    proto.n_fluids = nf;
    proto.flags = flags;
    for (int a = 0; a < 4; ++a) proto.h[a] = a < nf ? fl->h[a] : 0.0;
    proto.r_min = grid->r_min;
    proto.r_max = grid->r_max;
    proto.total_bytes = L.total;
    hipLaunchKernelGGL(k_header, dim3(1), dim3(256), 0, s, (sg_table_header *)tb, proto, selfbuf, L.npair,
                       with_dh ? 1 : 0);
    SG_HIP(hipGetLastError());
    return SG_OK;
}

sg_status sg_self_cell_launch(const sg_grid *grid, const double *ha, const double *hb, int n,
                              int which, double *d_out, hipStream_t s)
{
    if (n < 1 || n > SG_SELF_MAX || which < 0 || which > 2) return SG_ERR_ARG;
    SelfItems items{};
    for (int i = 0; i < n; ++i) {
        items.ha[i] = ha[i];
        items.hb[i] = hb[i];
        items.which[i] = which;
    }
    const double du = log(grid->r_max / grid->r_min) / grid->n_r;
    const double dphi = 2.0 * SG_PI / grid->n_phi;
    GLNodes gl;
    sg_gl_nodes(gl, du / dphi);
    hipLaunchKernelGGL(k_self_cell, dim3(n), dim3(256), 0, s, items, d_out, du, dphi, gl);
    SG_HIP(hipGetLastError());
    return SG_OK;
}

sg_status sg_eval_G0_launch(const void *x, void *G, int64_t n, sg_dtype dt, hipStream_t s)
{
    const int64_t nb = (n + 255) / 256;
    if (dt == SG_F64)
        hipLaunchKernelGGL(k_eval_G0<double>, dim3((unsigned)nb), dim3(256), 0, s, (const double *)x,
                           (double *)G, n);
    else
        hipLaunchKernelGGL(k_eval_G0<float>, dim3((unsigned)nb), dim3(256), 0, s, (const float *)x,
                           (float *)G, n);
    SG_HIP(hipGetLastError());
    return SG_OK;
}

sg_status sg_eval_F_launch(const void *x, void *F, void *dF, int64_t n, sg_dtype dt, hipStream_t s)
{
    const int64_t nb = (n + 255) / 256;
    if (dt == SG_F64)
        hipLaunchKernelGGL(k_eval_F<double>, dim3((unsigned)nb), dim3(256), 0, s, (const double *)x,
                           (double *)F, (double *)dF, n);
    else
        hipLaunchKernelGGL(k_eval_F<float>, dim3((unsigned)nb), dim3(256), 0, s, (const float *)x,
                           (float *)F, (float *)dF, n);
    SG_HIP(hipGetLastError());
    return SG_OK;
}
