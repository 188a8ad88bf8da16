// sg_table.h -- internal declarations shared by the library's translation units.
#pragma once
#include "sg_internal.h"

#define SG_GL_N 24          // largest Gauss-Legendre order across the self cell (eta)
#define SG_GLX_N 16         // Gauss-Legendre order per radial panel (xi)
#define SG_PANELS 7         // geometric xi panels [0,4^-6], [4^-(j+1), 4^-j]
#define SG_GLT_N 24         // Gauss-Legendre order of the graded xi rule (xi = t^4)
#define SG_OWN_RMAX 8.0     // largest (half cell side) / H of the graded rule
#define SG_SELF_MAX 64      // items per self-cell launch
#define SG_SELF_PARTS 4     // blocks per own-cell item of a table build

// Nodes of the own-cell rules.  eta: order ne, chosen from the cell's aspect
// ratio.  xi: the graded rule (tx, tw), or the panel rule (xr, wr per panel).
struct GLNodes {
    int ne;
    double x[SG_GL_N], w[SG_GL_N];
    double xr[SG_GLX_N], wr[SG_GLX_N];
    double tx[SG_GLT_N], tw[SG_GLT_N];
};

// Node idx of the rule with nx xi nodes: xi, the eta node's s in [0, 1] (see
// OwnEta) and the weight, the Jacobian's xi included.
//
// Both xi rules integrate over [0, 1] with a logarithm at 0.  xi = t^4 takes
// the logarithm down to t^7 log t, and 24 nodes then leave less than 7e-17 of
// the field, its h derivatives and the potential (in 32-digit arithmetic, half
// sides of 0.03 to 7.9 H, heights equal and 10 apart).  In double a field's
// two halves cancel to about a half side, which leaves 2e-15 on cells of 0.05,
// 5e-14 on cells of 0.003 with equal heights, 1e-12 with heights 10 to 300
// apart.  The rule holds while the cell is not much larger than H: at half side
// / H = 16 the derivatives are at 1e-11, so beyond SG_OWN_RMAX the panels
// resolve the transition of F at distances ~ H, the innermost one graded
// likewise (its logarithm left 1e-12 to 1e-10 in the potential of cells 10 to
// 1000 H across; 4e-16 with the grading).
__device__ inline void sg_own_node(const GLNodes &gl, int nx, int idx, double &xi, double &s, double &wgt)
{
    const int ix = idx / gl.ne, j = idx % gl.ne;
    s = gl.x[j];
    if (nx == SG_GLT_N) {
        xi = gl.tx[ix];
        wgt = gl.tw[ix] * gl.w[j] * xi;
        return;
    }
    const int pnl = ix / SG_GLX_N, i = ix % SG_GLX_N;
    const double hi = ldexp(1.0, -2 * (SG_PANELS - 1 - pnl));
    const double t = gl.xr[i];
    xi = pnl == 0 ? hi * (t * t) * (t * t) : 0.25 * hi + 0.75 * hi * t;
    wgt = hi * (pnl == 0 ? 4.0 * t * t * t : 0.75) * gl.wr[i] * gl.w[j] * xi;
}

// The triangle X = a xi, phi = b xi eta has its nearest singularities at eta
// = +-i a/b (the other triangle at +-i b/a).  eta = q sinh(s asinh(1/q)), q
// that ratio, moves them to a distance that shrinks only with log(1/q): in
// 32-digit arithmetic 16 nodes leave less than 7e-17 at an aspect of 2, 24 nodes
// 2.4e-16 at 390 (plain Gauss-Legendre: 48 nodes 1e-13 at 20, 4e-7 at 100).
struct OwnEta {
    double q, L;
    __device__ inline OwnEta(double num, double den) : q(num / den), L(asinh(den / num)) {}
    __device__ inline double at(double s, double &w) const
    {
        const double e = sinh(s * L);
        w *= q * L * sqrt(1.0 + e * e);
        return q * e;
    }
};

// xi nodes for an own cell of half sides a, b (in ln r and phi) and aspect
// ratio h (the smallest of the heights involved, over r).
__device__ inline int sg_own_nx(double a, double b, double h)
{
    return fmax(a, b) <= SG_OWN_RMAX * h ? SG_GLT_N : SG_PANELS * SG_GLX_N;
}

struct SelfItems {
    double ha[SG_SELF_MAX], hb[SG_SELF_MAX];
    int which[SG_SELF_MAX];
};

void sg_gl_nodes(GLNodes &gl, double aspect);  // aspect: cell sides' ratio (either way round)
// Worst aspect ratio of the cells of a uniform radial grid: ln(1 + dr/(2r)) and
// -ln(1 - dr/(2r)) against dphi / 2, at the innermost and outermost rings.
inline double sg_lin_aspect(const sg_grid &g, double dphi)
{
    const double dr = (g.r_max - g.r_min) / g.n_r;
    const double hi = -log1p(-0.5 * dr / (g.r_min + 0.5 * dr)), lo = log1p(0.5 * dr / (g.r_max - 0.5 * dr));
    const double p = 2.0 * hi / dphi, q = 0.5 * dphi / lo;
    return p > q ? p : q;
}
size_t sg_table_ws_bytes(int nr, int nphi);
sg_status sg_table_build(const sg_grid *grid, const sg_fluids *fl, uint32_t flags, void *d_table,
                         void *d_ws, hipStream_t s);
sg_status sg_self_cell_launch(const sg_grid *grid, const double *ha, const double *hb, int n,
                              int which, double *d_out, hipStream_t s);
sg_status sg_eval_F_launch(const void *x, void *F, void *dF, int64_t n, sg_dtype dt, hipStream_t s);
sg_status sg_eval_G0_launch(const void *x, void *G, int64_t n, sg_dtype dt, hipStream_t s);

__global__ void k_twiddles(float2 *tw_phi, int nphi);
__global__ void k_self_cell(SelfItems items, double *out, double du, double dphi, GLNodes gl);
// Own-cell integrals on a uniform radial grid (defined with the semi-spectral
// path): item = pair * n_r * per + cell, H double [F][n_r * per].
__global__ void k_ss_self_lin(const double *H, int nf, int nr, int per, double rmin, double dr, double dphi,
                              int pot, int which, double *out, GLNodes gl);
__global__ void k_self_cell_ring(const double *H, int nf, int nr, double lnrmin, double du, double dphi, int which,
                                 double *out, GLNodes gl);
// Own-cell integrals on the log grid for every pair and cell (nphi = 1: one
// value per ring), H [F][n_r * nphi]: out[pair][cell].
template <typename T>
void sg_self_cells(const T *H, int nf, int nr, int nphi, double lnrmin, double du, double dphi, double *out,
                   hipStream_t s);
template <typename T>
void sg_pot_cells(const T *H, const double *h, int nf, int nr, int nphi, double lnrmin, double du, double dphi,
                  int per_row, double *out, int which, hipStream_t s);
__global__ void k_fill_f64(double *p, int64_t n, double v);
