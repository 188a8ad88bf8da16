// sg_direct.hip -- O(N^2) direct summation of the exact kernel (Sect. 2.2,
// the 2D force through the kernel, divided by Sigma_b) for general per-cell
// scale heights, in float or double.
//
// For target cell i (fluid b) and source cell k != i (fluid a) on the log-r x
// uniform-phi grid, with X = u_i - u_k and phi = phi_i - phi_k:
//   s^2        = r_i r_k (4 sinh^2(X/2) + 4 sin^2(phi/2))    (cancellation-free)
//   H_ab^2     = (H_a[k]^2 + H_b[i]^2) / 2,  x = s^2 / (8 H_ab^2)
//   K_ab / s   = F(x) / (8 sqrt(pi) H_ab^3) = V(1/x) (s^2/8)^{-3/2} / (8 sqrt(pi))
//   e_s . e_r  = (r_i - r_k cos phi)/s = r_k (e^X - cos phi)/s,
//   e_s . e_phi = r_k sin phi / s,
//   g_r  -= Sigma_a[k] A_k (K/s) r_k (expm1(X) + 2 sin^2(phi/2)),
//   g_phi -= Sigma_a[k] A_k (K/s) r_k sin phi.
// The offset factors depend only on (i_r - k_r) and (j - l) and are tabulated
// once per call in double (rounded for the float path).  On a uniform radial
// grid (SG_LINEAR_R: centres r_min + (i + 1/2) dr, sector areas r dr dphi)
// the radial factors 4 sinh^2(X/2) = (r_i - r_k)^2 / (r_i r_k) and
// expm1(X) = (r_i - r_k) / r_k are formed per source row instead, with r_i - r_k
// = (i - k) dr (the difference of float radii left 1e-4 of the field of an
// annulus of r_max / r_min = 1.01).
//
// H = h r (d_H == NULL) makes the kernel between two rings a function of the
// azimuth offset alone: k_ring_sum evaluates it once per offset and sums it
// against the source row as a Toeplitz product.  The rest of this comment is
// about the general sum with a scale height per cell (and of rings of few cells).
//
// Layout: one thread per target cell (256 per workgroup), all target fluids
// in registers; the source loop runs over whole radial rows so every
// per-source quantity is wave-uniform (scalar loads); the source rows are
// split over blockIdx.y when there are too few targets to fill 256 CUs, and
// the per-split partial sums are reduced in a fixed order by a second kernel
// that also adds the self term and, with SG_INDIRECT, the indirect term
// (deterministic; no atomics).
//
// Accumulation (both precisions): the sources of a row are taken in chunks of
// SG_DCHUNK azimuths, each chunk summed into a fresh partial, and the chunk
// partials are added to the running total with an error-free transformation
// (Knuth's TwoSum), whose rounding errors are carried in a second
// accumulator.  A single running sum over all 2^21 sources of a 1024 x 2048
// disc would lose about three digits to the cancellation between the pull of
// the inner and of the outer disc; chunking bounds the plain-sum part to 64
// terms and the compensated outer sum is exact to first order, so the result
// sits at the rounding floor of the individual terms.  Each split hands
// (sum, carried error) to the reduction, which adds them in double.
#include <algorithm>

#include "sg_direct.h"
#include "sg_kfn.h"
#include "sg_table.h"

template <typename T> struct DirectArgs {
    int nr, nphi, rps;   // rows per split
    int lin;             // uniform radial grid
    T dr;                // its spacing
    int64_t N;
    const T *rrow, *sx, *ex, *sph, *snp, *mass, *H2;
    T *partial;          // [split][fluid][component][hi, lo][N]
};

#define SG_DCHUNK 64

// s + v = (s', e') exactly (Knuth's TwoSum); the error goes into c.  No
// products, so contraction into FMAs cannot change it.
template <typename T> __device__ inline void sg_two_sum_acc(T &s, T &c, T v)
{
    const T t = s + v;
    const T bp = t - s;
    c += (s - (t - bp)) + (v - bp);
    s = t;
}

// The float sums take lengths in units of the power of two below r_min: a
// pair's factor (s^2/8)^{-3/2} and the masses r^3 Sigma would otherwise leave
// float's range where lengths are far from 1 (discs in metres or centimetres:
// subnormal from s = 1e13 on).  The field does not depend on the unit of length,
// the potential is proportional to it; a power of two costs no rounding.
template <typename T> static double length_unit(const sg_grid &g)
{
    return sizeof(T) == 4 ? ldexp(1.0, ilogb(g.r_min)) : 1.0;
}

// Ring radius: log grid (lin = 0) or uniform grid (a = r_min, b = dr).
__device__ inline double dir_radius(int lin, double lnrmin, double du, double rmin, double dr, int i)
{
    return lin ? rmin + (i + 0.5) * dr : exp(lnrmin + (i + 0.5) * du);
}

template <typename T>
__global__ void k_direct_prep(int nr, int nphi, int nf, double lnrmin, double du, double dphi,
                              const double *h, const T *sigma, const T *H, T *rrow, T *sx, T *ex,
                              T *sph, T *snp, T *mass, T *H2, int lin, double rmin, double dr, double *Hd,
                              int scaled, double unit)
{
    // lnrmin, rmin, dr and the radii here in units of unit; sigma, H and Hd not
    const int64_t N = (int64_t)nr * nphi;
    const int64_t tid = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = tid; i < nr; i += stride) rrow[i] = (T)dir_radius(lin, lnrmin, du, rmin, dr, (int)i);
    for (int64_t p = tid; p < 2 * nr - 1; p += stride) {
        const double X = (double)(p - (nr - 1)) * du;
        const double s = sinh(0.5 * X);
        sx[p] = (T)(4.0 * s * s);
        ex[p] = (T)expm1(X);
    }
    for (int64_t q = tid; q < nphi; q += stride) {
        const double s = sinpi((double)q / nphi);
        sph[q] = (T)(4.0 * s * s);
        snp[q] = (T)sinpi(2.0 * (double)q / nphi);
    }
    for (int64_t k = tid; k < nf * N; k += stride) {
        const int64_t cell = k % N;
        const int ir = (int)(cell / nphi);
        const double r = dir_radius(lin, lnrmin, du, rmin, dr, ir);
        // scaled: times the pair sums' constant, -r_k / (8 sqrt(pi)) (field, 1)
        // or -1 / (2 sqrt(pi)) (potential, 2)
        const double c = scaled == 1 ? -r / (8.0 * SG_SQRT_PI) : scaled == 2 ? -0.5 / SG_SQRT_PI : 1.0;
        mass[k] = (T)((double)sigma[k] * (lin ? r * dr : r * r * du) * dphi * c);
        const double Hk = H ? (double)H[k] / unit : h[k / N] * r;
        H2[k] = (T)(0.5 * Hk * Hk);  // H_ab^2 = H2_a + H2_b
        if (lin && H) Hd[k] = (double)H[k];  // double H per cell for the own-cell integrals
    }
    if (lin && !H)  // double H per ring
        for (int64_t k = tid; k < (int64_t)nf * nr; k += stride)
            Hd[k] = h[k / nr] * (dir_radius(1, 0.0, 0.0, rmin, dr, (int)(k % nr)) * unit);
}

// General sum (a scale height per cell): VALU bound.  Per source one
// reciprocal square root (of s^2/8) serves every pair of fluids, per pair one
// V(u) (17 float instructions with its table reads, 10 where the whole wave is
// beyond x = 64).  Two fluids, 101 x 250 cells in float: 1.4 ms, 1.8e12 pairs/s
// (2.9 ms with a reciprocal square root and the 9-node trapezoid per pair); the
// double potential of 96 x 200 cells 0.78 ms (2.35 ms at first, 0.96 ms with F(x)
// per pair), bound by the 96 bytes of table per lane and pair.
template <typename T, int NF>
__global__ void __launch_bounds__(256) k_direct(DirectArgs<T> A)
{
    __shared__ __attribute__((aligned(16))) T wq[FQuad<T>::TABLE];
    sg_fill_v(wq, SG_FN_V);
    __syncthreads();
    const int64_t t = blockIdx.x * (int64_t)256 + threadIdx.x;
    if (t >= A.N) return;
    const int nphi = A.nphi, nr = A.nr;
    const int ir = (int)(t / nphi), j = (int)(t % nphi);
    const T ri = A.rrow[ir];
    T hb2[NF], accr[NF], accp[NF], errr[NF], errp[NF];
#pragma unroll
    for (int b = 0; b < NF; ++b) {
        hb2[b] = A.H2[b * A.N + t];
        accr[b] = T(0);
        accp[b] = T(0);
        errr[b] = T(0);
        errp[b] = T(0);
    }
    const int r0 = blockIdx.y * A.rps;
    const int r1 = min(nr, r0 + A.rps);
    for (int kr = r0; kr < r1; ++kr) {
        const T rk = A.rrow[kr];
        T SX, EX;
        if (A.lin) {
            const T d = T(ir - kr) * A.dr;
            SX = d * d / (ri * rk);
            EX = d / rk;
        } else {
            const int p = ir - kr + nr - 1;
            SX = A.sx[p];
            EX = A.ex[p];
        }
        const T rr8 = ri * rk * T(0.125);
        const int64_t kbase = (int64_t)kr * nphi;
        const int lself = kr == ir ? j : -1;  // the own cell: l == j on the own ring
        for (int l0 = 0; l0 < nphi; l0 += SG_DCHUNK) {
            const int l1 = min(nphi, l0 + SG_DCHUNK);
            T pr[NF], pp[NF];  // this chunk's partial sums
#pragma unroll
            for (int b = 0; b < NF; ++b) {
                pr[b] = T(0);
                pp[b] = T(0);
            }
            for (int l = l0; l < l1; ++l) {
                const int64_t k = kbase + l;
                int q = j - l;
                q += q < 0 ? nphi : 0;
                const T sp = A.sph[q];
                const bool self = l == lself;
                const T rs = sg_rsqrt(self ? T(1) : rr8 * (SX + sp)), rs2 = rs * rs;  // s^2 / 8
                const T rs3 = self ? T(0) : rs2 * rs;
                const T emc = EX + T(0.5) * sp;
                const T sn = A.snp[q];
#pragma unroll
                for (int b = 0; b < NF; ++b) {
                    const T ub = hb2[b] * rs2;
                    T c = T(0);
#pragma unroll
                    for (int a = 0; a < NF; ++a)
                        c += A.mass[a * A.N + k] * sg_v<SG_FN_V>(A.H2[a * A.N + k] * rs2 + ub, wq);
                    c *= rs3;
                    pr[b] += c * emc;
                    pp[b] += c * sn;
                }
            }
#pragma unroll
            for (int b = 0; b < NF; ++b) {
                sg_two_sum_acc(accr[b], errr[b], pr[b]);
                sg_two_sum_acc(accp[b], errp[b], pp[b]);
            }
        }
    }
#pragma unroll
    for (int b = 0; b < NF; ++b) {
        T *o = A.partial + (int64_t)(blockIdx.y * NF + b) * 4 * A.N + t;
        o[0] = accr[b];
        o[A.N] = errr[b];
        o[2 * A.N] = accp[b];
        o[3 * A.N] = errp[b];
    }
}

// ------------------------------------------------- ring sums (H = h r)
// One block: target ring blockIdx.x / ntile (a tile of TJ = 8 JT of its
// azimuths), target fluid blockIdx.z, source rings of split blockIdx.y.  Per
// source ring and fluid the kernel is a vector over the azimuth offset q (K_r
// even, K_phi odd: nphi/2 + 1 evaluations), staged in LDS in the order of
// l - j so that the sum over the source azimuths l is a Toeplitz product:
// thread (jt, g) holds the 8 targets j0 = 8 jt .. j0 + 7 of its tile, loads 8
// offsets and 8 masses at a time and does 64 FMAs per component on them and
// the previous 8 offsets.  The 256 / JT groups g share the work as KS source
// rings at a time times LG interleaved 64-azimuth chunks; their sums are
// combined in a fixed order at the end.
//
// FP32 / FP64 VALU bound, two FMAs per pair of cells and fluid pair (one for
// the potential) in place of a kernel evaluation.  The whole call: 256 x 512 in
// float 0.99 ms (35e12 FMA/s of 39e12), against 21.4 ms with a kernel
// evaluation per pair; 64 x 128 in double 41 us (this kernel 21) against 690 us.
// 8 x 8 per step keeps LDS below the VALU
// (per wave 6 16-byte reads for 128 FMAs in float, 12 in double); rows are
// padded by 16 bytes per 8 elements, which puts the 8 lanes of a 16-byte
// access phase (one element group apart) on different banks.
#define SG_RING_LDS (48 << 10)  // staged rows per block: three blocks per CU
struct RingShape {
    int JT, KS, LG;   // threads along j, source rings staged at a time, chunk groups
    int ntile, TL;    // azimuth tiles of a target ring; staged source azimuths (multiple of 8)
    int rps;          // source rings per split (multiple of KS)
    size_t lds;
};

template <typename T> struct RingPad {
    static constexpr int G = 8 + 16 / (int)sizeof(T);  // elements per padded group of 8
};

template <typename T, int NC>
static RingShape ring_shape(int nr, int nphi, int nf, int smax)
{
    const int jtmax = sizeof(T) == 4 ? 256 : 128, tlmax = sizeof(T) == 4 ? 1024 : 512;
    RingShape P;
    const int g8 = (nphi + 7) / 8;
    P.ntile = (g8 + jtmax - 1) / jtmax;
    P.JT = (g8 + P.ntile - 1) / P.ntile;
    P.TL = std::min(8 * g8, tlmax);
    const int S = 256 / P.JT, nch = (P.TL + 63) / 64;
    P.LG = std::min(nch, S);
    const size_t row = (size_t)(P.JT + P.TL / 8) * RingPad<T>::G, per = sizeof(T) * (NC * row + P.TL);
    P.KS = std::max(1, std::min({S / P.LG, nr, (int)(SG_RING_LDS / per)}));
    // splits: about 2048 blocks, within the partial-sum buffer
    const int64_t blocks = (int64_t)nr * P.ntile * nf;
    const int64_t want = std::max<int64_t>(1, std::min<int64_t>((2048 + blocks - 1) / blocks, smax));
    int rps = (int)((nr + want - 1) / want);
    P.rps = (rps + P.KS - 1) / P.KS * P.KS;
    P.lds = std::max(P.KS * per, sizeof(T) * (size_t)P.JT * P.KS * P.LG * 16);
    return P;
}

// Kernel per unit mass between ring ir (fluid b) and source ring kr (fluid a)
// at azimuth offset q: (g_r, g_phi), or the potential.
template <typename T, int NC>
__device__ inline void ring_kernel(const DirectArgs<T> &A, int ir, int kr, int a, int b, int q, const T *wq, T (&K)[NC])
{
    const T ri = A.rrow[ir], rk = A.rrow[kr];
    T SX, EX;
    if (A.lin) {
        const T d = T(ir - kr) * A.dr;
        SX = d * d / (ri * rk);
        EX = d / rk;
    } else {
        const int p = ir - kr + A.nr - 1;
        SX = A.sx[p];
        EX = A.ex[p];
    }
    const T sp = A.sph[q];
    const T H2ab = A.H2[a * A.N + (int64_t)kr * A.nphi] + A.H2[b * A.N + (int64_t)ir * A.nphi];
    const bool self = kr == ir && q == 0;
    const T rs = sg_rsqrt(self ? T(1) : ri * rk * T(0.125) * (SX + sp)), rs2 = rs * rs;  // s^2 / 8
    if constexpr (NC == 2) {
        const T c = self ? T(0) : T(-1.0 / (8.0 * SG_SQRT_PI)) * rk * sg_v<SG_FN_V>(H2ab * rs2, wq) * (rs2 * rs);
        K[0] = c * (EX + T(0.5) * sp);
        K[1] = c * A.snp[q];
    } else {
        K[0] = self ? T(0) : T(-0.5 / SG_SQRT_PI) * sg_v<SG_FN_VG>(H2ab * rs2, wq) * rs;
    }
}

template <typename T, int NC>
__global__ void __launch_bounds__(256) k_ring_sum(DirectArgs<T> A, RingShape P, int nf)
{
    extern __shared__ __attribute__((aligned(16))) char smem[];
    __shared__ __attribute__((aligned(16))) T wq[FQuad<T>::TABLE];
    constexpr int PG = RingPad<T>::G;
    sg_fill_v(wq, NC == 2 ? SG_FN_V : SG_FN_VG);
    const int ir = blockIdx.x / P.ntile, jb = (blockIdx.x % P.ntile) * 8 * P.JT, b = blockIdx.z;
    const int nphi = A.nphi, rowg = P.JT + P.TL / 8;
    T *D = (T *)smem, *M = D + (size_t)P.KS * NC * rowg * PG;
    const int jt = threadIdx.x % P.JT, g = threadIdx.x / P.JT;
    const int ks = g % P.KS, lg = g / P.KS;
    const bool act = lg < P.LG;
    T acc[NC][8], err[NC][8];
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int r = 0; r < 8; ++r) acc[c][r] = err[c][r] = T(0);
    const int r0 = blockIdx.y * P.rps, r1 = min(A.nr, r0 + P.rps);
    const bool whole = nphi <= P.TL;  // every offset of the row is staged at once
    for (int k0 = r0; k0 < r1; k0 += P.KS)
        for (int l0 = 0; l0 < nphi; l0 += P.TL)
            for (int a = 0; a < nf; ++a) {
                __syncthreads();  // the weights; the previous stage's readers
                const int tl = min(P.TL, nphi - l0), lpad = (tl + 7) & ~7;
                // element y of a row: offset x = l - j = y + l0 - jb - TJ, q = -x mod nphi
                const int x0 = l0 - jb - 8 * P.JT, wn = 8 * P.JT + lpad;
                const int per = whole ? nphi / 2 + 1 : wn;
                for (int e = threadIdx.x; e < P.KS * per; e += 256) {
                    const int s = e / per, v = e - s * per, kr = k0 + s;
                    int q = v;
                    if (!whole) {
                        q = (int)(-(int64_t)(x0 + v) % nphi);
                        q += q < 0 ? nphi : 0;
                    }
                    T K[NC];
#pragma unroll
                    for (int c = 0; c < NC; ++c) K[c] = T(0);
                    if (kr < r1) ring_kernel<T, NC>(A, ir, kr, a, b, q, wq, K);
                    T *row = D + (size_t)s * NC * rowg * PG;
                    auto put = [&](int y, T sgn) {
                        T *d = row + (y >> 3) * PG + (y & 7);
                        d[0] = K[0];
                        if constexpr (NC == 2) d[(size_t)rowg * PG] = sgn * K[1];
                    };
                    if (!whole) {
                        put(v, T(1));
                        continue;
                    }
                    // x = -q and x = +q (where K_phi changes sign), every period
                    // (jb < nphi and TJ < nphi + 8, so x0 > -2 nphi - 8)
                    for (int x = -q; x >= x0; x -= nphi)
                        if (x < x0 + wn) put(x - x0, T(1));
                    for (int x = -q + nphi; x < x0 + wn; x += nphi)
                        if (x >= x0) put(x - x0, T(1));
                    for (int x = q; x >= x0; x -= nphi)
                        if (x < x0 + wn) put(x - x0, T(-1));
                    for (int x = q + nphi; x < x0 + wn; x += nphi)
                        if (x >= x0) put(x - x0, T(-1));
                }
                for (int e = threadIdx.x; e < P.KS * lpad; e += 256) {
                    const int s = e / lpad, l = e - s * lpad;
                    M[s * P.TL + l] =
                        (k0 + s < r1 && l < tl) ? A.mass[a * A.N + (int64_t)(k0 + s) * nphi + l0 + l] : T(0);
                }
                __syncthreads();
                if (!act) continue;
                const T *dr = D + (size_t)ks * NC * rowg * PG + (P.JT - jt) * PG, *mr = M + ks * P.TL;
                const int ng = lpad / 8;
                for (int c0 = 8 * lg; c0 < ng; c0 += 8 * P.LG) {
                    T part[NC][8], prev[NC][8];
#pragma unroll
                    for (int c = 0; c < NC; ++c)
#pragma unroll
                        for (int r = 0; r < 8; ++r) {
                            part[c][r] = T(0);
                            prev[c][r] = dr[(size_t)c * rowg * PG + (c0 - 1) * PG + r];
                        }
                    const int c1 = min(ng, c0 + 8);
                    for (int cg = c0; cg < c1; ++cg) {
                        T m[8];
#pragma unroll
                        for (int i = 0; i < 8; ++i) m[i] = mr[8 * cg + i];
#pragma unroll
                        for (int c = 0; c < NC; ++c) {
                            T cur[8];
#pragma unroll
                            for (int i = 0; i < 8; ++i) cur[i] = dr[(size_t)c * rowg * PG + cg * PG + i];
#pragma unroll
                            for (int i = 0; i < 8; ++i)
#pragma unroll
                                for (int r = 0; r < 8; ++r)
                                    part[c][r] += m[i] * (i >= r ? cur[i - r] : prev[c][8 + i - r]);
#pragma unroll
                            for (int i = 0; i < 8; ++i) prev[c][i] = cur[i];
                        }
                    }
#pragma unroll
                    for (int c = 0; c < NC; ++c)
#pragma unroll
                        for (int r = 0; r < 8; ++r) sg_two_sum_acc(acc[c][r], err[c][r], part[c][r]);
                }
            }
    // the groups' sums, added in group order, one component after the other:
    // red[group][jt][sum, error][8]
    T *red = (T *)smem;
    const int ngr = P.KS * P.LG;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        __syncthreads();
        if (act) {
            T *o = red + (size_t)(g * P.JT + jt) * 16;
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                o[r] = acc[c][r];
                o[8 + r] = err[c][r];
            }
        }
        __syncthreads();
        for (int j = threadIdx.x; j < 8 * P.JT; j += 256) {
            if (jb + j >= nphi) continue;
            T sum = T(0), er = T(0);
            for (int q = 0; q < ngr; ++q) {
                const T *o = red + (size_t)(q * P.JT + (j >> 3)) * 16 + (j & 7);
                sg_two_sum_acc(sum, er, o[0]);
                er += o[8];
            }
            T *o = A.partial + ((int64_t)(blockIdx.y * nf + b) * 2 * NC + 2 * c) * A.N + (int64_t)ir * nphi + jb + j;
            o[0] = sum;
            o[A.N] = er;
        }
    }
}

// Indirect term (SG_INDIRECT; Sect. 5.4 and the appendix "Indirect term"):
//   A + i B = sum_a sqrt(2) sum_k Sigma_a[k] A_k K_a(d_k) e^{i phi_k},
//   K_a(d) = pi^{-1/2} H_a^{-2} (d/4) F(d^2/4),  d_k = r_k / H_a[k],
// in double for both precisions (a reduction over the cells, like the self
// term).  Block b sums a fixed strided set of cells and the blocks' sums are
// added in order by one thread, so the result is deterministic.
#define SG_IND_BLOCKS 1024
template <typename T>
__global__ void __launch_bounds__(256) k_indirect_part(int nr, int nphi, int nf, double lnrmin, double du,
                                                       double dphi, const double *h, const T *sigma,
                                                       const T *H, double2 *part, int lin, double rmin,
                                                       double dr)
{
    __shared__ __attribute__((aligned(16))) double wq[FQuad<double>::TABLE];
    __shared__ double ra[256], rb[256];
    sg_fill64(wq, SG_FN_F);
    __syncthreads();
    const int64_t N = (int64_t)nr * nphi, total = nf * N;
    double sa = 0.0, sb = 0.0;
    for (int64_t k = blockIdx.x * (int64_t)256 + threadIdx.x; k < total; k += (int64_t)gridDim.x * 256) {
        const int a = (int)(k / N);
        const int64_t cell = k % N;
        const int ir = (int)(cell / nphi), j = (int)(cell % nphi);
        const double r = dir_radius(lin, lnrmin, du, rmin, dr, ir);
        const double Hk = H ? (double)H[k] : h[a] * r;
        const double d = r / Hk;
        const double Ka = 1.0 / (SG_SQRT_PI * Hk * Hk) * (0.25 * d) * sg_F64(0.25 * d * d, wq);
        const double w = SG_SQRT2 * (double)sigma[k] * (lin ? r * dr : r * r * du) * dphi * Ka;
        double sp, cp;
        sincos((j + 0.5) * dphi, &sp, &cp);
        sa += w * cp;
        sb += w * sp;
    }
    ra[threadIdx.x] = sa;
    rb[threadIdx.x] = sb;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (threadIdx.x < o) {
            ra[threadIdx.x] += ra[threadIdx.x + o];
            rb[threadIdx.x] += rb[threadIdx.x + o];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = make_double2(ra[0], rb[0]);
}

__global__ void k_indirect_fin(const double2 *part, int n, double2 *AB)
{
    if (threadIdx.x != 0) return;
    double a = 0.0, b = 0.0;
    for (int i = 0; i < n; ++i) {
        a += part[i].x;
        b += part[i].y;
    }
    *AB = make_double2(a, b);
}

// self: per pair (log grid, H = h r), per cell (percell = 1) or, on a
// uniform grid without per-cell H, per ring (percell = 2); the own-cell
// values are cell averages per (du dphi), or per (dr / r_i) dphi on a
// uniform grid (lin; rmin, dr give r_i).
template <typename T, int NF>
__global__ void k_direct_reduce(const T *partial, int S, int64_t N, const double *self,
                                int percell, int with_self, const T *sigma, double dudphi,
                                const double2 *ind, int nphi, T *gr, T *gp, int lin, double rmin, double dr)
{
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (t >= N) return;
    double ir = 0.0, ip = 0.0;  // indirect acceleration at this cell (all targets)
    if (ind) {
        const double2 AB = *ind;
        double sp, cp;
        sincos(((double)(t % nphi) + 0.5) * (2.0 * SG_PI / nphi), &sp, &cp);
        ir = -(AB.x * cp + AB.y * sp);
        ip = -(-AB.x * sp + AB.y * cp);
    }
#pragma unroll
    for (int b = 0; b < NF; ++b) {
        // the splits' (sum, carried error) pairs, added in double in a fixed
        // order (compensated, so the double pass adds no error of its own
        // that matters for either precision)
        double sr = 0.0, er = 0.0, sp = 0.0, ep = 0.0;
        for (int s = 0; s < S; ++s) {
            const T *pp = partial + (int64_t)(s * NF + b) * 4 * N + t;
            sg_two_sum_acc(sr, er, (double)pp[0]);
            sg_two_sum_acc(sr, er, (double)pp[N]);
            sg_two_sum_acc(sp, ep, (double)pp[2 * N]);
            sg_two_sum_acc(sp, ep, (double)pp[3 * N]);
        }
        sr += er;
        sp += ep;
        if (with_self) {
            const int ir = (int)(t / nphi);
            const double w = lin ? dr / (rmin + (ir + 0.5) * dr) * (2.0 * SG_PI / nphi) : dudphi;
            const int64_t nring = N / nphi;
            double st = 0.0;
#pragma unroll
            for (int a = 0; a < NF; ++a) {
                const int pair = a * NF + b;
                const double kb = percell == 1   ? self[(int64_t)pair * N + t]
                                  : percell == 2 ? self[(int64_t)pair * nring + ir]
                                                 : self[pair];
                st -= w * (double)sigma[a * N + t] * kb;
            }
            sr += st;
        }
        if (ind) {
            sr += ir;
            sp += ip;
        }
        gr[b * N + t] = (T)sr;
        gp[b * N + t] = (T)sp;
    }
}

// --------------------------------------------------------------- potential
// Conservative potential (Sect. 5.5, appendix "Conservative force"):
//   Phi_b(i) = sum_a sum_{k != i} Sigma_a[k] A_k P_ab(s_ik),
//   P_ab(s) = -e^y K0(y) / (2 sqrt(pi) H_ab),  y = s^2/(8 H_ab^2),
// H_ab from the source cell's H_a and the target cell's H_b; the own cell
// adds Sigma_a[i] times the cell integral of P_ab (k_pot_cells).  Same
// layout and splitting as the field sum; one accumulator per target fluid.
template <typename T, int NF>
__global__ void __launch_bounds__(256) k_potential(DirectArgs<T> A)
{
    __shared__ __attribute__((aligned(16))) T wq[FQuad<T>::TABLE];
    sg_fill_v(wq, SG_FN_VG);
    __syncthreads();
    const int64_t t = blockIdx.x * (int64_t)256 + threadIdx.x;
    if (t >= A.N) return;
    const int nphi = A.nphi, nr = A.nr;
    const int ir = (int)(t / nphi), j = (int)(t % nphi);
    const T ri = A.rrow[ir];
    T hb2[NF], acc[NF], err[NF];
#pragma unroll
    for (int b = 0; b < NF; ++b) {
        hb2[b] = A.H2[b * A.N + t];
        acc[b] = T(0);
        err[b] = T(0);
    }
    const int r0 = blockIdx.y * A.rps;
    const int r1 = min(nr, r0 + A.rps);
    for (int kr = r0; kr < r1; ++kr) {
        const int p = ir - kr + nr - 1;
        const T SX = A.sx[p];
        const T rr8 = ri * A.rrow[kr] * T(0.125);
        const int64_t kbase = (int64_t)kr * nphi;
        for (int l0 = 0; l0 < nphi; l0 += SG_DCHUNK) {
            const int l1 = min(nphi, l0 + SG_DCHUNK);
            T pc[NF];  // this chunk's partial sums
#pragma unroll
            for (int b = 0; b < NF; ++b) pc[b] = T(0);
            for (int l = l0; l < l1; ++l) {
                const int64_t k = kbase + l;
                int q = j - l;
                q += q < 0 ? nphi : 0;
                const bool self = (k == t);
                const T rs = sg_rsqrt(self ? T(1) : rr8 * (SX + A.sph[q])), rs2 = rs * rs;  // s^2 / 8
#pragma unroll
                for (int b = 0; b < NF; ++b) {
                    const T ub = hb2[b] * rs2;
                    T c = T(0);
#pragma unroll
                    for (int a = 0; a < NF; ++a)
                        c += A.mass[a * A.N + k] * sg_v<SG_FN_VG>(A.H2[a * A.N + k] * rs2 + ub, wq);
                    pc[b] += c * (self ? T(0) : rs);
                }
            }
#pragma unroll
            for (int b = 0; b < NF; ++b) sg_two_sum_acc(acc[b], err[b], pc[b]);
        }
    }
#pragma unroll
    for (int b = 0; b < NF; ++b) {
        T *o = A.partial + (int64_t)(blockIdx.y * NF + b) * 2 * A.N + t;
        o[0] = acc[b];
        o[A.N] = err[b];
    }
}

template <typename T, int NF>
__global__ void k_potential_reduce(const T *partial, int S, int64_t N, int nphi, const double *self,
                                   int per_row, int with_self, const T *sigma, T *pot, double unit)
{
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (t >= N) return;
    const int64_t si = per_row ? t / nphi : t;
    const int64_t per = per_row ? N / nphi : N;
#pragma unroll
    for (int b = 0; b < NF; ++b) {
        double sum = 0.0, e = 0.0;
        for (int s = 0; s < S; ++s) {
            const T *pp = partial + (int64_t)(s * NF + b) * 2 * N + t;
            sg_two_sum_acc(sum, e, (double)pp[0]);
            sg_two_sum_acc(sum, e, (double)pp[N]);
        }
        sum = (sum + e) * unit;
        if (with_self) {
            double st = 0.0;
#pragma unroll
            for (int a = 0; a < NF; ++a) st += (double)sigma[a * N + t] * self[(int64_t)(a * NF + b) * per + si];
            sum += st;
        }
        pot[b * N + t] = (T)sum;
    }
}

// -------------------------------------------- self-gravitating scale heights
// H_f^sg = sqrt(2/pi) H_f f(Qt), Qt = (sum_f 1/Q_f)^-1 (Sect. 2.1), with
// f(x) = pi/(4x) [sqrt(1 + 8x^2/pi) - 1] evaluated as the equal
// 2x / (sqrt(1 + 8x^2/pi) + 1), which does not cancel at small x.
__global__ void k_hsg(int64_t n, int nf, const double *H, const double *Q, double *Hsg)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        double inv = 0.0;
        for (int f = 0; f < nf; ++f) inv += 1.0 / Q[f * n + i];
        const double x = 1.0 / inv;
        const double fx = 2.0 * x / (sqrt(1.0 + 8.0 * x * x / SG_PI) + 1.0);
        for (int f = 0; f < nf; ++f) Hsg[f * n + i] = sqrt(2.0 / SG_PI) * H[f * n + i] * fx;
    }
}

sg_status sg_hsg_launch(int64_t n, int nf, const double *H, const double *Q, double *Hsg, hipStream_t s)
{
    int64_t nb = (n + 255) / 256;
    if (nb > 65536) nb = 65536;
    hipLaunchKernelGGL(k_hsg, dim3((unsigned)nb), dim3(256), 0, s, n, nf, H, Q, Hsg);
    SG_HIP(hipGetLastError());
    return SG_OK;
}

// ------------------------------------------------------------------- host
static int direct_splits(int nr, int64_t N)
{
    const int64_t gx = (N + 255) / 256;
    int64_t S = (2048 + gx - 1) / gx;
    if (S < 1) S = 1;
    if (S > nr) S = nr;
    const int rps = (int)((nr + S - 1) / S);
    return (nr + rps - 1) / rps;
}

size_t sg_direct_ws_bytes(int nr, int nphi, int nf, sg_dtype dt, int percell)
{
    const size_t es = dt == SG_F64 ? 8 : 4;
    const int64_t N = (int64_t)nr * nphi;
    const int S = direct_splits(nr, N);
    size_t o = 0;
    o += sg_align256(es * nr);
    o += 2 * sg_align256(es * (2 * (size_t)nr - 1));
    o += 2 * sg_align256(es * nphi);
    o += 2 * sg_align256(es * nf * N);
    o += sg_align256(sizeof(double) * nf * nf * (percell ? N : nr));
    o += sg_align256(es * (size_t)S * nf * 4 * N);
    o += sg_align256(sizeof(double) * 4);
    o += sg_align256(sizeof(double2) * (SG_IND_BLOCKS + 1));
    return o;
}

// H = h r sums by the general kernels (one pair of cells at a time) on many
// rings of few azimuths: a ring pair then has fewer terms than the 8 x 8 step of
// the ring sums, whose staging is left (a barrier per KS rings of few
// evaluations).  Ring sums / general kernels in us, one fluid: field in float
// 6000 x 1 3010 / 163, 1000 x 6 193 / 150, 750 x 8 108 / 109; in double 6000 x 1
// 4190 / 265, 1000 x 5 267 / 217, 1000 x 6 226 / 220 (four fluids 1640 / 1920);
// potential 6000 x 1 1500 / 490, 1500 x 4 382 / 355, 4000 x 5 1240 / 1300.  On
// fewer rings the general kernels' chains are the longer ones: 1000 x 1 213 /
// 257, 250 x 4 91 / 162, potential 1000 x 1 247 / 349; four fluids 500 x 1 545 /
// 815, 900 x 1 1390 / 787.
template <typename T, int NC> static bool few_azimuths(int nr, int nphi, int nf)
{
    const int rings = NC == 1 ? 1500 : nphi == 1 ? 1100 - 100 * nf : 1000;
    return nr >= rings && nphi < (NC == 1 ? 5 : sizeof(T) == 8 ? 6 : 8);
}

// H = h r: the ring sums into at most smax splits; returns the splits used.
template <typename T, int NC> static int ring_sum(const DirectArgs<T> &A, int nf, int smax, hipStream_t s)
{
    const RingShape P = ring_shape<T, NC>(A.nr, A.nphi, nf, smax);
    const int S = (A.nr + P.rps - 1) / P.rps;
    hipLaunchKernelGGL((k_ring_sum<T, NC>), dim3((unsigned)(A.nr * P.ntile), (unsigned)S, (unsigned)nf), dim3(256),
                       (unsigned)P.lds, s, A, P, nf);
    return S;
}

template <typename T>
static sg_status direct_run(const sg_grid *g, int nf, const double *h, const T *sigma, const T *H,
                            T *gr, T *gp, uint32_t flags, void *ws, hipStream_t s)
{
    const int nr = g->n_r, nphi = g->n_phi;
    const int64_t N = (int64_t)nr * nphi;
    const double du = log(g->r_max / g->r_min) / nr;
    const double dphi = 2.0 * SG_PI / nphi;
    const double lnrmin = log(g->r_min), unit = length_unit<T>(*g);
    const int lin = (flags & SG_LINEAR_R) ? 1 : 0;
    const double dr = (g->r_max - g->r_min) / nr;
    int S = direct_splits(nr, N);
    const int rps = (nr + S - 1) / S;
    char *o = (char *)ws;
    auto take = [&](size_t bytes) {
        char *p = o;
        o += sg_align256(bytes);
        return p;
    };
    T *rrow = (T *)take(sizeof(T) * nr);
    T *sx = (T *)take(sizeof(T) * (2 * (size_t)nr - 1));
    T *ex = (T *)take(sizeof(T) * (2 * (size_t)nr - 1));
    T *sph = (T *)take(sizeof(T) * nphi);
    T *snp = (T *)take(sizeof(T) * nphi);
    T *mass = (T *)take(sizeof(T) * nf * N);
    T *H2 = (T *)take(sizeof(T) * nf * N);
    const int percell = H != nullptr;
    const bool by_cell = percell || few_azimuths<T, 2>(nr, nphi, nf);
    double *self = (double *)take(sizeof(double) * nf * nf * (percell ? N : nr));
    T *partial = (T *)take(sizeof(T) * (size_t)S * nf * 4 * N);
    // uniform grid: double H for the own-cell integrals, per cell or per ring,
    // in the partial-sum buffer (at least nf N doubles; written before the sum)
    double *Hd = (double *)partial;
    double *dh = (double *)take(sizeof(double) * 4);
    double2 *ipart = (double2 *)take(sizeof(double2) * (SG_IND_BLOCKS + 1));
    double2 *iab = ipart + SG_IND_BLOCKS;

    // h lives on the host: pass through a kernel argument copy in device memory
    // is avoided by writing it with a fill kernel.
    for (int f = 0; f < nf; ++f) hipLaunchKernelGGL(k_fill_f64, dim3(1), dim3(64), 0, s, dh + f, (int64_t)1, h[f]);
    SG_HIP(hipGetLastError());
    {
        int64_t work = nf * N > 2 * nr ? nf * N : 2 * nr;
        if (work < nphi) work = nphi;
        int64_t nb = (work + 255) / 256;
        if (nb > 65536) nb = 65536;
        hipLaunchKernelGGL(k_direct_prep<T>, dim3((unsigned)nb), dim3(256), 0, s, nr, nphi, nf,
                           log(g->r_min / unit), du, dphi, (const double *)dh, sigma, H, rrow, sx, ex, sph, snp,
                           mass, H2, lin, g->r_min / unit, dr / unit, Hd, by_cell ? 1 : 0, unit);
        SG_HIP(hipGetLastError());
    }
    const int with_self = !(flags & SG_SELF_CELL_EXCLUDE);
    if (with_self) {
        GLNodes gl;
        sg_gl_nodes(gl, lin ? sg_lin_aspect(*g, dphi) : du / dphi);
        if (lin) {
            const int per = percell ? nphi : 1;
            const int64_t items = (int64_t)nf * nf * nr * per;
            hipLaunchKernelGGL(k_ss_self_lin, dim3((unsigned)items), dim3(256), 0, s, (const double *)Hd, nf, nr,
                               per, g->r_min, dr, dphi, 0, 0, self, gl);
        } else if (percell) {
            sg_self_cells<T>(H, nf, nr, nphi, lnrmin, du, dphi, self, s);
        } else {
            SelfItems it{};
            for (int a = 0; a < nf; ++a)
                for (int b = 0; b < nf; ++b) {
                    it.ha[a * nf + b] = h[a];
                    it.hb[a * nf + b] = h[b];
                    it.which[a * nf + b] = 0;
                }
            hipLaunchKernelGGL(k_self_cell, dim3(nf * nf), dim3(256), 0, s, it, self, du, dphi, gl);
        }
        SG_HIP(hipGetLastError());
    }
    const bool ind = (flags & SG_INDIRECT) != 0;
    if (ind) {
        int64_t nb = (nf * N + 255) / 256;
        if (nb > SG_IND_BLOCKS) nb = SG_IND_BLOCKS;
        hipLaunchKernelGGL(k_indirect_part<T>, dim3((unsigned)nb), dim3(256), 0, s, nr, nphi, nf, lnrmin,
                           du, dphi, (const double *)dh, sigma, H, ipart, lin, g->r_min, dr);
        hipLaunchKernelGGL(k_indirect_fin, dim3(1), dim3(64), 0, s, (const double2 *)ipart, (int)nb, iab);
        SG_HIP(hipGetLastError());
    }
    DirectArgs<T> A;
    A.nr = nr;
    A.nphi = nphi;
    A.rps = rps;
    A.lin = lin;
    A.dr = (T)(dr / unit);
    A.N = N;
    A.rrow = rrow;
    A.sx = sx;
    A.ex = ex;
    A.sph = sph;
    A.snp = snp;
    A.mass = mass;
    A.H2 = H2;
    A.partial = partial;
    if (by_cell) {
        dim3 grid((unsigned)((N + 255) / 256), (unsigned)S);
        switch (nf) {
        case 1: hipLaunchKernelGGL((k_direct<T, 1>), grid, dim3(256), 0, s, A); break;
        case 2: hipLaunchKernelGGL((k_direct<T, 2>), grid, dim3(256), 0, s, A); break;
        case 3: hipLaunchKernelGGL((k_direct<T, 3>), grid, dim3(256), 0, s, A); break;
        default: hipLaunchKernelGGL((k_direct<T, 4>), grid, dim3(256), 0, s, A); break;
        }
    } else {
        S = ring_sum<T, 2>(A, nf, S, s);
    }
    SG_HIP(hipGetLastError());
    const unsigned nb = (unsigned)((N + 255) / 256);
    const double2 *indp = ind ? (const double2 *)iab : nullptr;
    const int smode = percell ? 1 : (lin ? 2 : 0);
#define SG_RED(NF)                                                                                      \
    hipLaunchKernelGGL((k_direct_reduce<T, NF>), dim3(nb), dim3(256), 0, s, partial, S, N, self, smode,    \
                       with_self, sigma, du * dphi, indp, nphi, gr, gp, lin, g->r_min, dr)
    switch (nf) {
    case 1: SG_RED(1); break;
    case 2: SG_RED(2); break;
    case 3: SG_RED(3); break;
    default: SG_RED(4); break;
    }
#undef SG_RED
    SG_HIP(hipGetLastError());
    return SG_OK;
}

size_t sg_potential_ws_bytes(int nr, int nphi, int nf, sg_dtype dt, int percell)
{
    const size_t es = dt == SG_F64 ? 8 : 4;
    const int64_t N = (int64_t)nr * nphi;
    const int S = direct_splits(nr, N);
    size_t o = 0;
    o += sg_align256(es * nr);
    o += 2 * sg_align256(es * (2 * (size_t)nr - 1));
    o += 2 * sg_align256(es * nphi);
    o += 2 * sg_align256(es * nf * N);
    o += sg_align256(sizeof(double) * nf * nf * (percell ? N : nr));
    o += sg_align256(es * (size_t)S * nf * 2 * N);
    o += sg_align256(sizeof(double) * 4);
    return o;
}

template <typename T>
static sg_status potential_run(const sg_grid *g, int nf, const double *h, const T *sigma, const T *H,
                               T *pot, uint32_t flags, void *ws, hipStream_t s)
{
    const int nr = g->n_r, nphi = g->n_phi;
    const int64_t N = (int64_t)nr * nphi;
    const double du = log(g->r_max / g->r_min) / nr;
    const double dphi = 2.0 * SG_PI / nphi;
    const double lnrmin = log(g->r_min), unit = length_unit<T>(*g);
    int S = direct_splits(nr, N);
    const int rps = (nr + S - 1) / S;
    char *o = (char *)ws;
    auto take = [&](size_t bytes) {
        char *p = o;
        o += sg_align256(bytes);
        return p;
    };
    T *rrow = (T *)take(sizeof(T) * nr);
    T *sx = (T *)take(sizeof(T) * (2 * (size_t)nr - 1));
    T *ex = (T *)take(sizeof(T) * (2 * (size_t)nr - 1));
    T *sph = (T *)take(sizeof(T) * nphi);
    T *snp = (T *)take(sizeof(T) * nphi);
    T *mass = (T *)take(sizeof(T) * nf * N);
    T *H2 = (T *)take(sizeof(T) * nf * N);
    const int percell = H != nullptr;
    const bool by_cell = percell || few_azimuths<T, 1>(nr, nphi, nf);
    double *self = (double *)take(sizeof(double) * nf * nf * (percell ? N : nr));
    T *partial = (T *)take(sizeof(T) * (size_t)S * nf * 2 * N);
    double *dh = (double *)take(sizeof(double) * 4);
    for (int f = 0; f < nf; ++f)
        hipLaunchKernelGGL(k_fill_f64, dim3(1), dim3(64), 0, s, dh + f, (int64_t)1, h ? h[f] : 0.0);
    SG_HIP(hipGetLastError());
    {
        int64_t work = nf * N > 2 * nr ? nf * N : 2 * nr;
        if (work < nphi) work = nphi;
        int64_t nb = (work + 255) / 256;
        if (nb > 65536) nb = 65536;
        hipLaunchKernelGGL(k_direct_prep<T>, dim3((unsigned)nb), dim3(256), 0, s, nr, nphi, nf,
                           log(g->r_min / unit), du, dphi, (const double *)dh, sigma, H, rrow, sx, ex, sph, snp,
                           mass, H2, 0, 0.0, 0.0, nullptr, by_cell ? 2 : 0, unit);
        SG_HIP(hipGetLastError());
    }
    const int with_self = !(flags & SG_SELF_CELL_EXCLUDE);
    if (with_self) {
        sg_pot_cells<T>(H, (const double *)dh, nf, nr, nphi, lnrmin, du, dphi, percell ? 0 : 1, self, 0, s);
        SG_HIP(hipGetLastError());
    }
    DirectArgs<T> A;
    A.lin = 0;
    A.dr = T(0);
    A.nr = nr;
    A.nphi = nphi;
    A.rps = rps;
    A.N = N;
    A.rrow = rrow;
    A.sx = sx;
    A.ex = ex;
    A.sph = sph;
    A.snp = snp;
    A.mass = mass;
    A.H2 = H2;
    A.partial = partial;
    if (by_cell) {
        dim3 grid((unsigned)((N + 255) / 256), (unsigned)S);
        switch (nf) {
        case 1: hipLaunchKernelGGL((k_potential<T, 1>), grid, dim3(256), 0, s, A); break;
        case 2: hipLaunchKernelGGL((k_potential<T, 2>), grid, dim3(256), 0, s, A); break;
        case 3: hipLaunchKernelGGL((k_potential<T, 3>), grid, dim3(256), 0, s, A); break;
        default: hipLaunchKernelGGL((k_potential<T, 4>), grid, dim3(256), 0, s, A); break;
        }
    } else {
        S = ring_sum<T, 1>(A, nf, S, s);
    }
    SG_HIP(hipGetLastError());
    const unsigned nb = (unsigned)((N + 255) / 256);
#define SG_PRED(NF)                                                                                      \
    hipLaunchKernelGGL((k_potential_reduce<T, NF>), dim3(nb), dim3(256), 0, s, partial, S, N, nphi, self, \
                       percell ? 0 : 1, with_self, sigma, pot, unit)
    switch (nf) {
    case 1: SG_PRED(1); break;
    case 2: SG_PRED(2); break;
    case 3: SG_PRED(3); break;
    default: SG_PRED(4); break;
    }
#undef SG_PRED
    SG_HIP(hipGetLastError());
    return SG_OK;
}

sg_status sg_potential_launch(const sg_grid *g, int nf, const double *h, const void *sigma,
                              const void *H, void *pot, sg_dtype dt, uint32_t flags, void *ws,
                              hipStream_t s)
{
    if (dt == SG_F64)
        return potential_run<double>(g, nf, h, (const double *)sigma, (const double *)H, (double *)pot,
                                     flags, ws, s);
    return potential_run<float>(g, nf, h, (const float *)sigma, (const float *)H, (float *)pot, flags,
                                ws, s);
}

sg_status sg_direct_launch(const sg_grid *g, int nf, const double *h, const void *sigma,
                           const void *H, void *gr, void *gp, sg_dtype dt, uint32_t flags,
                           void *ws, hipStream_t s)
{
    if (dt == SG_F64)
        return direct_run<double>(g, nf, h, (const double *)sigma, (const double *)H, (double *)gr,
                                  (double *)gp, flags, ws, s);
    return direct_run<float>(g, nf, h, (const float *)sigma, (const float *)H, (float *)gr,
                             (float *)gp, flags, ws, s);
}
