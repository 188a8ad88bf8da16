// sg_fftpath.hip -- sg_field_fft: batched three-pass log-polar FFT
// convolution, one cached plan per batch signature (run from a captured HIP
// graph when a pass has several launch classes, else enqueued directly).
#include <algorithm>
#include <cstddef>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <tuple>
#include <map>
#include <memory>
#include <mutex>
#include <vector>

#include <hip/hip_ext.h>

#include "sg_fftpath.h"
#include "sg_semispec.h"
#include "sg_passes.h"

// ---------------------------------------------------------------- kernels
// Workgroup b takes workgroup job w = sg_xcd_remap(b, K); gridDim.x is a
// multiple of 8 K (a whole number of XCD clusters of K consecutive workgroup
// jobs).  Twiddles depend only on the transform length, so one table serves
// every disc of a launch.  SF selects the radix order of the transforms
// (small radix first); SF and K are tuning parameters.
//
// Passes 1 and 3 give each workgroup whole row quads and move the
// intermediates tile by tile (sg_blk_index): elements 2l and 2l+1 of a tile
// are one 16-byte access, 8 lanes cover a tile, and the values are exchanged
// with the transforms through each group's LDS plane.

// Pass 1: group g takes job base + g = (fluid f, row pair j): rows 2j and
// 2j + 1 of fluid f as the real and imaginary parts of one complex transform.
// Two jobs fill a row quad, so a workgroup has G >= 2 groups (even).
// Padding rows (row counts below 4) read the last real row.
template <int N, int GM> struct P1Shape {
    static constexpr int P = FftShape<N>::P, T = FftShape<N>::T;
    static constexpr int G = GM * (256 / T > 2 ? 256 / T : 2);
    static constexpr int WGS = G * T;
    static constexpr int K = 1;
};

template <int N, int NF, bool SF, int GM>
__global__ void __launch_bounds__((P1Shape<N, GM>::WGS))
k_pass1(const DiscDev *discs, const WJob *wj, int nj, const float2 *twp, int kc, OneDisc one)
{
    using S = P1Shape<N, GM>;
    constexpr int P = S::P, T = S::T, G = S::G, W = LdsPlane<float>::elems(N);
    constexpr int NG = (N / 2 + 1 + 3) / 4;  // column groups (tiles per row quad)
    __shared__ __attribute__((aligned(16))) float2 lds[W * G];
    const int g = threadIdx.x / T, t = threadIdx.x % T;
    const int w = sg_uniform(sg_xcd_remap(blockIdx.x, kc));
    if (w >= nj) return;
    DiscDev D;
    const WJob job = pass_job<1>(discs, wj, one, w, G, D);
    const int cb = job.base, cn = job.n;
    const int nr = D.nr, half = sg_blk_rows(nr) / 2;  // row pairs per fluid
    const LdsPlane<float> pl{lds + W * g};
    TwRegC<N, SF> tw;
    tw.load(twp, t);
    // 1. two real rows as one complex transform (with species: the sum of
    //    the group's species rows, in species order)
    float2 z[P];
    {
        const int idx = g < cn ? cb + g : cb;
        const int f = idx / half, j = idx % half;
        const uint32_t r1 = (uint32_t)min(2 * j, nr - 1) * N + t;
        const uint32_t r2 = (uint32_t)min(2 * j + 1, nr - 1) * N + t;
        if (sg_uniform(D.ns) == 0) {
            const uint32_t o = (uint32_t)f * nr * N;
#pragma unroll
            for (int p = 0; p < P; ++p)
                z[p] = make_float2(gld1(D.sigma, o + r1 + T * p), gld1(D.sigma, o + r2 + T * p));
        } else {
#pragma unroll
            for (int p = 0; p < P; ++p) z[p] = make_float2(0.f, 0.f);
            const DiscDev *sp = discs + job.disc;
            const int cnt = sp->gcount[f];
            for (int k = 0; k < cnt; ++k) {
                const uint32_t o = (uint32_t)sp->gsp[f][k] * nr * N;
#pragma unroll
                for (int p = 0; p < P; ++p) {
                    z[p].x += gld1(D.sigma, o + r1 + T * p);
                    z[p].y += gld1(D.sigma, o + r2 + T * p);
                }
            }
        }
    }
    fft<N, false>(z, t, pl, tw);
#pragma unroll
    for (int p = 0; p < P; ++p) pl.st(t + T * p, z[p]);
    __syncthreads();
    // 2. Hermitian split in place: slot m <- X1[m], slot N - m <- X2[m]
    //    (0 < m < N/2); slots 0 and N/2 keep Z = X1 + i X2 (both real there)
#pragma unroll
    for (int p = 0; p < P / 2; ++p) {
        const int m = t + T * p;
        if (m == 0) continue;
        const float2 Z = pl.ld(m), C = pl.ld(N - m);
        pl.st(m, make_float2(0.5f * (Z.x + C.x), 0.5f * (Z.y - C.y)));
        pl.st(N - m, make_float2(0.5f * (Z.y + C.y), -0.5f * (Z.x - C.x)));
    }
    __syncthreads();
    // 3. tile stores: row quad k of the workgroup = jobs cb + 2k, cb + 2k + 1
    //    (one fluid); its row r comes from group 2k + r/2, X1 (r even) or X2
    const size_t fs = sg_blk_field_elems(N, nr);
    for (int e = threadIdx.x; e < (G / 2) * NG * 8; e += S::WGS) {
        const int k = e / (NG * 8), q = (e / 8) % NG, l = e & 7;
        if (2 * k >= cn) continue;
        const int j0 = cb + 2 * k;
        const int f = j0 / half, i0 = 2 * (j0 % half);
        const int c = 4 * q + (l >> 1), r0 = 2 * (l & 1);
        // rows r0 and r0 + 1: X1 and X2 of group 2k + r0/2
        const LdsPlane<float> X{lds + W * (2 * k + (r0 >> 1))};
        float2 v0 = make_float2(0.f, 0.f), v1 = make_float2(0.f, 0.f);
        if (c == 0 || c == N / 2) {
            const float2 Z = X.ld(c);
            v0 = make_float2(Z.x, 0.f);
            v1 = make_float2(Z.y, 0.f);
        } else if (c < N / 2) {
            v0 = X.ld(c);
            v1 = X.ld(N - c);
        } else if (c == N / 2 + 1) {
            // spare slot: the real columns 0 and N/2 packed as X[0] + i X[N/2]
            // (pass 2 transforms them as one column)
            const float2 Z0 = X.ld(0), ZN = X.ld(N / 2);
            v0 = make_float2(Z0.x, ZN.x);
            v1 = make_float2(Z0.y, ZN.y);
        }
        gst2x2(D.st + f * fs + sg_blk_tile(q, i0, nr) + 2 * l, v0, v1);
    }
}

// Pass 2 launch shape: a column is carried by NF * T threads; for two fluids
// the two halves each own one fluid (forward transform of that source fluid,
// then spectral multiply and inverse transforms for that target fluid), so
// no thread holds more than one fluid's accumulators.
template <int NU, int NF, int GM> struct P2Shape {
    static constexpr int P = FftShape<NU>::P, T = FftShape<NU>::T;
    static constexpr int CT = NF * T;
    static constexpr int G = GM * (256 / CT > 1 ? 256 / CT : 1);
    static constexpr int WGS = G * CT;
    static constexpr int K = G >= 4 ? 1 : 4 / G;
};

// Loads of pass-2 column job m for half h: Sigma~_h at rows t + T p (p < P/2;
// the upper half of the padded column is zero) and the unique kernel-spectrum
// values K(k_lo), k_lo = t + T j (j < P/2), and K(NU/2) of every source a.
// Job 0 is the pair of the real columns 0 and n_phi/2: pass 1 stores their
// packed Sigma~[0] + i Sigma~[n_phi/2] in column slot n_phi/2 + 1, and the
// table holds (K0 + KN)/2 and (K0 - KN)/2 (K_r of the two columns) in that
// slot's K_r and K_phi places, so the job loads from slot n_phi/2 + 1.
template <int NU>
__device__ inline void p2_load_sh(const DiscDev &D, int m, int h, int t, float2 (&sh)[FftShape<NU>::P / 2])
{
    constexpr int P = FftShape<NU>::P, T = FftShape<NU>::T, H = P / 2, NR = NU / 2;
    const uint32_t fs = (uint32_t)sg_blk_field_elems(D.nphi, NR);
#pragma unroll
    for (int p = 0; p < H; ++p) sh[p] = gld2(D.st, h * fs + (uint32_t)sg_blk_index(m, t + T * p, NR));
}

// spectra of source a for target h
template <int NU, int NF>
__device__ inline void p2_load_k(const DiscDev &D, int m, int a, int h, int t, float2 (&K)[2][FftShape<NU>::P / 2],
                                 float2 (&KN)[2])
{
    constexpr int P = FftShape<NU>::P, T = FftShape<NU>::T, H = P / 2, NR = NU / 2;
    constexpr uint32_t kk = NR + 1;
#pragma unroll
    for (int cc = 0; cc < 2; ++cc) {
        const uint32_t o = (((uint32_t)m * (NF * NF) + a * NF + h) * 2 + cc) * kk;
#pragma unroll
        for (int j = 0; j < H; ++j) K[cc][j] = gld2(D.spec, o + t + T * j);
        KN[cc] = gld2(D.spec, o + NR);
    }
}

template <int NU, int NF>
__device__ inline void p2_issue(const DiscDev &D, int m, int h, int t, float2 (&sh)[FftShape<NU>::P / 2],
                                float2 (&K)[NF][2][FftShape<NU>::P / 2], float2 (&KN)[NF][2])
{
    p2_load_sh<NU>(D, m, h, t, sh);
#pragma unroll
    for (int a = 0; a < NF; ++a) p2_load_k<NU, NF>(D, m, a, h, t, K[a], KN[a]);
}

// Pass 2, one column job m in [0, n_phi/2] per group of NF * T threads (half
// h owns fluid h; NF = 1 has one half); one workgroup job per workgroup (the
// spectra of a column are too many registers to load one job ahead):
//   1. issue all loads: Sigma~_h and the kernel spectra; the spectra arrive
//      while the zero-padded forward u transform of Sigma~_h runs;
//   2. both halves put their natural-order spectra in LDS; thread t reads
//      Sigma^_a at k_lo and at the mirrors k_hi = NU - k_lo (k_hi = NU/2 for
//      t = 0, j = 0) for every a.  K(k_hi) is K(k_lo) conjugated (negated
//      too for K_phi), so every stored spectrum value is loaded exactly once;
//   3. multiply-accumulate g^_{h,c}(k) = sum_a K_c^{a h}(k) Sigma^_a(k) at the
//      2 (P/2) frequencies;
//   4. the products go to LDS in natural order and come back in the
//      transform distribution; inverse u transforms of the (r, phi) pair; the
//      first n_r outputs are stored.
template <int NU, int NF, bool SF, int GM>
__global__ void __launch_bounds__((P2Shape<NU, NF, GM>::WGS)) __attribute__((amdgpu_waves_per_eu(4)))
k_pass2(const DiscDev *discs, const WJob *wj, int nj, const float2 *twu, int kc, OneDisc one)
{
    using S = P2Shape<NU, NF, GM>;
    constexpr int P = S::P, T = S::T, H = P / 2;
    constexpr int NR = NU / 2;
    constexpr int W = LdsPlane<float>::elems(NU);
    __shared__ __attribute__((aligned(16))) float2 lds[W * S::G * 2 * NF];
    const int g = threadIdx.x / S::CT;
    const int h = (threadIdx.x % S::CT) / T;
    const int t = threadIdx.x % T;
    const int w = sg_uniform(sg_xcd_remap(blockIdx.x, kc));
    if (w >= nj) return;
    float2 *base = lds + W * g * 2 * NF;
    // planes: F_h (forward / output r) and X_h (spectrum / output phi)
    const LdsPlane<float> pl[2] = {LdsPlane<float>{base + W * (2 * h)},
                                   LdsPlane<float>{base + W * (2 * h + 1)}};
    DiscDev D;
    const WJob job = pass_job<2>(discs, wj, one, w, S::G, D);
    const int cb = job.base, cn = job.n;
    const int m = g < cn ? cb + g : cb;
    const bool pr = m == 0;  // columns 0 and n_phi/2 as one job
    const int mm = pr ? D.nphi / 2 + 1 : m;
    // 1. loads (three or four groups: the spectra of one source at a time,
    //    the next source's loaded while the current one is multiplied)
    constexpr int KA = NF <= 2 ? NF : 1;
    float2 sh[H], K[KA][2][H], KN[KA][2];
    if constexpr (NF <= 2) {
        p2_issue<NU, NF>(D, mm, h, t, sh, K, KN);
    } else {
        p2_load_sh<NU>(D, mm, h, t, sh);
        p2_load_k<NU, NF>(D, mm, 0, h, t, K[0], KN[0]);
    }
    TwRegC<NU, SF> tw;
    tw.load(twu, t);
    // SG_INDIRECT: the workgroup holding column m = 1 also forms the star's
    // pull A + i B = sum_a c_a e^{i dphi/2} conj(sum_rows Sigma~_a[row][1])
    // (c_a: table header) and adds its m = 1 coefficients to g^ of every
    // target (see ind_add below).  Uniform branch: the whole workgroup takes
    // part in the reduction.
    float2 dr = make_float2(0.f, 0.f), dp = make_float2(0.f, 0.f);
    const bool ind = (D.flags & SG_INDIRECT) && cb <= 1 && 1 < cb + cn;
    if (ind) {
        float2 ps = make_float2(0.f, 0.f);
#pragma unroll
        for (int p = 0; p < H; ++p) ps = c_add(ps, sh[p]);
        float2 *red = lds;  // the planes are not in use yet
        red[threadIdx.x] = ps;
        __syncthreads();
        for (int o = T / 2; o > 0; o >>= 1) {
            if (t < o) red[threadIdx.x] = c_add(red[threadIdx.x], red[threadIdx.x + o]);
            __syncthreads();
        }
        if (m == 1) {
            const double half = SG_PI / D.nphi;  // dphi / 2
            const double ce = cos(half), se = sin(half);
            double A = 0.0, B = 0.0;
#pragma unroll
            for (int a = 0; a < NF; ++a) {
                const float2 S = red[g * S::CT + a * T];
                const double ca = D.ind[a];
                // c_a e^{i dphi/2} conj(S)
                A += ca * (ce * S.x + se * S.y);
                B += ca * (se * S.x - ce * S.y);
            }
            // m = 1 coefficients of -(A cos phi + B sin phi) and
            // -(-A sin phi + B cos phi): -(A - iB) e^{i dphi/2}/2, -(B + iA) e^{i dphi/2}/2
            dr = make_float2((float)(-0.5 * (A * ce + B * se)), (float)(-0.5 * (A * se - B * ce)));
            dp = make_float2((float)(-0.5 * (B * ce - A * se)), (float)(-0.5 * (B * se + A * ce)));
        }
        __syncthreads();
    }
    // forward transform of the own fluid
    {
        float2 v[1][P];
#pragma unroll
        for (int p = 0; p < P; ++p) v[0][p] = p < H ? sh[p] : make_float2(0.f, 0.f);
        const LdsPlane<float> p1[1] = {pl[0]};
        fft_m<NU, false, 1>(v, t, p1, tw);
        // 2. spectra of all fluids at k_lo and k_hi
#pragma unroll
        for (int p = 0; p < P; ++p) pl[1].st(t + T * p, v[0][p]);
    }
    __syncthreads();
    float2 olo[2][H], ohi[2][H];
    if constexpr (NF <= 2) {
    float2 slo[NF][H], shi[NF][H];
#pragma unroll
    for (int a = 0; a < NF; ++a) {
        const LdsPlane<float> X{base + W * (2 * a + 1)};
#pragma unroll
        for (int j = 0; j < H; ++j) {
            const int klo = t + T * j;
            const int khi = (j == 0 && t == 0) ? NR : NU - klo;
            slo[a][j] = X.ld(klo);
            shi[a][j] = X.ld(khi);
        }
    }
    __syncthreads();
    // 3. multiply-accumulate at k_lo and k_hi.  The pair job (columns 0 and
    // n_phi/2, both real in phi): Z = S0 + i SN with S0(k) = (Z(k) + conj
    // Z(-k))/2 and SN(k) = (Z(k) - conj Z(-k))/(2i), so the packed product is
    // Y = K0 S0 + i KN SN = A Z(k) + B conj Z(-k), A, B = (K0 +- KN)/2 (K_r of
    // the two columns; A(-k) = conj A(k), and likewise B).  Plane 0 is A Z, a
    // regular r product.  Plane 1 runs the phi product with B, giving
    // a1 = B Z(k_lo) and a2 = -conj(B) Z(k_hi); B conj Z(-k) is then
    // -conj(a2) at k_lo and conj(a1) at k_hi (at k_lo = 0, k_hi = NU/2, where
    // B is real and each frequency is its own mirror, conj(a1) and
    // -conj(a2)).  Both parts go to plane 0, whose inverse transform is then
    // y = g0 + i gN.
#pragma unroll
    for (int cc = 0; cc < 2; ++cc)
#pragma unroll
        for (int j = 0; j < H; ++j) {
            const bool ny = j == 0 && t == 0;
            float2 a1 = make_float2(0.f, 0.f), a2 = make_float2(0.f, 0.f);
#pragma unroll
            for (int a = 0; a < NF; ++a) {
                const float2 k1 = K[a][cc][j];
                // mirror: conj (K_r) or minus conj (K_phi); Nyquist reads K(NU/2)
                float2 k2 = ny ? KN[a][cc] : k1;
                k2 = cc == 0 ? make_float2(k2.x, -k2.y) : make_float2(-k2.x, k2.y);
                const float2 lo = slo[a][j], hi = shi[a][j];
                a1.x += k1.x * lo.x - k1.y * lo.y;
                a1.y += k1.x * lo.y + k1.y * lo.x;
                a2.x += k2.x * hi.x - k2.y * hi.y;
                a2.y += k2.x * hi.y + k2.y * hi.x;
            }
            if (cc == 1 && pr) {
                // added to plane 0 (one inverse transform gives y); plane 1 stays zero
                const float2 c1 = make_float2(a1.x, -a1.y), c2 = make_float2(-a2.x, a2.y);
                olo[0][j] = c_add(olo[0][j], ny ? c1 : c2);
                ohi[0][j] = c_add(ohi[0][j], ny ? c2 : c1);
                a1 = make_float2(0.f, 0.f);
                a2 = make_float2(0.f, 0.f);
            }
            olo[cc][j] = a1;
            ohi[cc][j] = a2;
        }
    } else {
        // three or four groups: the same products accumulated source by source
#pragma unroll
        for (int cc = 0; cc < 2; ++cc)
#pragma unroll
            for (int j = 0; j < H; ++j) {
                olo[cc][j] = make_float2(0.f, 0.f);
                ohi[cc][j] = make_float2(0.f, 0.f);
            }
#pragma unroll
        for (int a = 0; a < NF; ++a) {
            float2 Kn[2][H], KNn[2];
            if (a + 1 < NF) p2_load_k<NU, NF>(D, mm, a + 1, h, t, Kn, KNn);
            const LdsPlane<float> X{base + W * (2 * a + 1)};
#pragma unroll
            for (int j = 0; j < H; ++j) {
                const bool ny = j == 0 && t == 0;
                const int klo = t + T * j;
                const int khi = ny ? NR : NU - klo;
                const float2 lo = X.ld(klo), hi = X.ld(khi);
#pragma unroll
                for (int cc = 0; cc < 2; ++cc) {
                    const float2 k1 = K[0][cc][j];
                    float2 k2 = ny ? KN[0][cc] : k1;
                    k2 = cc == 0 ? make_float2(k2.x, -k2.y) : make_float2(-k2.x, k2.y);
                    olo[cc][j].x += k1.x * lo.x - k1.y * lo.y;
                    olo[cc][j].y += k1.x * lo.y + k1.y * lo.x;
                    ohi[cc][j].x += k2.x * hi.x - k2.y * hi.y;
                    ohi[cc][j].y += k2.x * hi.y + k2.y * hi.x;
                }
            }
            if (a + 1 < NF) {
#pragma unroll
                for (int cc = 0; cc < 2; ++cc) {
#pragma unroll
                    for (int j = 0; j < H; ++j) K[0][cc][j] = Kn[cc][j];
                    KN[0][cc] = KNn[cc];
                }
            }
        }
        if (pr) {
#pragma unroll
            for (int j = 0; j < H; ++j) {
                const bool ny = j == 0 && t == 0;
                const float2 a1 = olo[1][j], a2 = ohi[1][j];
                const float2 c1 = make_float2(a1.x, -a1.y), c2 = make_float2(-a2.x, a2.y);
                olo[0][j] = c_add(olo[0][j], ny ? c1 : c2);
                ohi[0][j] = c_add(ohi[0][j], ny ? c2 : c1);
                olo[1][j] = make_float2(0.f, 0.f);
                ohi[1][j] = make_float2(0.f, 0.f);
            }
        }
        __syncthreads();  // every target has read the spectrum planes
    }
    // 4. back to the transform distribution, inverse pair, first n_r outputs
#pragma unroll
    for (int cc = 0; cc < 2; ++cc)
#pragma unroll
        for (int j = 0; j < H; ++j) {
            const int klo = t + T * j;
            const int khi = (j == 0 && t == 0) ? NR : NU - klo;
            pl[cc].st(klo, olo[cc][j]);
            pl[cc].st(khi, ohi[cc][j]);
        }
    __syncthreads();
    float2 acc[2][P];
#pragma unroll
    for (int cc = 0; cc < 2; ++cc)
#pragma unroll
        for (int p = 0; p < P; ++p) acc[cc][p] = pl[cc].ld(t + T * p);
    __syncthreads();
    fft_m<NU, true, 2>(acc, t, pl, tw);
    if (ind && m == 1) {
#pragma unroll
        for (int p = 0; p < H; ++p) {
            acc[0][p] = c_add(acc[0][p], dr);
            acc[1][p] = c_add(acc[1][p], dp);
        }
    }
    if (g < cn) {
        const uint32_t fs = (uint32_t)sg_blk_field_elems(D.nphi, NR);
        if (pr) {
            // y = g0 + i gN; the phi outputs of both columns are zero
            const int mh = D.nphi / 2;
            const uint32_t orr = (h * 2) * fs, op = (h * 2 + 1) * fs;
#pragma unroll
            for (int p = 0; p < H; ++p) {
                const float2 y = acc[0][p];
                const uint32_t i0 = (uint32_t)sg_blk_index(0, t + T * p, NR);
                const uint32_t i1 = (uint32_t)sg_blk_index(mh, t + T * p, NR);
                gst2(D.gh, orr + i0, make_float2(y.x, 0.f));
                gst2(D.gh, orr + i1, make_float2(y.y, 0.f));
                gst2(D.gh, op + i0, make_float2(0.f, 0.f));
                gst2(D.gh, op + i1, make_float2(0.f, 0.f));
            }
        } else {
#pragma unroll
            for (int cc = 0; cc < 2; ++cc)
#pragma unroll
                for (int p = 0; p < H; ++p)
                    gst2(D.gh, (h * 2 + cc) * fs + (uint32_t)sg_blk_index(m, t + T * p, NR), acc[cc][p]);
        }
    }
}

// Pass 3: group g takes job base + g = (target fluid b, row i): inverse phi
// transform of g^_r + i g^_phi, whose real and imaginary parts are g_r and
// g_phi.  The half spectra arrive tile by tile and are expanded into each
// group's plane: z[m] = A[m] + i B[m], z[N - m] = conj A[m] + i conj B[m].
template <int N, int NF, bool SF, int GM>
__global__ void __launch_bounds__((PassShape<N, GM>::WGS))
k_pass3(const DiscDev *discs, const WJob *wj, int nj, const float2 *twp, int kc, OneDisc one)
{
    using S = PassShape<N, GM>;
    constexpr int P = S::P, T = S::T, G = S::G, W = LdsPlane<float>::elems(N);
    constexpr int NG = (N / 2 + 1 + 3) / 4;
    __shared__ __attribute__((aligned(16))) float2 lds[W * G];
    const int g = threadIdx.x / T, t = threadIdx.x % T;
    const int w = sg_uniform(sg_xcd_remap(blockIdx.x, kc));
    if (w >= nj) return;
    DiscDev D;
    const WJob job = pass_job<3>(discs, wj, one, w, G, D);
    const int cb = job.base, cn = job.n;
    const int nr = D.nr, nrp = sg_blk_rows(nr);
    const size_t fs = sg_blk_field_elems(N, nr);
    // 1. tile loads of the row quads into the planes
    for (int e = threadIdx.x; e < (G / 4) * NG * 8; e += S::WGS) {
        const int k = e / (NG * 8), q = (e / 8) % NG, l = e & 7;
        if (4 * k >= cn) continue;
        const int j0 = cb + 4 * k;  // first job of the quad: same fluid for all 4
        const int b = j0 / nrp, i0 = j0 % nrp;
        const float2 *A = D.gh + (size_t)(b * 2) * fs + sg_blk_tile(q, i0, nr) + 2 * l;
        float2 va[2], vb[2];
        gld2x2(A, va[0], va[1]);
        gld2x2(A + fs, vb[0], vb[1]);
        const int c = 4 * q + (l >> 1), r0 = 2 * (l & 1);
        if (c > N / 2) continue;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const float2 a = va[u], bb = vb[u];
            const LdsPlane<float> X{lds + W * (4 * k + r0 + u)};
            X.st(c, make_float2(a.x - bb.y, a.y + bb.x));
            if (c != 0 && c != N / 2) X.st(N - c, make_float2(a.x + bb.y, bb.x - a.y));
        }
    }
    __syncthreads();
    const LdsPlane<float> pl{lds + W * g};
    float2 z[P];
#pragma unroll
    for (int p = 0; p < P; ++p) z[p] = pl.ld(t + T * p);
    __syncthreads();
    TwRegC<N, SF> tw;
    tw.load(twp, t);
    // 2. inverse transform, two real rows out
    fft<N, true>(z, t, pl, tw);
    const int idx = cb + g;
    const int b = idx / nrp, i = idx % nrp;
    if (g < cn && i < nr) {
        const size_t o = (size_t)b * nr * N + (size_t)i * N;
#pragma unroll
        for (int p = 0; p < P; ++p) {
            gst1nt(D.gr + o, t + T * p, z[p].x);  // outputs: streamed past the caches
            gst1nt(D.gp + o, t + T * p, z[p].y);
        }
    }
}

// ------------------------------------------------------------- launching

using KernelFn = void (*)(const DiscDev *, const WJob *, int, const float2 *, int, OneDisc);

struct PassKernel {
    KernelFn fn;
    int wgs, G, K;    // K: default XCD cluster size
    int tb = 0;       // semi-spectral pass: target rows per workgroup job
    int lds_per_row = 0, lds_fixed = 0;  // its dynamic LDS: per radial row, fixed
    KernelFn fn_one = nullptr;           // its kernel for one disc by value (null: fn takes both)
};

// Shapes above 1024 threads do not exist (null kernel).
template <int N, int NF, bool SF, int GM> static PassKernel pk1()
{
    using S = P1Shape<N, GM>;
    if constexpr (S::WGS > 1024) return PassKernel{nullptr, 0, 0, 0};
    else return {k_pass1<N, NF, SF, GM>, S::WGS, S::G, S::K};
}
template <int N, int NF, bool SF, int GM> static PassKernel pk2()
{
    using S = P2Shape<N, NF, GM>;
    if constexpr (S::WGS > 1024 || (NF > 2 && GM > 1)) return PassKernel{nullptr, 0, 0, 0};
    else return {k_pass2<N, NF, SF, GM>, S::WGS, S::G, S::K};
}
template <int N, int NF, bool SF, int GM> static PassKernel pk3()
{
    using S = PassShape<N, GM>;
    if constexpr (S::WGS > 1024) return PassKernel{nullptr, 0, 0, 0};
    else return {k_pass3<N, NF, SF, GM>, S::WGS, S::G, S::K};
}

template <bool SF, int GM> static PassKernel pick_kernel(int pass, int n, int nf)
{
#define SG_CASE(F, L) \
    case L: return nf == 1 ? F<L, 1, SF, GM>() : F<L, 2, SF, GM>();
#define SG_SIZES(F)                                                                               \
    SG_CASE(F, 4) SG_CASE(F, 8) SG_CASE(F, 16) SG_CASE(F, 32) SG_CASE(F, 64) SG_CASE(F, 128)      \
    SG_CASE(F, 256) SG_CASE(F, 512) SG_CASE(F, 1024) SG_CASE(F, 2048)
    if (pass == 1) {
        switch (n) { SG_SIZES(pk1) }
    } else if (pass == 2) {
        if (nf > 2) {  // three or four groups (passes 1 and 3 do not depend on the count)
#define SG_CASE34(L) \
    case L: return nf == 3 ? pk2<L, 3, SF, GM>() : pk2<L, 4, SF, GM>();
            switch (n) {
                SG_CASE34(4) SG_CASE34(8) SG_CASE34(16) SG_CASE34(32) SG_CASE34(64) SG_CASE34(128)
                SG_CASE34(256) SG_CASE34(512) SG_CASE34(1024) SG_CASE34(2048)
            }
#undef SG_CASE34
            return PassKernel{nullptr, 0, 0, 0};
        }
        switch (n) { SG_SIZES(pk2) SG_CASE(pk2, 4096) }
    } else {
        switch (n) { SG_SIZES(pk3) }
    }
#undef SG_SIZES
#undef SG_CASE
    return PassKernel{nullptr, 0, 0, 0};
}

// Semi-spectral middle pass (variant = gm: 1, 2, 3).
static bool ss_pass_kernel(int nf, int gm, PassKernel &out)
{
    SsPassInfo k;
    if (!sg_ss_pass_kernel(nf, gm, k)) return false;
    out = PassKernel{k.fn, k.wgs, 1, 1, k.tb, k.lds_per_row, k.lds_fixed, k.fn_one};
    return true;
}

static bool pass_kernel(int pass, int n, int nf, bool sf, int gm, PassKernel &out)
{
    if (gm == 2) out = sf ? pick_kernel<true, 2>(pass, n, nf) : pick_kernel<false, 2>(pass, n, nf);
    else out = sf ? pick_kernel<true, 1>(pass, n, nf) : pick_kernel<false, 1>(pass, n, nf);
    return out.fn != nullptr;
}

// Radix order has a choice only when the length is not a power of 8.
static bool has_small_radix(int n)
{
    while (n >= 8) n /= 8;
    return n > 1;
}

// ------------------------------------------------------------- batch plan
// Tuning parameters of one launch: radix order, tile shape (transforms per
// workgroup times gm), XCD cluster size (0: the default).
struct Variant {
    int sf = 0, gm = 1, K = 0;
};

// A launch class: one pass over the discs sharing a transform length and a
// fluid count; the middle pass of semi-spectral discs (ss) forms classes of
// its own, keyed by n_r (len).
struct ClassSpec {
    int pass, len, nf, ss;
    std::vector<int> discs;
};

struct Launch {
    PassKernel k;
    Variant v;
    int K;            // cluster size in use
    size_t wj_off;    // offset (in WJob units) into the workgroup-job table
    int nj;           // workgroup jobs of this launch
    int jobs;         // jobs of its first disc (of a one-disc batch: all)
    int grid;         // workgroups (a multiple of 8 K)
    const float2 *tw; // twiddles of this launch's transform length
    int pass;
    size_t lds;       // dynamic LDS bytes
};

struct Plan {
    std::vector<DiscDev> discs;
    std::vector<WJob> wjobs;
    std::vector<Launch> launches;
};

size_t sg_fft_disc_ws_bytes(const sg_disc &d)
{
    const size_t fs = sg_blk_field_elems(d.grid.n_phi, d.grid.n_r);
    return sg_align256(sizeof(float2) * fs * d.fluids.n_fluids) +
           sg_align256(sizeof(float2) * fs * 2 * d.fluids.n_fluids);
}

// Jobs of one disc in a pass: pass 1 (fluid, row pair), pass 2 columns m <= n_phi/2
// (semi-spectral: (m, target fluid, block of tb target rows)), pass 3 (target
// fluid, row) pairs; rows padded to sg_blk_rows.
static int pass_jobs(const sg_disc &d, int pass, int tb)
{
    const int nf = d.fluids.n_fluids, nrp = sg_blk_rows(d.grid.n_r);
    if (pass == 1) return nf * nrp / 2;
    if (pass == 2) {
        if (d.flags & SG_SEMI_SPECTRAL) return (d.grid.n_phi / 2 + 1) * nf * ((d.grid.n_r + tb - 1) / tb);
        return d.grid.n_phi / 2;  // job 0 carries columns 0 and n_phi/2
    }
    return nf * nrp;
}

// Grid of a launch: whole XCD clusters of 8 K workgroups, one per
// workgroup job.
static int launch_grid(int nj, int K)
{
    const int cluster = 8 * K;
    return (nj + cluster - 1) / cluster * cluster;
}

// Workgroup jobs of a class: G jobs per workgroup job, each disc padded to a
// whole number of clusters of K workgroup jobs so that cache-line sharing
// stays inside one disc.
static void class_wjobs(const sg_disc *discs, const ClassSpec &c, int G, int K, int tb, std::vector<WJob> &out)
{
    out.clear();
    for (int di : c.discs) {
        const int cnt = pass_jobs(discs[di], c.pass, tb);
        for (int b = 0; b < cnt; b += G) out.push_back({di, b, std::min(G, cnt - b), 0});
        while (out.size() % K) out.push_back({di, 0, 0, 0});
    }
}

static std::vector<ClassSpec> plan_classes(const sg_disc *discs, int n)
{
    std::vector<ClassSpec> out;
    for (int pass = 1; pass <= 3; ++pass) {
        std::map<std::tuple<int, int, int>, std::vector<int>> classes;
        for (int i = 0; i < n; ++i) {
            const int ss = pass == 2 && (discs[i].flags & SG_SEMI_SPECTRAL) ? 1 : 0;
            const int len = pass == 2 ? (ss ? discs[i].grid.n_r : 2 * discs[i].grid.n_r) : discs[i].grid.n_phi;
            classes[{ss, len, discs[i].fluids.n_fluids}].push_back(i);
        }
        for (auto &kv : classes)
            out.push_back({pass, std::get<1>(kv.first), std::get<2>(kv.first), std::get<0>(kv.first), kv.second});
    }
    return out;
}

// Tuned variants, keyed by (pass, length, fluids, shape hash of the class).
using TuneKey = std::tuple<int, int, int, uint64_t>;
static std::map<TuneKey, Variant> g_tuned;

static TuneKey tune_key(const sg_disc *discs, const ClassSpec &c)
{
    uint64_t h = 1469598103934665603ull;  // FNV-1a over the disc shapes
    auto mix = [&](uint64_t v) {
        for (int b = 0; b < 8; ++b) {
            h ^= (v >> (8 * b)) & 0xff;
            h *= 1099511628211ull;
        }
    };
    for (int di : c.discs) {
        mix((uint64_t)discs[di].grid.n_r);
        mix((uint64_t)discs[di].grid.n_phi);
    }
    if (c.ss) mix(0x5353ull);
    return TuneKey{c.pass, c.len, c.nf, h};
}

// Default variant of a class: semi-spectral classes pick the middle-pass
// shape by n_r; the FFT passes start from the plain shape.
static Variant default_variant(const ClassSpec &c)
{
    Variant v;
    if (c.ss) v.gm = sg_ss_default_variant(c.len);
    return v;
}

static bool make_launch(const sg_disc *discs, const Plan &P, const ClassSpec &c, Variant v, Launch &La,
                        std::vector<WJob> &wj)
{
    PassKernel k;
    if (c.ss ? !ss_pass_kernel(c.nf, v.gm, k) : !pass_kernel(c.pass, c.len, c.nf, v.sf != 0, v.gm, k))
        return false;
    La.k = k;
    La.v = v;
    La.K = v.K > 0 ? v.K : k.K;
    La.lds = 0;
    if (c.ss) {  // the longest staged column: a full mode's n_r or a banded mode's window
        int cs = 0;
        for (int di : c.discs) {
            const DiscDev &D = P.discs[di];
            cs = std::max(cs, D.nr);
            if (D.ss_wmax >= 0) cs = std::max(cs, k.tb + 2 * D.ss_wmax + 4);
        }
        La.lds = (size_t)k.lds_per_row * cs + k.lds_fixed;
    }
    class_wjobs(discs, c, k.G, La.K, k.tb, wj);
    La.nj = (int)wj.size();
    La.jobs = pass_jobs(discs[c.discs[0]], c.pass, k.tb);
    La.grid = launch_grid(La.nj, La.K);
    const DiscDev &D0 = P.discs[c.discs[0]];
    La.tw = c.pass == 2 ? D0.tw_u : D0.tw_phi;
    La.pass = c.pass;
    La.wj_off = 0;
    return true;
}

static void fill_discs(const sg_disc *discs, int n, char *ws, Plan &P)
{
    P.discs.resize(n);
    size_t off = 0;
    for (int i = 0; i < n; ++i) {
        const sg_disc &d = discs[i];
        const char *tb = (const char *)d.table;
        DiscDev &D = P.discs[i];
        D.sigma = d.sigma;
        D.gr = d.g_r;
        D.gp = d.g_phi;
        D.modes = nullptr;
        D.ss_wmax = -1;
        if (d.flags & SG_SEMI_SPECTRAL) {
            // staged column of the widest banded mode of this grid (the band
            // rule without SG_SS_FULL, so that any table of the grid fits)
            const SsLayout B = sg_ss_layout(d.grid.n_r, d.grid.n_phi, d.fluids.n_fluids, sg_ss_du(d.grid, d.flags), false);
            D.ss_wmax = B.max_w;
            const SsLayout L = sg_ss_layout(d.grid.n_r, d.grid.n_phi, d.fluids.n_fluids, 1.0, true);
            D.spec = (const float2 *)(tb + L.off_coef);
            D.modes = (const SsMode *)(tb + L.off_modes);
            D.dspec = nullptr;
            D.tw_u = nullptr;
            D.tw_phi = (const float2 *)(tb + L.off_tw_phi);
            D.ind = nullptr;
        } else {
            const TableLayout L = sg_table_layout(d.grid.n_r, d.grid.n_phi, d.fluids.n_fluids, d.flags);
            D.spec = (const float2 *)(tb + L.off_spec);
            D.dspec = (d.flags & SG_WITH_DH) ? (const float2 *)(tb + L.off_dspec) : nullptr;
            D.tw_u = (const float2 *)(tb + L.off_tw_u);
            D.tw_phi = (const float2 *)(tb + L.off_tw_phi);
            D.ind = (const double *)(tb + offsetof(sg_table_header, ind_coef));
        }
        const size_t fs = sg_blk_field_elems(d.grid.n_phi, d.grid.n_r);
        D.st = (float2 *)(ws + off);
        D.gh = (float2 *)(ws + off + sg_align256(sizeof(float2) * fs * d.fluids.n_fluids));
        off += sg_fft_disc_ws_bytes(d);
        D.nr = d.grid.n_r;
        D.nphi = d.grid.n_phi;
        D.nf = d.fluids.n_fluids;
        D.flags = d.flags;
        D.ns = d.n_species;
        D.gcount[0] = D.gcount[1] = D.gcount[2] = D.gcount[3] = 0;
        for (int s = 0; s < d.n_species; ++s) {
            const int gp = d.species_group[s];
            D.gsp[gp][D.gcount[gp]++] = (uint8_t)s;
        }
    }
}

// One launch per class, with the tuned variant where one is known.
static bool build_plan(const sg_disc *discs, int n, char *ws, Plan &P)
{
    fill_discs(discs, n, ws, P);
    std::vector<WJob> wj;
    for (const ClassSpec &c : plan_classes(discs, n)) {
        Variant v = default_variant(c);
        auto it = g_tuned.find(tune_key(discs, c));
        if (it != g_tuned.end()) v = it->second;
        Launch La;
        if (!make_launch(discs, P, c, v, La, wj)) return false;
        La.wj_off = P.wjobs.size();
        P.wjobs.insert(P.wjobs.end(), wj.begin(), wj.end());
        P.launches.push_back(La);
    }
    return true;
}

struct Cached {
    void *dmem = nullptr;      // descriptors + jobs on the device (none for a one-disc plan)
    hipGraphExec_t exec = nullptr;
    hipGraph_t graph = nullptr;
    uint64_t last_use = 0;
    Plan plan;
};

// At most SG_CACHE_MAX signatures keep their plan and graph; beyond that the
// least recently used one is released (after a device synchronisation, so it
// is idle).  Callers that pass new buffers on every call (one-off outputs)
// therefore cannot grow the cache without bound.
#define SG_CACHE_MAX 256
static std::mutex g_mu;
static std::map<std::vector<uint64_t>, Cached *> g_cache;
static uint64_t g_tick = 0;

// Batches of one disc (without species) are cached by shape alone: nothing of
// theirs is kept on the device, and each call fills the descriptor that its
// launches take by value with the addresses it was given.
static bool one_disc(const sg_disc *discs, int n) { return n == 1 && discs[0].n_species == 0; }

// The radii are part of a semi-spectral disc's key: they set the band of its
// modes and so the staged column (ss_wmax).  A plan of narrower bands makes
// the middle pass drop the modes that exceed it.
static void push_radii(std::vector<uint64_t> &k, const sg_disc &d)
{
    if (!(d.flags & SG_SEMI_SPECTRAL)) return;
    uint64_t w[2];
    memcpy(&w[0], &d.grid.r_min, 8);
    memcpy(&w[1], &d.grid.r_max, 8);
    k.insert(k.end(), w, w + 2);
}

static std::vector<uint64_t> shape_signature(const sg_disc &d)
{
    std::vector<uint64_t> k(3);
    int dev = 0;
    (void)hipGetDevice(&dev);
    k[0] = (1ull << 40) | (uint64_t)dev;  // no batch signature begins so
    k[1] = ((uint64_t)d.grid.n_r << 32) | (uint32_t)d.grid.n_phi;
    k[2] = ((uint64_t)d.fluids.n_fluids << 32) | d.flags;
    push_radii(k, d);
    return k;
}

static std::vector<uint64_t> signature(const sg_disc *discs, int n, void *ws)
{
    std::vector<uint64_t> k;
    k.reserve(n * 9 + 2);
    int dev = 0;
    (void)hipGetDevice(&dev);
    k.push_back((uint64_t)dev);
    k.push_back((uint64_t)(uintptr_t)ws);
    for (int i = 0; i < n; ++i) {
        const sg_disc &d = discs[i];
        k.push_back(((uint64_t)d.grid.n_r << 32) | (uint32_t)d.grid.n_phi);
        k.push_back(((uint64_t)d.fluids.n_fluids << 32) | d.flags);
        uint64_t sp = (uint64_t)(uint32_t)d.n_species;
        for (int s = 0; s < 8 && s < d.n_species; ++s) sp |= (uint64_t)d.species_group[s] << (8 + 4 * s);
        k.push_back(sp);
        k.push_back((uint64_t)(uintptr_t)d.sigma);
        k.push_back((uint64_t)(uintptr_t)d.g_r);
        k.push_back((uint64_t)(uintptr_t)d.g_phi);
        k.push_back((uint64_t)(uintptr_t)d.table);
        push_radii(k, d);
    }
    return k;
}

static sg_status launch_one(const DiscDev *dd, const WJob *wj, const Launch &L, hipStream_t s)
{
    hipLaunchKernelGGL(L.k.fn, dim3(L.grid), dim3(L.k.wgs), (unsigned)L.lds, s, dd, wj + L.wj_off, L.nj, L.tw,
                       L.K, OneDisc{});
    SG_HIP(hipGetLastError());
    return SG_OK;
}

// The addresses of a one-disc call.
struct OneCall {
    const char *table;
    char *ws;
    const float *sigma;
    float *gr, *gp;
};

static OneCall one_call(const sg_disc &d, void *ws)
{
    return {(const char *)d.table, (char *)ws, d.sigma, d.g_r, d.g_phi};
}

// What launch L of a one-disc plan passes: the plan's offsets at the call's
// addresses.  tw: the pass's twiddles.
static OneDisc one_disc_at(const DiscDev &P, const OneCall &c, const Launch &L, const float2 *&tw)
{
    auto tab = [&](const void *p) -> const char * { return c.table + (uintptr_t)p; };
    float2 *const st = (float2 *)c.ws, *const gh = (float2 *)(c.ws + (uintptr_t)P.gh);
    OneDisc o{};
    if (L.pass == 1) {
        o.in = c.sigma;
        o.out = st;
    } else if (L.pass == 3) {
        o.in = gh;
        o.out = c.gr;
        o.out2 = c.gp;
    } else {
        o.in = tab(P.spec);
        o.in2 = tab((P.flags & SG_SEMI_SPECTRAL) ? (const void *)P.modes : (const void *)P.ind);
        o.out = st;
        o.out2 = gh;
    }
    o.nr = P.nr;
    o.nphi = P.nphi;
    o.nf = P.nf;
    o.flags = P.flags;
    o.ss_wmax = P.ss_wmax;
    o.jobs = L.jobs;
    tw = (const float2 *)tab(L.tw);
    return o;
}

static const WJob *cached_wjobs(const Cached &C)
{
    return (const WJob *)((const char *)C.dmem + sg_align256(sizeof(DiscDev) * C.plan.discs.size()));
}

// Launch L of a plan, of a one-disc plan with the call's descriptor; events
// (may be null) take the kernel's own start and end.
static sg_status launch_plan(const Cached &C, const OneCall &one, const Launch &L, hipStream_t s,
                             hipEvent_t e0 = nullptr, hipEvent_t e1 = nullptr)
{
    const DiscDev *dd = (const DiscDev *)C.dmem;
    const WJob *wj = dd ? cached_wjobs(C) + L.wj_off : nullptr;
    const float2 *tw = L.tw;
    const OneDisc o = dd ? OneDisc{} : one_disc_at(C.plan.discs[0], one, L, tw);
    const KernelFn fn = !dd && L.k.fn_one ? L.k.fn_one : L.k.fn;
    if (e0)
        hipExtLaunchKernelGGL(fn, dim3(L.grid), dim3(L.k.wgs), (uint32_t)L.lds, s, e0, e1, 0, dd, wj, L.nj, tw, L.K, o);
    else
        hipLaunchKernelGGL(fn, dim3(L.grid), dim3(L.k.wgs), (unsigned)L.lds, s, dd, wj, L.nj, tw, L.K, o);
    SG_HIP(hipGetLastError());
    return SG_OK;
}

static sg_status enqueue(const Cached &C, const OneCall &one, hipStream_t s)
{
    for (const Launch &L : C.plan.launches) {
        const sg_status st = launch_plan(C, one, L, s);
        if (st != SG_OK) return st;
    }
    return SG_OK;
}

// Graph capture of a plan: the launch classes of one pass (discs of other
// transform lengths or fluid counts) do not depend on each other, so each
// pass forks them onto parallel branches of the graph (auxiliary capture
// streams joined back before the next pass), and classes whose kernels are
// too small to fill the GPU on their own (short transforms, few rows) run
// side by side instead of one after the other.  The caller creates the
// auxiliary streams and events (fork_resources) before the capture and
// destroys them after it ends.
struct ForkRes {
    std::vector<hipStream_t> aux;
    std::vector<hipEvent_t> ev;
    ~ForkRes()
    {
        for (auto e : ev)
            if (e) (void)hipEventDestroy(e);
        for (auto a : aux)
            if (a) (void)hipStreamDestroy(a);
    }
};

static sg_status fork_resources(const Cached &C, ForkRes &R)
{
    const auto &Ls = C.plan.launches;
    size_t widest = 1, nev = 0;
    for (size_t i = 0; i < Ls.size();) {
        size_t j = i;
        while (j < Ls.size() && Ls[j].pass == Ls[i].pass) ++j;
        widest = std::max(widest, j - i);
        if (j - i > 1) nev += j - i;
        i = j;
    }
    R.aux.assign(widest - 1, nullptr);
    R.ev.assign(nev, nullptr);
    for (auto &a : R.aux) SG_HIP(hipStreamCreateWithFlags(&a, hipStreamNonBlocking));
    for (auto &e : R.ev) SG_HIP(hipEventCreateWithFlags(&e, hipEventDisableTiming));
    return SG_OK;
}

static sg_status enqueue_forked(const Cached &C, hipStream_t s, const ForkRes &R)
{
    const auto &Ls = C.plan.launches;
    const DiscDev *dd = (const DiscDev *)C.dmem;
    const WJob *wj = cached_wjobs(C);
    size_t i = 0, e = 0;
    while (i < Ls.size()) {
        size_t j = i;
        while (j < Ls.size() && Ls[j].pass == Ls[i].pass) ++j;
        const int nb = (int)(j - i);  // classes of this pass
        if (nb == 1) {
            const sg_status st = launch_one(dd, wj, Ls[i], s);
            if (st != SG_OK) return st;
            i = j;
            continue;
        }
        const hipEvent_t fork = R.ev[e];  // R.ev[e + k]: join of branch k
        SG_HIP(hipEventRecord(fork, s));
        for (int k = 1; k < nb; ++k) {
            SG_HIP(hipStreamWaitEvent(R.aux[k - 1], fork, 0));
            const sg_status st = launch_one(dd, wj, Ls[i + k], R.aux[k - 1]);
            if (st != SG_OK) return st;
            SG_HIP(hipEventRecord(R.ev[e + k], R.aux[k - 1]));
        }
        const sg_status st = launch_one(dd, wj, Ls[i], s);
        if (st != SG_OK) return st;
        for (int k = 1; k < nb; ++k) SG_HIP(hipStreamWaitEvent(s, R.ev[e + k], 0));
        e += nb;
        i = j;
    }
    return SG_OK;
}

// A plan runs from a captured graph only when some pass has several launch
// classes, which the graph runs on parallel branches.  A plain chain (one
// launch per pass) is enqueued directly: on gfx950 a graph launch puts a few
// microseconds of GPU-side latency in front of its first kernel (measured on
// the two-fluid 1024 x 2048 disc: 81.4 -> 74.4 us per cold step, 65 -> 58 us
// warm), while a forked plan gains more from its branches than it pays
// (64-disc batch: 0.355 ms graphed, 0.362 ms enqueued serially).
// SG_NO_GRAPH=1 enqueues every plan directly.
static bool plan_has_forks(const Plan &P)
{
    for (size_t i = 1; i < P.launches.size(); ++i)
        if (P.launches[i].pass == P.launches[i - 1].pass) return true;
    return false;
}

static bool use_graph(const Plan &P)
{
    const char *e = getenv("SG_NO_GRAPH");
    return !(e && e[0] == '1') && plan_has_forks(P);
}

static void destroy(Cached *C)
{
    if (C->exec) (void)hipGraphExecDestroy(C->exec);
    if (C->graph) (void)hipGraphDestroy(C->graph);
    if (C->dmem) (void)hipFree(C->dmem);
    delete C;
}

// Plan, device tables and graph of a batch signature (built on first use).
// Caller holds g_mu.
static sg_status get_cached(const sg_disc *discs, int n, void *ws, Cached *&out)
{
    const bool single = one_disc(discs, n);
    auto key = single ? shape_signature(discs[0]) : signature(discs, n, ws);
    auto it = g_cache.find(key);
    if (it != g_cache.end()) {
        out = it->second;
        out->last_use = ++g_tick;
        return SG_OK;
    }
    if (g_cache.size() >= SG_CACHE_MAX) {
        auto lru = g_cache.begin();
        for (auto jt = g_cache.begin(); jt != g_cache.end(); ++jt)
            if (jt->second->last_use < lru->second->last_use) lru = jt;
        SG_HIP(hipDeviceSynchronize());
        destroy(lru->second);
        g_cache.erase(lru);
    }
    std::unique_ptr<Cached, void (*)(Cached *)> own(new Cached, destroy);
    Cached *const C = own.get();
    C->last_use = ++g_tick;
    sg_disc at0 = discs[0];  // a one-disc plan holds offsets
    at0.table = nullptr;
    if (!build_plan(single ? &at0 : discs, n, single ? nullptr : (char *)ws, C->plan)) return SG_ERR_UNSUPPORTED;
    if (single) {
        g_cache[key] = C;
        out = own.release();
        return SG_OK;
    }
    const size_t bd = sg_align256(sizeof(DiscDev) * n);
    const size_t bytes = bd + sizeof(WJob) * C->plan.wjobs.size();
    SG_HIP(hipMalloc(&C->dmem, bytes));
    if (hipMemcpy(C->dmem, C->plan.discs.data(), sizeof(DiscDev) * n, hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy((char *)C->dmem + bd, C->plan.wjobs.data(), sizeof(WJob) * C->plan.wjobs.size(),
                  hipMemcpyHostToDevice) != hipSuccess)
        return SG_ERR_HIP;
    if (use_graph(C->plan)) {
        hipStream_t cs;
        SG_HIP(hipStreamCreateWithFlags(&cs, hipStreamNonBlocking));
        ForkRes R;
        bool ok = fork_resources(*C, R) == SG_OK;
        ok = ok && hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal) == hipSuccess;
        sg_status st = ok ? enqueue_forked(*C, cs, R) : SG_ERR_HIP;
        hipGraph_t gph = nullptr;
        ok = hipStreamEndCapture(cs, &gph) == hipSuccess && ok && st == SG_OK;
        if (ok) ok = hipGraphInstantiate(&C->exec, gph, nullptr, nullptr, 0) == hipSuccess;
        (void)hipStreamDestroy(cs);
        C->graph = gph;
        if (!ok) return SG_ERR_HIP;
    }
    g_cache[key] = C;
    out = own.release();
    return SG_OK;
}

sg_status sg_fft_run(const sg_disc *discs, int n, void *ws, hipStream_t s)
{
    std::lock_guard<std::mutex> lk(g_mu);
    Cached *C = nullptr;
    const OneCall one = one_call(discs[0], ws);
    const sg_status st = get_cached(discs, n, ws, C);
    if (st != SG_OK) return st;
    if (C->exec) {
        SG_HIP(hipGraphLaunch(C->exec, s));
        return SG_OK;
    }
    return enqueue(*C, one, s);
}

// One step, every launch in plan order with a start and a stop event
// attached to the launch itself (hipExtLaunchKernel: the events take the
// kernel's own start and end, not a marker between launches), with nothing
// run before it: a caller that evicts the caches first times a cold step.
// ms[p] = the summed kernel time of pass p's launches.
static sg_status profile_one_step(const Cached &C, const OneCall &one, hipStream_t s, float *ms)
{
    const size_t nl = C.plan.launches.size();
    std::vector<hipEvent_t> ev(2 * nl, nullptr);
    sg_status st = SG_OK;
    for (auto &e : ev)
        if (st == SG_OK && hipEventCreate(&e) != hipSuccess) st = SG_ERR_HIP;
    for (size_t i = 0; i < nl && st == SG_OK; ++i)
        st = launch_plan(C, one, C.plan.launches[i], s, ev[2 * i], ev[2 * i + 1]);
    if (st == SG_OK && nl && hipEventSynchronize(ev[2 * nl - 1]) != hipSuccess) st = SG_ERR_HIP;
    for (int p = 0; p < 3; ++p) ms[p] = 0.f;
    for (size_t i = 0; i < nl && st == SG_OK; ++i) {
        float t = 0.f;
        if (hipEventElapsedTime(&t, ev[2 * i], ev[2 * i + 1]) != hipSuccess) st = SG_ERR_HIP;
        ms[C.plan.launches[i].pass - 1] += t;
    }
    for (auto &e : ev)
        if (e) (void)hipEventDestroy(e);
    return st;
}

// Per-pass timing: each pass's launches are enqueued `reps` times back to
// back between two HIP events on `s` (no graph), after one untimed complete
// run; ms[p] is the mean milliseconds per launch of pass p + 1 (all of its
// launch classes).  Back-to-back launches of the same pass leave each one's
// duration with only the launch gap added, which is what a kernel trace
// reports per dispatch.
// (reps == 1: profile_one_step above.)
sg_status sg_fft_profile(const sg_disc *discs, int n, void *ws, hipStream_t s, int reps, float *ms)
{
    std::lock_guard<std::mutex> lk(g_mu);
    Cached *C = nullptr;
    const OneCall one = one_call(discs[0], ws);
    sg_status st = get_cached(discs, n, ws, C);
    if (st != SG_OK) return st;
    if (reps == 1) return profile_one_step(*C, one, s, ms);
    st = enqueue(*C, one, s);
    if (st != SG_OK) return st;
    hipEvent_t ev[4] = {nullptr, nullptr, nullptr, nullptr};
    for (auto &e : ev) SG_HIP(hipEventCreate(&e));
    for (int pass = 1; pass <= 3 && st == SG_OK; ++pass) {
        if (pass == 1 && hipEventRecord(ev[0], s) != hipSuccess) st = SG_ERR_HIP;
        for (int r = 0; r < reps && st == SG_OK; ++r)
            for (const Launch &L : C->plan.launches)
                if (L.pass == pass && st == SG_OK) st = launch_plan(*C, one, L, s);
        if (st == SG_OK && hipEventRecord(ev[pass], s) != hipSuccess) st = SG_ERR_HIP;
    }
    if (st == SG_OK && hipEventSynchronize(ev[3]) != hipSuccess) st = SG_ERR_HIP;
    for (int p = 0; p < 3 && st == SG_OK; ++p) {
        float t = 0.f;
        if (hipEventElapsedTime(&t, ev[p], ev[p + 1]) != hipSuccess) st = SG_ERR_HIP;
        ms[p] = t / reps;
    }
    for (auto &e : ev) (void)hipEventDestroy(e);
    return st;
}

static void release_locked()
{
    (void)hipDeviceSynchronize();
    for (auto &kv : g_cache) destroy(kv.second);
    g_cache.clear();
}

int sg_fft_cache_entries()
{
    std::lock_guard<std::mutex> lk(g_mu);
    return (int)g_cache.size();
}

void sg_fft_release()
{
    std::lock_guard<std::mutex> lk(g_mu);
    release_locked();
}

// ------------------------------------------------------------- autotuner
// Relative RMS difference of two float buffers: acc[0] += sum (a - b)^2,
// acc[1] += sum b^2 (double, one atomic pair per workgroup).
__global__ void __launch_bounds__(256) k_cmp(const float *a, const float *b, size_t n, double *acc)
{
    __shared__ double red[2][256];
    double d2 = 0.0, b2 = 0.0;
    for (size_t i = blockIdx.x * (size_t)256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) {
        const double x = a[i], y = b[i];
        d2 += (x - y) * (x - y);
        b2 += y * y;
    }
    red[0][threadIdx.x] = d2;
    red[1][threadIdx.x] = b2;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (threadIdx.x < o) {
            red[0][threadIdx.x] += red[0][threadIdx.x + o];
            red[1][threadIdx.x] += red[1][threadIdx.x + o];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        atomicAdd(&acc[0], red[0][0]);
        atomicAdd(&acc[1], red[1][0]);
    }
}

// Output buffers of a class: (pointer, float count) per written region.
static void class_outputs(const sg_disc *discs, const Plan &P, const ClassSpec &c,
                          std::vector<std::pair<float *, size_t>> &out)
{
    out.clear();
    for (int di : c.discs) {
        const DiscDev &D = P.discs[di];
        const size_t fs = sg_blk_field_elems(D.nphi, D.nr);
        const size_t cells = (size_t)D.nr * D.nphi * D.nf;
        if (c.pass == 1) out.push_back({(float *)D.st, 2 * fs * D.nf});
        else if (c.pass == 2) out.push_back({(float *)D.gh, 4 * fs * D.nf});
        else {
            out.push_back({D.gr, cells});
            out.push_back({D.gp, cells});
        }
    }
    (void)discs;
}

namespace {
struct TuneScratch {
    void *dd = nullptr;   // DiscDev array
    void *wj = nullptr;   // WJob table of the candidate
    size_t wj_cap = 0;
    float *ref = nullptr; // reference outputs of the class
    size_t ref_cap = 0;
    double *acc = nullptr;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    ~TuneScratch()
    {
        if (e0) (void)hipEventDestroy(e0);
        if (e1) (void)hipEventDestroy(e1);
        if (dd) (void)hipFree(dd);
        if (wj) (void)hipFree(wj);
        if (ref) (void)hipFree(ref);
        if (acc) (void)hipFree(acc);
    }
};
}  // namespace

static sg_status tune_upload_wj(TuneScratch &S, const std::vector<WJob> &wj)
{
    const size_t bytes = sizeof(WJob) * wj.size();
    if (bytes > S.wj_cap) {
        if (S.wj) (void)hipFree(S.wj);
        S.wj = nullptr;
        SG_HIP(hipMalloc(&S.wj, bytes));
        S.wj_cap = bytes;
    }
    SG_HIP(hipMemcpy(S.wj, wj.data(), bytes, hipMemcpyHostToDevice));
    return SG_OK;
}

static sg_status tune_time(TuneScratch &S, const Launch &L, hipStream_t s, int reps, float &ms)
{
    for (int r = 0; r < 2; ++r)
        if (launch_one((const DiscDev *)S.dd, (const WJob *)S.wj, L, s) != SG_OK) return SG_ERR_HIP;
    SG_HIP(hipEventRecord(S.e0, s));
    for (int r = 0; r < reps; ++r)
        if (launch_one((const DiscDev *)S.dd, (const WJob *)S.wj, L, s) != SG_OK) return SG_ERR_HIP;
    SG_HIP(hipEventRecord(S.e1, s));
    SG_HIP(hipEventSynchronize(S.e1));
    SG_HIP(hipEventElapsedTime(&ms, S.e0, S.e1));
    ms /= reps;
    return SG_OK;
}

static sg_status tune_compare(TuneScratch &S, const std::vector<std::pair<float *, size_t>> &outs,
                              hipStream_t s, double &rel)
{
    SG_HIP(hipMemsetAsync(S.acc, 0, 2 * sizeof(double), s));
    size_t off = 0;
    for (const auto &o : outs) {
        const int grid = (int)std::min<size_t>((o.second + 255) / 256, 2048);
        hipLaunchKernelGGL(k_cmp, dim3(grid), dim3(256), 0, s, o.first, S.ref + off, o.second, S.acc);
        SG_HIP(hipGetLastError());
        off += o.second;
    }
    double h[2] = {0.0, 0.0};
    SG_HIP(hipMemcpyAsync(h, S.acc, sizeof(h), hipMemcpyDeviceToHost, s));
    SG_HIP(hipStreamSynchronize(s));
    rel = h[1] > 0.0 ? std::sqrt(h[0] / h[1]) : (h[0] > 0.0 ? 1.0 : 0.0);
    if (!(rel == rel)) rel = 1.0;  // NaN
    return SG_OK;
}

static void load_tune_file();
static void save_tune_file();

sg_status sg_fft_tune(const sg_disc *discs, int n, void *ws, hipStream_t s, sg_tune_result *res, int cap,
                      int *nres)
{
    std::lock_guard<std::mutex> lk(g_mu);
    load_tune_file();
    int count = 0;
    TuneScratch S;
    Plan P;
    fill_discs(discs, n, (char *)ws, P);
    SG_HIP(hipMalloc(&S.dd, sizeof(DiscDev) * n));
    SG_HIP(hipMemcpy(S.dd, P.discs.data(), sizeof(DiscDev) * n, hipMemcpyHostToDevice));
    SG_HIP(hipMalloc(&S.acc, 2 * sizeof(double)));
    SG_HIP(hipEventCreate(&S.e0));
    SG_HIP(hipEventCreate(&S.e1));
    const int reps = 10;
    std::vector<WJob> wj;
    std::vector<std::pair<float *, size_t>> outs;
    for (const ClassSpec &c : plan_classes(discs, n)) {
        // reference: the default variant
        Launch L0;
        const Variant v0 = default_variant(c);
        if (!make_launch(discs, P, c, v0, L0, wj)) return SG_ERR_UNSUPPORTED;
        sg_status st = tune_upload_wj(S, wj);
        if (st != SG_OK) return st;
        if (launch_one((const DiscDev *)S.dd, (const WJob *)S.wj, L0, s) != SG_OK) return SG_ERR_HIP;
        class_outputs(discs, P, c, outs);
        size_t total = 0;
        for (const auto &o : outs) total += o.second;
        if (total > S.ref_cap) {
            if (S.ref) (void)hipFree(S.ref);
            S.ref = nullptr;
            SG_HIP(hipMalloc(&S.ref, total * sizeof(float)));
            S.ref_cap = total;
        }
        size_t off = 0;
        for (const auto &o : outs) {
            SG_HIP(hipMemcpyAsync(S.ref + off, o.first, o.second * sizeof(float), hipMemcpyDeviceToDevice, s));
            off += o.second;
        }
        float ms0 = 0.f;
        st = tune_time(S, L0, s, reps, ms0);
        if (st != SG_OK) return st;
        // candidates
        Variant best = v0;
        float ms_best = ms0;
        double rel_best = 0.0;
        int ncand = 0, nrej = 0;
        for (int sf = 0; sf <= (!c.ss && has_small_radix(c.len) ? 1 : 0); ++sf)
            for (int gm = 1; gm <= (c.ss ? 4 : 2); ++gm)
                for (int K : {1, 2, 4, 8}) {
                    const Variant v{sf, gm, K};
                    Launch L;
                    if (!make_launch(discs, P, c, v, L, wj)) continue;  // shape does not exist
                    if (L.K == L0.K && sf == v0.sf && gm == v0.gm) continue;  // the reference itself
                    ++ncand;
                    st = tune_upload_wj(S, wj);
                    if (st != SG_OK) return st;
                    if (launch_one((const DiscDev *)S.dd, (const WJob *)S.wj, L, s) != SG_OK) return SG_ERR_HIP;
                    double rel = 1.0;
                    st = tune_compare(S, outs, s, rel);
                    if (st != SG_OK) return st;
                    if (rel > 1e-5) {  // a candidate must reproduce the reference first
                        ++nrej;
                        continue;
                    }
                    float ms = 0.f;
                    st = tune_time(S, L, s, reps, ms);
                    if (st != SG_OK) return st;
                    if (ms < ms_best) {
                        ms_best = ms;
                        best = v;
                        rel_best = rel;
                    }
                }
        // leave the class's outputs as the chosen variant writes them
        Launch Lb;
        make_launch(discs, P, c, best, Lb, wj);
        st = tune_upload_wj(S, wj);
        if (st != SG_OK) return st;
        if (launch_one((const DiscDev *)S.dd, (const WJob *)S.wj, Lb, s) != SG_OK) return SG_ERR_HIP;
        SG_HIP(hipStreamSynchronize(s));
        g_tuned[tune_key(discs, c)] = best;
        if (res && count < cap) {
            sg_tune_result &r = res[count];
            r.pass = c.pass;
            r.length = c.len;
            r.n_fluids = c.nf;
            r.n_jobs = Lb.nj;
            r.small_radix_first = best.sf;
            r.groups_per_wg = c.ss ? Lb.v.gm : Lb.k.G;
            r.cluster = Lb.K;
            r.candidates = ncand;
            r.rejected = nrej;
            r.rel_best = (float)rel_best;
            r.ms_default = ms0;
            r.ms_best = ms_best;
        }
        ++count;
    }
    if (nres) *nres = count;
    // cached plans were built before this tuning: rebuild on next use
    release_locked();
    save_tune_file();
    return SG_OK;
}

// Optional persistent cache: SG_TUNE_CACHE names a text file with one line
// "pass length fluids shape_hash sf gm K" per tuned class; read once, and
// rewritten after every tuning call.
static bool g_tune_file_loaded = false;

static void load_tune_file()
{
    if (g_tune_file_loaded) return;
    g_tune_file_loaded = true;
    const char *path = getenv("SG_TUNE_CACHE");
    if (!path || !path[0]) return;
    FILE *f = fopen(path, "r");
    if (!f) return;
    int pass, len, nf, sf, gm, K;
    unsigned long long h;
    while (fscanf(f, "%d %d %d %llx %d %d %d", &pass, &len, &nf, &h, &sf, &gm, &K) == 7)
        if (pass >= 1 && pass <= 3 && nf >= 1 && nf <= 4 && sf >= 0 && sf <= 1 && gm >= 1 && gm <= 4 &&
            (K == 0 || K == 1 || K == 2 || K == 4 || K == 8))
            g_tuned[TuneKey{pass, len, nf, (uint64_t)h}] = Variant{sf, gm, K};
    fclose(f);
}

static void save_tune_file()
{
    const char *path = getenv("SG_TUNE_CACHE");
    if (!path || !path[0]) return;
    FILE *f = fopen(path, "w");
    if (!f) return;
    for (const auto &kv : g_tuned)
        fprintf(f, "%d %d %d %llx %d %d %d\n", std::get<0>(kv.first), std::get<1>(kv.first),
                std::get<2>(kv.first), (unsigned long long)std::get<3>(kv.first), kv.second.sf, kv.second.gm,
                kv.second.K);
    fclose(f);
}
