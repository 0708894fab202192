// The spherical method (paper Sec. 4 eqs. DTensor, WTensor, YYY,
// SphericalMethod, RTensor; Sec. 5.4; App. B) on the device, FP64.
//
// Everything up to the coupling is in real harmonics S_lm (S_l0 = Y_l0, S_lm =
// (-1)^m sqrt(2) Re Y_l^m, S_l,-m = (-1)^m sqrt(2) Im Y_l^m, m > 0): the
// monomials and the plane wave are real in them up to i^lam and i^L, so the
// contraction over geometries is one real product instead of four.  Geometries
// (a primitive pair of a shell pair: one Gaussian centre P_g and exponent p_g)
// are sorted by l_A + l_B, largest first; a polynomial of degree l_A + l_B
// has harmonics lam <= l_A + l_B only, so rows of lam need the first ext[lam]
// geometries.  Together, for 10 heavy atoms (s, p, d shells), 12 states, lmax 24
// and 24 radii, a fourteenth of the operations of the complex contraction over
// all geometries and rows.
//
//   sph_geom_kernel    per geometry the W tensor summed over its component
//                      pairs with their packed transition weights,
//                        W^s_g[n lam mu] = sum_c Tp_s(c) sum_{u+v+w=n} e^x_u e^y_v e^z_w Theta^{uvw}_{lam mu}
//                      (real Theta), from the 1D rows of the pair precompute;
//   sph_ylm_kernel     4 pi S_LM(P^_g) for L <= lmax + 4;
//   sph_bessel_kernel  j_L(q |P_g|) (Miller's downward recurrence from far above
//                      max(L, x), normalised with j_0 = sin x / x or j_1,
//                      whichever is larger; the two-term power series below x =
//                      1e-4) and the Gaussian;
//   sph_b_kernel,      for each radius q, the contraction over geometries
//   sph_q_kernel         Q^s[lam mu][L M](q) = sum_g b^s_g[lam mu](q) a_g[L M](q),
//                        b = e^{-q^2/4p} sum_n (-1)^{(n-lam)/2} q^n W^s_g[n lam mu],
//                        a = 4 pi j_L(q |P_g|) S_LM(P^_g);
//   sph_couple_kernel  to complex harmonics (i^{lam+L} and the unitary mixing of
//                      +-mu and +-M), then
//                      R^s_lm(q) = sum_{lam mu, L} G^{mu, m-mu}_{lam L l} Q^s[lam mu][L, m-mu]
//                      (eq. RTensor with the Gaunt coefficients of eq. YYY);
//   sph_legendre_kernel / sph_phi_kernel
//                      the angular grid f^s(q, theta_i, phi_j) = sum_lm R_lm Y_l^m
//                      (eq. SphericalMethod) as a Legendre stage per theta and a
//                      Fourier stage per phi; sph_avg_kernel <|f|^2>_Omega.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "engine.h"

namespace scff {

namespace {

constexpr int kLam = (kSphMaxN + 1) * (kSphMaxN + 1);   // 25 harmonics lam <= 4
constexpr int kMaxHarm = kSphMaxL + kSphMaxN + 1;       // harmonic degrees, at most

__device__ __forceinline__ int lam_of(int li) { return li < 1 ? 0 : li < 4 ? 1 : li < 9 ? 2 : li < 16 ? 3 : 4; }

// Coefficients of the upward recurrence of the normalised associated Legendre
// functions (Condon-Shortley phase), P_l = a (cos P_{l-1} - b P_{l-2}), for
// m <= l <= L at [l (l + 1) / 2 + m]; at l = m: x = P_mm / (sin P_{m-1,m-1}).
__device__ void legendre_table(int L, double2* ab) {
    const int n = (L + 1) * (L + 2) / 2;
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
        int l = (int)((sqrt(8.0 * i + 1.0) - 1.0) * 0.5);
        while (l * (l + 1) / 2 > i) --l;
        while ((l + 1) * (l + 2) / 2 <= i) ++l;
        const int m = i - l * (l + 1) / 2;
        double2 v = make_double2(0.0, 0.0);
        if (l == m) {
            v.x = m ? -sqrt((2.0 * m + 1.0) / (2.0 * m)) : sqrt(1.0 / (4.0 * M_PI));
        } else if (l == m + 1) {
            v.x = sqrt(2.0 * m + 3.0);
        } else {
            v.x = sqrt((4.0 * l * l - 1.0) / ((double)l * l - (double)m * m));
            v.y = sqrt(((l - 1.0) * (l - 1.0) - (double)m * m) / (4.0 * (l - 1.0) * (l - 1.0) - 1.0));
        }
        ab[i] = v;
    }
}

// One wave per geometry, lane b = entry (n, lam, mu) of its W tensor; entries
// of n <= l_A + l_B only (the others are zero and never read).
// W[(b ns + s) n_geo + g].  A thread per geometry, which also walked its
// harmonics, took 3.2 ms (10 heavy atoms); this and sph_ylm_kernel 0.13 ms each.
__global__ __launch_bounds__(256) void sph_geom_kernel(const SphGeom* __restrict__ geo, int n_geo,
                                                       const VRowDev* __restrict__ rows,
                                                       const int4* __restrict__ trow,
                                                       const double* __restrict__ tp64, int ns,
                                                       const double* __restrict__ theta, const int* __restrict__ uvw_idx,
                                                       const int* __restrict__ nfirst, int n_nlm,
                                                       double4* __restrict__ gdat, double* __restrict__ W) {
    const int lane = threadIdx.x & 63, g = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
    if (g >= n_geo) return;
    const SphGeom G = geo[g];
    if (lane == 0) {
        const int4 t0 = trow[G.term0 + G.pp];
        const double Px = rows[t0.x].P, Py = rows[t0.y].P, Pz = rows[t0.z].P;
        const double d = sqrt(Px * Px + Py * Py + Pz * Pz);
        const double th = d > 0.0 ? acos(fmin(1.0, fmax(-1.0, Pz / d))) : 0.0;
        const double ph = d > 0.0 ? atan2(Py, Px) : 0.0;
        gdat[g] = make_double4(d, th, ph, rows[t0.x].inv4p);
    }
    const int nb = nfirst[G.lsum + 1], b = min(lane, nb - 1);
    double acc[kMaxStates];
#pragma unroll
    for (int s = 0; s < kMaxStates; ++s) acc[s] = 0.0;
    for (int c = 0; c < G.ncp; ++c) {
        const int4 tr = trow[G.term0 + c * G.npp + G.pp];
        const VRowDev& rx = rows[tr.x];
        const VRowDev& ry = rows[tr.y];
        const VRowDev& rz = rows[tr.z];
        double x = 0.0;
        for (int u = 0; u <= rx.deg; ++u)
            for (int v = 0; v <= ry.deg; ++v)
                for (int w = 0; w <= rz.deg; ++w) {   // Theta is zero where n is not u + v + w
                    const int a = uvw_idx[(u * (kSphMaxN + 1) + v) * (kSphMaxN + 1) + w];
                    x = fma(rx.e[u] * ry.e[v] * rz.e[w], theta[(size_t)a * n_nlm + b], x);
                }
        const double* tp = tp64 + (size_t)tr.w * ns;
#pragma unroll
        for (int s = 0; s < kMaxStates; ++s)
            if (s < ns) acc[s] = fma(tp[s], x, acc[s]);
    }
    if (lane >= nb) return;
#pragma unroll
    for (int s = 0; s < kMaxStates; ++s)
        if (s < ns) W[((size_t)b * ns + s) * n_geo + g] = acc[s];
}

// Y[g ncols + L^2 + L + M] = 4 pi S_LM(P^_g).  Lane m of a group walks l, so
// the lanes' writes of one l are neighbours.
__global__ __launch_bounds__(256) void sph_ylm_kernel(const double4* __restrict__ gdat, int n_geo, int Lmax,
                                                      double* __restrict__ Y) {
    __shared__ double2 ab[kMaxHarm * (kMaxHarm + 1) / 2];
    legendre_table(Lmax, ab);
    __syncthreads();
    const int gsz = Lmax < 32 ? 32 : 64, per = 256 / gsz;
    const int m = threadIdx.x & (gsz - 1), ncols = (Lmax + 1) * (Lmax + 1);
    if (m > Lmax) return;
    for (int g = blockIdx.x * per + threadIdx.x / gsz; g < n_geo; g += gridDim.x * per) {
        const double4 gg = gdat[g];
        double sn, cs, es, ec;
        sincos(gg.y, &sn, &cs);
        sincos(m * gg.z, &es, &ec);
        double pmm = ab[0].x;
        for (int k = 1; k <= m; ++k) pmm *= ab[k * (k + 1) / 2 + k].x * sn;
        const double f = 4.0 * M_PI * (m ? ((m & 1) ? -M_SQRT2 : M_SQRT2) : 1.0);
        ec *= f;
        es *= f;
        double* o = Y + (size_t)g * ncols;
        double p2 = 0.0, p1 = pmm;
        for (int l = m; l <= Lmax; ++l) {
            double cur = pmm;
            if (l > m) {
                const double2 k = ab[l * (l + 1) / 2 + m];
                cur = k.x * (cs * p1 - k.y * p2);
                p2 = p1;
                p1 = cur;
            }
            o[l * l + l + m] = cur * ec;
            if (m) o[l * l + l - m] = cur * es;
        }
    }
}

// Spherical Bessel functions and Gaussian of every (radius, geometry):
// J[(iq (Lmax + 2) + L) gs + g] = j_L(q |P_g|) for L <= Lmax and, at
// L = Lmax + 1, e^{-q^2 / 4p_g}; geometries padded to gs (copies of the last
// one: finite factors of zero rows).  One thread per (radius, geometry); the
// recurrence is written straight to the strided table.
__global__ void sph_bessel_kernel(const double4* __restrict__ gdat, int n_geo, int gs, int Lmax, const double* __restrict__ qs,
                                  int n_q, double* __restrict__ J) {
    const long long idx = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (idx >= (long long)n_q * gs) return;
    const int g = (int)(idx % gs), iq = (int)(idx / gs);
    const double4 gg = gdat[min(g, n_geo - 1)];
    const double q = qs[iq], x = q * gg.x;
    double* o = J + (size_t)iq * (Lmax + 2) * gs + g;
    o[(size_t)(Lmax + 1) * gs] = exp(-q * q * gg.w);
    if (x < 1e-4) {
        double df = 1.0, xl = 1.0;
        for (int L = 0; L <= Lmax; ++L) {
            if (L > 0) {
                df *= 2.0 * L + 1.0;
                xl *= x;
            }
            o[(size_t)L * gs] = xl / df * (1.0 - x * x / (2.0 * (2.0 * L + 3.0)));
        }
        return;
    }
    const int N = max(Lmax, (int)x) + 32;
    const double rx = 1.0 / x;
    double fp = 0.0, f = 1e-280, f1 = 0.0;
    for (int L = N; L >= 1; --L) {
        const double fm = (2.0 * L + 1.0) * rx * f - fp;   // f_{L-1}
        fp = f;
        f = fm;
        if (L - 1 <= Lmax) o[(size_t)(L - 1) * gs] = f;
        if (L - 1 == 1) f1 = f;
        if (fabs(f) > 1e250) {   // rescale everything kept so far
            f *= 1e-250;
            fp *= 1e-250;
            f1 *= 1e-250;
            for (int k = L - 1; k <= Lmax; ++k) o[(size_t)k * gs] *= 1e-250;
        }
    }
    double sn, cs;
    sincos(x, &sn, &cs);
    const double j0 = sn * rx, j1 = (sn * rx - cs) * rx;
    const double scale = fabs(j0) >= fabs(j1) ? j0 / f : j1 / f1;
    for (int L = 0; L <= Lmax; ++L) o[(size_t)L * gs] *= scale;
}

// Row operands of the contraction for a batch of nqb radii from iq0 on,
//   Bq[(k nrows + row) gs + g] = e^{-q^2/4p_g} sum_n (-1)^{(n-lam)/2} q^n W^s_g[n lam mu],
// row = (lam mu) ns + s, q = qs[iq0 + k], for the geometries that the row's tile
// of kQRows rows runs over (zero past the row's own, ext[lam]); the Gaussian is
// row Lmax + 1 of the radius's Bessel table.  One thread per (row, geometry): its
// W values (n = lam, lam + 2, .. <= 4) are loaded once for the batch.
constexpr int kQRows = 32, kQCols = 128, kQK = 16, kQRadii = 4;

__device__ __forceinline__ int tile_extent(const SphExt& ext, int tile, int ns) {
    return ext.n[lam_of(tile * kQRows / ns)];
}

__global__ __launch_bounds__(256) void sph_b_kernel(const double* __restrict__ W, const double* __restrict__ J,
                                                    const int* __restrict__ nlm_of, SphExt ext, int n_geo, int gs, int ns,
                                                    int Lmax, const double* __restrict__ qs, int iq0, int nqb,
                                                    double* __restrict__ Bq) {
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    const int row = blockIdx.y, nrows = ns * kLam;
    if (g >= ((tile_extent(ext, row / kQRows, ns) + kQK - 1) & ~(kQK - 1))) return;
    const int li = row / ns, st = row - li * ns, lam = lam_of(li);
    // slots m = 0..2 hold n = lam + 2 m (those the geometry has not are zero)
    double w[3];
#pragma unroll
    for (int m = 0; m < 3; ++m) {
        const int n = lam + 2 * m;
        w[m] = n <= kSphMaxN && g < ext.n[n] ? W[((size_t)nlm_of[n * kLam + li] * ns + st) * n_geo + g] : 0.0;
    }
    for (int k = 0; k < nqb; ++k) {
        const int iq = iq0 + k;
        const double q = qs[iq], q2 = q * q;
        const double ga = J[((size_t)iq * (Lmax + 2) + Lmax + 1) * gs + g];
        double p = ga;
        for (int n = 0; n < lam; ++n) p *= q;
        Bq[((size_t)k * nrows + row) * gs + g] = p * fma(q2, fma(q2, w[2], -w[1]), w[0]);
    }
}

// Tile: 32 rows x 128 columns (L M) x 4 radii (one per wave) per workgroup, a
// segment of the geometries in chunks of 16, on the FP64 matrix cores
// (v_mfma_f64_16x16x4_f64: lane l holds A[l % 16][l / 16], B[l / 16][l % 16] and
// the results D[4 i + l / 16][l % 16], i = 0..3).  The harmonics of a chunk do
// not depend on the radius: the waves share them in LDS and multiply each value
// by their own j_L on the way into the matrix cores, one product for two row
// blocks.  Row operand and j_L are the wave's own.  The loads of the next chunk
// are in flight while the current one is multiplied.  The tile's second 16 rows
// stop at their own extent.  Row tiles of long extents
// (small lam: few rows, most geometries) are cut into segments, so that all
// items are about equally long; their partial sums are added in order by
// sph_sum_kernel.  10 heavy atoms, 12 states, lmax 24, 24 radii: 29.9 ms (complex,
// all rows over all geometries) -> 2.4 ms, bound by the matrix cores (63 % busy
// with both blocks over the tile's extent, 2.67 ms) and the last round of
// workgroups; at one wave per SIMD (304 registers) 3.0 ms.
typedef double sph_double4 __attribute__((ext_vector_type(4)));
constexpr int kQLs = 12;   // degrees that 128 columns span, at most

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void sph_q_kernel(const double* __restrict__ J, const double* __restrict__ Y,
                                                    const double* __restrict__ Bq, const SphItem* __restrict__ items,
                                                    int n_geo, int gs, int nrows, int Lmax, int iq0, int nqb, int n_q,
                                                    double* __restrict__ Q, double* __restrict__ P) {
    __shared__ double Ys[kQK][kQCols + 1];
    __shared__ double As[kQRadii][kQRows][kQK + 1];
    __shared__ double Js[kQRadii][kQLs * (kQK + 1)];
    constexpr int NC = kQCols / 16;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane & 15, lk = lane >> 4;
    const int ncols = (Lmax + 1) * (Lmax + 1);
    const SphItem it = items[blockIdx.y];
    const int r0 = it.tile * kQRows, c0 = blockIdx.x * kQCols;
    const int kq = blockIdx.z * kQRadii + wave, kc = min(kq, nqb - 1);   // radius of the batch (clamped)

    // harmonics: column tid % 128 at geometries tid / 128 + 2 j
    const int cy = tid & (kQCols - 1), ky = tid >> 7;
    const double* Yc = Y + min(c0 + cy, ncols - 1);
    // row operand: row lane / 2, eight geometries from 8 (lane % 2)
    const int ra = lane >> 1, ka = 8 * (lane & 1);
    const double* Br = Bq + ((size_t)kc * nrows + min(r0 + ra, nrows - 1)) * gs + ka;
    // j_L: degrees L0 .. of the tile, entry (lane + 64 j) / 16 at geometry lane % 16
    const int L0 = (int)sqrt((double)c0 + 0.5), nL = (int)sqrt((double)min(c0 + kQCols - 1, ncols - 1) + 0.5) - L0 + 1;
    const double* Jq = J + (size_t)(iq0 + kc) * (Lmax + 2) * gs + (lane & 15);
    int jo[NC];
#pragma unroll
    for (int cb = 0; cb < NC; ++cb)
        jo[cb] = ((int)sqrt((double)min(c0 + 16 * cb + lr, ncols - 1) + 0.5) - L0) * (kQK + 1) + lk;

    sph_double4 acc[2][NC];
#pragma unroll
    for (int cb = 0; cb < NC; ++cb) acc[0][cb] = acc[1][cb] = (sph_double4){0.0, 0.0, 0.0, 0.0};
    double y[8], a[8], jl[3];
    auto load = [&](int g0) {
#pragma unroll
        for (int j = 0; j < 8; ++j) y[j] = Yc[(size_t)min(g0 + ky + 2 * j, n_geo - 1) * ncols];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const double2 v = *reinterpret_cast<const double2*>(Br + g0 + 2 * j);
            a[2 * j] = v.x;
            a[2 * j + 1] = v.y;
        }
#pragma unroll
        for (int j = 0; j < 3; ++j) jl[j] = Jq[(size_t)(L0 + min((lane >> 4) + 4 * j, nL - 1)) * gs + g0];
    };
    auto chunk = [&](int g0, auto both) {
        constexpr bool BOTH = decltype(both)::value;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            Ys[ky + 2 * j][cy] = y[j];
            As[wave][ra][ka + j] = a[j];
        }
#pragma unroll
        for (int j = 0; j < 3; ++j) Js[wave][((lane >> 4) + 4 * j) * (kQK + 1) + (lane & 15)] = jl[j];
        __syncthreads();
        if (g0 + kQK < it.k1) load(g0 + kQK);
#pragma unroll
        for (int ks = 0; ks < kQK / 4; ++ks) {
            const double a0 = As[wave][lr][4 * ks + lk], a1 = BOTH ? As[wave][16 + lr][4 * ks + lk] : 0.0;
#pragma unroll
            for (int cb = 0; cb < NC; ++cb) {
                const double b = Ys[4 * ks + lk][16 * cb + lr] * Js[wave][jo[cb] + 4 * ks];
                acc[0][cb] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b, acc[0][cb], 0, 0, 0);
                if (BOTH) acc[1][cb] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b, acc[1][cb], 0, 0, 0);
            }
        }
        __syncthreads();
    };
    load(it.k0);
    int g0 = it.k0;
    for (; g0 < min(it.k1, it.kb); g0 += kQK) chunk(g0, std::true_type{});
    for (; g0 < it.k1; g0 += kQK) chunk(g0, std::false_type{});
    if (kq >= nqb) return;
    const int iq = iq0 + kq;
    double* out = it.part < 0 ? Q + ((size_t)iq * nrows + r0) * ncols : P + ((size_t)it.part * n_q + iq) * kQRows * ncols;
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int cb = 0; cb < NC; ++cb)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int r = 16 * h + 4 * i + lk, col = c0 + 16 * cb + lr;
                if (r0 + r < nrows && col < ncols) out[(size_t)r * ncols + col] = acc[h][cb][i];
            }
}

// Q of the first n_tiles row tiles from their segments' partial sums.
__global__ __launch_bounds__(256) void sph_sum_kernel(const double* __restrict__ P, SphSegs segs, int nrows, int ncols,
                                                      int n_q, double* __restrict__ Q) {
    const int tile = blockIdx.z, iq = blockIdx.y;
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= min(kQRows, nrows - tile * kQRows) * ncols) return;
    const size_t ps = (size_t)n_q * kQRows * ncols;
    const double* p = P + (size_t)segs.first[tile] * ps + (size_t)iq * kQRows * ncols + i;
    double v = 0.0;
    for (int k = segs.first[tile]; k < segs.first[tile + 1]; ++k, p += ps) v += *p;
    Q[((size_t)iq * nrows + tile * kQRows) * ncols + i] = v;
}

__global__ void sph_couple_kernel(const double* __restrict__ Q, const double* __restrict__ gaunt, int ns, int lmax,
                                  int Lmax, int n_q, double2* __restrict__ R) {
    const int nl = (lmax + 1) * (lmax + 1), ncols = (Lmax + 1) * (Lmax + 1), nrows = ns * kLam;
    const long long idx = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (idx >= (long long)ns * n_q * nl) return;
    const int lm = (int)(idx % nl);
    const long long r1 = idx / nl;
    const int iq = (int)(r1 % n_q), s = (int)(r1 / n_q);
    const int l = (int)sqrt((double)lm + 0.5), m = lm - l * l - l;
    double2 acc = make_double2(0.0, 0.0);
    for (int lam = 0; lam <= kSphMaxN; ++lam)
        for (int mu = -lam; mu <= lam; ++mu) {
            const int li = lam * lam + lam + mu, am = abs(mu), M = m - mu, aM = abs(M);
            const double* Qp = Q + ((size_t)iq * nrows + (size_t)(lam * lam + lam + am) * ns + s) * ncols;
            const double* Qm = Q + ((size_t)iq * nrows + (size_t)(lam * lam + lam - am) * ns + s) * ncols;
            const double* gr = gaunt + ((size_t)li * nl + lm) * kSphGauntJ;
            // Y_mu's share of S_|mu| and S_-|mu| is k (1, i e): e = -1, k = (-1)^mu / sqrt 2
            // for mu > 0, e = 1, k = 1 / sqrt 2 for mu < 0, (1, 0) for mu = 0; M alike
            const double em = mu > 0 ? -1.0 : mu < 0 ? 1.0 : 0.0, eM = M > 0 ? -1.0 : M < 0 ? 1.0 : 0.0;
            const double k = (mu ? (mu > 0 && (mu & 1) ? -M_SQRT1_2 : M_SQRT1_2) : 1.0) *
                             (M ? (M > 0 && (M & 1) ? -M_SQRT1_2 : M_SQRT1_2) : 1.0);
            double2 sum = make_double2(0.0, 0.0);   // over L = |l - lam| + 2 j, with i^{2 j}
            double sg = k;
            for (int j = 0; j < kSphGauntJ; ++j, sg = -sg) {
                const int L = abs(l - lam) + 2 * j;
                if (L > l + lam) break;
                if (aM > L) continue;
                const int cp = L * L + L + aM, cm = L * L + L - aM;
                const double gv = sg * gr[j];
                sum.x = fma(gv, Qp[cp] - em * eM * Qm[cm], sum.x);
                sum.y = fma(gv, eM * Qp[cm] + em * Qm[cp], sum.y);
            }
            switch ((lam + abs(l - lam)) & 3) {   // i^{lam + L} at j = 0
                case 0: acc.x += sum.x; acc.y += sum.y; break;
                case 1: acc.x -= sum.y; acc.y += sum.x; break;
                case 2: acc.x -= sum.x; acc.y -= sum.y; break;
                default: acc.x += sum.y; acc.y -= sum.x; break;
            }
        }
    R[((size_t)s * n_q + iq) * nl + lm] = acc;
}

// F^s(q, theta_i, m) = sum_{l >= |m|} R^s_lm(q) P~_l^m(cos theta_i), with
// Y_l^m = P~_l^m(cos theta) e^{i m phi} (P~ the normalised associated Legendre
// function with the Condon-Shortley phase; P~_l^{-m} = (-1)^m P~_l^m).  Blocks of
// kLegStates states per thread share the recurrence.
constexpr int kLegStates = 4;
__global__ __launch_bounds__(256) void sph_legendre_kernel(const double2* __restrict__ R, int ns, int lmax, int n_q,
                                                           int n_theta, double2* __restrict__ F) {
    __shared__ double2 ab[kMaxHarm * (kMaxHarm + 1) / 2];
    legendre_table(lmax, ab);
    __syncthreads();
    const int nm = 2 * lmax + 1, nl = (lmax + 1) * (lmax + 1);
    const long long idx = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (idx >= (long long)n_q * n_theta * nm) return;
    const int mi = (int)(idx % nm);
    const long long r1 = idx / nm;
    const int it = (int)(r1 % n_theta), iq = (int)(r1 / n_theta);
    const int m = mi - lmax, am = abs(m);
    const double theta = n_theta > 1 ? M_PI * it / (n_theta - 1) : 0.0;
    double sn, cs;
    sincos(theta, &sn, &cs);
    double pmm = ab[0].x;
    for (int k = 1; k <= am; ++k) pmm *= ab[k * (k + 1) / 2 + k].x * sn;
    if (m < 0 && (am & 1)) pmm = -pmm;
    const int s0 = blockIdx.y * kLegStates;
    const double2* Rs = R + ((size_t)s0 * n_q + iq) * nl + m;
    double2 acc[kLegStates];
#pragma unroll
    for (int s = 0; s < kLegStates; ++s) acc[s] = make_double2(0.0, 0.0);
    double p2 = 0.0, p1 = pmm;
    for (int l = am; l <= lmax; ++l) {
        double cur = pmm;
        if (l > am) {
            const double2 k = ab[l * (l + 1) / 2 + am];
            cur = k.x * (cs * p1 - k.y * p2);
            p2 = p1;
            p1 = cur;
        }
#pragma unroll
        for (int s = 0; s < kLegStates; ++s)
            if (s0 + s < ns) {
                const double2 r = Rs[(size_t)s * n_q * nl + l * l + l];
                acc[s].x = fma(cur, r.x, acc[s].x);
                acc[s].y = fma(cur, r.y, acc[s].y);
            }
    }
#pragma unroll
    for (int s = 0; s < kLegStates; ++s)
        if (s0 + s < ns) F[((((size_t)s0 + s) * n_q + iq) * n_theta + it) * nm + mi] = acc[s];
}

// f^s(q, theta_i, phi_j) = sum_m F^s(q, theta_i, m) e^{i m phi_j}, phi_j = 2 pi j / n_phi:
// a polynomial in e^{i phi} (Horner), times e^{-i lmax phi}.
__global__ void sph_phi_kernel(const double2* __restrict__ F, int ns, int lmax, int n_q, int n_theta, int n_phi,
                               float2* __restrict__ f, float* __restrict__ f2) {
    const int nm = 2 * lmax + 1;
    const long long npts = (long long)n_q * n_theta * n_phi;
    const long long idx = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (idx >= npts) return;
    const int jp = (int)(idx % n_phi), s = blockIdx.y;
    const long long r1 = idx / n_phi;   // q, theta
    double es, ec, bs, bc;
    sincospi(2.0 * jp / n_phi, &es, &ec);
    sincospi(2.0 * (((long long)jp * lmax) % n_phi) / n_phi, &bs, &bc);
    const double2* Fs = F + ((size_t)s * n_q * n_theta + r1) * nm;
    double2 a = Fs[nm - 1];
    for (int mi = nm - 2; mi >= 0; --mi) {
        const double2 v = Fs[mi];
        const double re = fma(-a.y, es, fma(a.x, ec, v.x));
        a.y = fma(a.y, ec, fma(a.x, es, v.y));
        a.x = re;
    }
    const double2 acc = make_double2(a.x * bc + a.y * bs, a.y * bc - a.x * bs);
    const size_t o = (size_t)s * npts + idx;
    if (f) f[o] = make_float2((float)acc.x, (float)acc.y);
    if (f2) f2[o] = (float)(acc.x * acc.x + acc.y * acc.y);
}

// One wave per (state, radius).
__global__ __launch_bounds__(256) void sph_avg_kernel(const double2* __restrict__ R, int n, int lmax,
                                                      double* __restrict__ avg) {
    const int nl = (lmax + 1) * (lmax + 1);
    const int idx = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (idx >= n) return;
    const double2* Rs = R + (size_t)idx * nl;
    double a = 0.0;
    for (int i = lane; i < nl; i += 64) a = fma(Rs[i].x, Rs[i].x, fma(Rs[i].y, Rs[i].y, a));
    for (int h = 32; h > 0; h >>= 1) a += __shfl_xor(a, h);
    if (lane == 0) avg[idx] = a / (4.0 * M_PI);
}

}  // namespace

hipError_t launch_sph_geom(const SphGeom* geo, int n_geo, const VRowDev* rows, const int4* trow, const double* tp64,
                           int ns, const double* theta, const int* uvw_idx, const int* nfirst, int n_nlm, int Lmax,
                           double4* gdat, double* Y, double* W, hipStream_t st) {
    if (n_geo <= 0) return hipSuccess;
    if (ns > kMaxStates || n_nlm > 64 || Lmax >= kMaxHarm) return hipErrorInvalidValue;
    hipLaunchKernelGGL(sph_geom_kernel, dim3((n_geo + 3) / 4), dim3(256), 0, st, geo, n_geo, rows, trow, tp64, ns,
                       theta, uvw_idx, nfirst, n_nlm, gdat, W);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(sph_ylm_kernel, dim3(std::min((n_geo + 7) / 8, 1024)), dim3(256), 0, st, gdat, n_geo, Lmax, Y);
    return hipGetLastError();
}

// Row tiles and their segments: items of about equal work (products of 16 rows and
// 16 geometries), enough for six workgroups per CU over the
// column tiles and radii, of at least 32 products each; split = false: one segment
// per tile.
void sph_plan(const SphExt& ext, int ns, int Lmax, int n_q, int n_cu, bool split, std::vector<SphItem>& items, SphSegs& segs) {
    const int nrows = ns * kLam, ncols = (Lmax + 1) * (Lmax + 1), tiles = (nrows + kQRows - 1) / kQRows;
    auto chunks = [&](int row) {   // extent of 16 rows from `row`
        if (row >= nrows) return 0;
        int l = 0;
        while ((l + 1) * (l + 1) <= row / ns) ++l;
        return (ext.n[l] + kQK - 1) / kQK;
    };
    long long total = 0;
    for (int r = 0; r < nrows; r += 16) total += chunks(r);
    const long long wgs = (long long)((ncols + kQCols - 1) / kQCols) * ((n_q + kQRadii - 1) / kQRadii);
    const long long want = std::max<long long>(1, 6LL * n_cu / wgs), len = std::max<long long>(32, (total + want - 1) / want);
    items.clear();
    segs.n_split = 0;
    int parts = 0;
    for (int t = 0; t < tiles; ++t) {
        const int k = chunks(t * kQRows), kb = chunks(t * kQRows + 16);   // kb <= k: extents fall with lam
        const int n = split ? std::max(1, (int)((k + kb + len - 1) / len)) : 1;
        // the chunk at which j / n of the tile's products are done
        auto at = [&](int j) {
            const long long w = ((long long)k + kb) * j / n;
            return (int)(w <= 2 * kb ? w / 2 : w - kb);
        };
        int used = 0;
        for (int j = 0; j < n; ++j) used += at(j + 1) > at(j);
        if (used > 1) {   // extents fall with the tile, too: the tiles that are cut come first
            segs.first[segs.n_split++] = parts;
            for (int j = 0; j < n; ++j)
                if (at(j + 1) > at(j)) items.push_back({t, at(j) * kQK, at(j + 1) * kQK, kb * kQK, parts++});
        } else {
            items.push_back({t, 0, k * kQK, kb * kQK, -1});
        }
    }
    segs.first[segs.n_split] = parts;
}

hipError_t launch_sph_q(const double4* gdat, const double* Y, const double* W, const SphExt& ext, int n_geo, int ns,
                        int Lmax, const int* nlm_of, const double* qs, int n_q, double* J, double* Bq, int nqb,
                        const SphItem* items, int n_items, const SphSegs& segs, double* Q, double* P, hipStream_t st) {
    if (nqb < 1 || n_items < 1 || n_items > 65535 || (segs.n_split && !P)) return hipErrorInvalidValue;
    const int gs = sph_geo_stride(n_geo);
    const long long nb = (long long)n_q * gs;
    hipLaunchKernelGGL(sph_bessel_kernel, dim3((unsigned)((nb + 255) / 256)), dim3(256), 0, st, gdat, n_geo, gs, Lmax, qs,
                       n_q, J);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int nrows = ns * kLam, ncols = (Lmax + 1) * (Lmax + 1);
    if (nrows > 65535) return hipErrorInvalidValue;
    for (int iq0 = 0; iq0 < n_q; iq0 += nqb) {
        const int nk = std::min(nqb, n_q - iq0);
        hipLaunchKernelGGL(sph_b_kernel, dim3((gs + 255) / 256, nrows), dim3(256), 0, st, W, J, nlm_of, ext, n_geo, gs, ns,
                           Lmax, qs, iq0, nk, Bq);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        hipLaunchKernelGGL(sph_q_kernel, dim3((ncols + kQCols - 1) / kQCols, n_items, (nk + kQRadii - 1) / kQRadii),
                           dim3(256), 0, st, J, Y, Bq, items, n_geo, gs, nrows, Lmax, iq0, nk, n_q, Q, P);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    if (segs.n_split)
        hipLaunchKernelGGL(sph_sum_kernel, dim3((kQRows * ncols + 255) / 256, n_q, segs.n_split), dim3(256), 0, st, P,
                           segs, nrows, ncols, n_q, Q);
    return hipGetLastError();
}

hipError_t launch_sph_couple(const double* Q, const double* gaunt, int ns, int lmax, int Lmax, int n_q, double2* R,
                             hipStream_t st) {
    const long long n = (long long)ns * n_q * (lmax + 1) * (lmax + 1);
    hipLaunchKernelGGL(sph_couple_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, Q, gaunt, ns, lmax, Lmax,
                       n_q, R);
    return hipGetLastError();
}

hipError_t launch_sph_grid(const double2* R, int ns, int lmax, int n_q, int n_theta, int n_phi, double2* F, float2* f,
                           float* f2, hipStream_t st) {
    const long long n1 = (long long)n_q * n_theta * (2 * lmax + 1);
    hipLaunchKernelGGL(sph_legendre_kernel, dim3((unsigned)((n1 + 255) / 256), (ns + kLegStates - 1) / kLegStates),
                       dim3(256), 0, st, R, ns, lmax, n_q, n_theta, F);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const long long n2 = (long long)n_q * n_theta * n_phi;
    hipLaunchKernelGGL(sph_phi_kernel, dim3((unsigned)((n2 + 255) / 256), ns), dim3(256), 0, st, F, ns, lmax, n_q,
                       n_theta, n_phi, f, f2);
    return hipGetLastError();
}

hipError_t launch_sph_avg(const double2* R, int ns, int lmax, int n_q, double* avg, hipStream_t st) {
    const int n = ns * n_q;
    hipLaunchKernelGGL(sph_avg_kernel, dim3((n + 3) / 4), dim3(256), 0, st, R, n, lmax, avg);
    return hipGetLastError();
}

}  // namespace scff
