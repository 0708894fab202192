// Device-side pair precompute and packing (FP64) of the form-factor engine.
//
// Paper Sec. 5.3: the q-independent pair coefficients (eqs. sigmaTidbits,
// positionTidbits, bCoefficients, Mij) are computed once per molecule and
// reused; eq. Ccoefficients gives the monomial form of each 1D polynomial.
// Sec. 5.3 also thresholds Cartesian pair terms per transition; here the
// threshold acts on a q-independent magnitude bound so the dropped part is
// controlled.  Everything below runs on the device from device-resident T:
//
//   rows_terms_kernel
//                   one 1D V-tensor row per (primitive pair, axis, power
//                   pair): P, 1/(4p), e_u (all q-independent factors folded),
//                   and its bound sum_u |e_u| max_q |q|^u e^{-q^2/4p}; per
//                   (component pair, primitive pair) term: its 3 rows and
//                   bound; per component pair Tp(s) = (T_mn + T_nm) c_m c_n s_f;
//                   per shell pair the partial sums of |Tp| * bound
//   tot_kernel      tot_s = sum over all terms of |Tp(s)| * bound
//   weight_kernel   w(t) = max_s |Tp(s)| bound(t) / tot_s, integer histogram
//                   of binary exponents
//   thresh_kernel   largest 2^b with sum_{e <= b} count_e 2^e <= eps: dropping
//                   every w < 2^b keeps, for every transition, the dropped
//                   bounds below eps * tot_s
// Grid kernel's layout (run_prep, run_prep_layout), by the contracted axis, called z
// here whichever of the grid's it is:
//   zcount_kernel   kept terms of every z row (one per primitive pair and
//                   power pair of the axis), flags of the referenced rows, and
//                   per state the largest bound of a row's contribution
//   scan            one scan numbers the rows (a zero row, the x and y rows,
//                   the z rows) and sorts the z rows by term count (most terms
//                   first, ties in row order)
//   zmeta_kernel    scales of the states; what the host reads back, once
//   zlayout_kernel  rows compacted; z rows in k-steps of 32: their term
//                   records (x row, y row), scaled weights and scales
// Small problems are bound by the number of launches and copies: 29 before, 15
// now for a 4-heavy-atom, one-state, 32^3 grid with its tables (200 -> 147 us).
// Layout by component pairs, for the export (run_prep_pairs):
//   count/vkeys     kept terms per component pair, split into virtual pairs
//                   of <= 9 terms, keyed by length (longest first, ties in pair
//                   order)
//   unit/layout     units of 8 virtual pairs, term slots, packed FP32 Tp
#include <hip/hip_runtime.h>
#include <hipcub/hipcub.hpp>

#include <algorithm>
#include <cstring>
#include <cstdint>

#include "engine.h"

namespace scff {

namespace {

__device__ __constant__ int kCartD[3][6][3] = {
    {{0, 0, 0}},
    {{1, 0, 0}, {0, 1, 0}, {0, 0, 1}},
    {{2, 0, 0}, {1, 1, 0}, {1, 0, 1}, {0, 2, 0}, {0, 1, 1}, {0, 0, 2}},
};

__device__ __forceinline__ int ncart_d(int l) { return (l + 1) * (l + 2) / 2; }

// (u + 2m)! / (m! u! 2^m), u + 2m <= 4
__device__ __forceinline__ double hmono(int u, int m) {
    const double f[5] = {1, 1, 2, 6, 24};
    return f[u + 2 * m] / (f[m] * f[u] * (double)(1 << m));
}

// component pair index within a shell pair -> (c1, c2)
__device__ __forceinline__ void cp_decode(int c, bool same, int ncB, int& c1, int& c2) {
    if (!same) {
        c1 = c / ncB;
        c2 = c - c1 * ncB;
        return;
    }
    // triangular: pairs (c1 <= c2) in row-major order
    int row = 0, rem = c;
    while (rem >= ncB - row) {
        rem -= ncB - row;
        ++row;
    }
    c1 = row;
    c2 = row + rem;
}

constexpr int kHistBias = 1100;   // binary exponents -1100 .. +99
constexpr int kHistBins = 1200;

}  // namespace

// ------------------------------------------------------------------ kernels

// One workgroup per shell pair: its rows, then its terms and component pairs
// (which need the bounds of its own rows only), and the pair's share of tot.
__global__ __launch_bounds__(128) void rows_terms_kernel(
    const PrepShell* __restrict__ sh, const int4* __restrict__ sp, const double* __restrict__ xyz,
    const double* __restrict__ exps, const double* __restrict__ coefs, const double* __restrict__ n1d, int nr,
    const int* __restrict__ sp_cp, const int* __restrict__ bf0, const double* __restrict__ cnorm,
    const double* __restrict__ T, int nbf, int ns, double spin, VRowDev* __restrict__ rows, double* __restrict__ rowsum,
    int* __restrict__ used, unsigned* __restrict__ small, int nsmall, int4* __restrict__ trow,
    double* __restrict__ tbound, double* __restrict__ tp64, double* __restrict__ bsum,
    double* __restrict__ part) {
    const int isp = blockIdx.x;
    const int4 s = sp[isp];   // sA, sB, row_off, term_off
    const PrepShell A_ = sh[s.x], B_ = sh[s.y];
    const int lA = A_.l, lB = B_.l, npb = B_.nprim;
    const int ncls = (lA + 1) * (lB + 1);
    const int nrows = A_.nprim * npb * 3 * ncls;
    const double* A = xyz + 3 * A_.atom;
    const double* B = xyz + 3 * B_.atom;
    const double AB2 = (A[0] - B[0]) * (A[0] - B[0]) + (A[1] - B[1]) * (A[1] - B[1]) + (A[2] - B[2]) * (A[2] - B[2]);
    for (int r = threadIdx.x; r < nrows; r += blockDim.x) {
        const int cls = r % ncls;
        const int ax = (r / ncls) % 3;
        const int pp = r / (3 * ncls);
        const int k = pp / npb, l = pp - k * npb;
        const int i = cls / (lB + 1), j = cls - i * (lB + 1);
        const int ka = A_.off + k, lb = B_.off + l;
        const double al = exps[ka], be = exps[lb];
        const double p = al + be, inv2p = 0.5 / p;
        const double P = (al * A[ax] + be * B[ax]) / p;     // eq. positionTidbits
        const double PA = P - A[ax], PB = P - B[ax];
        const double pa[3] = {1.0, PA, PA * PA}, pb[3] = {1.0, PB, PB * PB};
        const double bin[3][3] = {{1, 0, 0}, {1, 1, 0}, {1, 2, 1}};
        // b_t: coefficients of y^t in (y + PA)^i (y + PB)^j (eq. bCoefficients)
        double bt[5] = {0, 0, 0, 0, 0};
        for (int k1 = 0; k1 <= i; ++k1)
            for (int k2 = 0; k2 <= j; ++k2) bt[k1 + k2] += bin[i][k1] * bin[j][k2] * pa[i - k1] * pb[j - k2];
        // scale: 1D primitive norms; on x also d_k d_l (pi/p)^{3/2} e^{-al be/p |AB|^2} (eq. Mij)
        double scale = n1d[3 * ka + i] * n1d[3 * lb + j];
        if (ax == 0) scale *= coefs[ka] * coefs[lb] * (M_PI / p) * sqrt(M_PI / p) * exp(-al * be / p * AB2);
        VRowDev out{};
        out.P = P;
        out.inv4p = 0.25 / p;
        out.deg = i + j;
        out.axis = ax;
        double sum = 0.0;
        for (int u = 0; u <= i + j; ++u) {
            // e_u of eq. Ccoefficients with sigma_ij^2 = 1/(2p), divided by i^u
            double e = 0.0, pw = 1.0;
            for (int q = 0; q < u; ++q) pw *= inv2p;
            for (int m = 0; u + 2 * m <= i + j; ++m) {
                e += bt[u + 2 * m] * hmono(u, m) * pw;
                pw *= inv2p;
            }
            out.e[u] = e * scale;
            // max_q |q|^u exp(-q^2/(4p)) = (2 p u / e)^{u/2}
            const double mpk = u == 0 ? 1.0 : pow(2.0 * p * u / M_E, 0.5 * u);
            sum += fabs(out.e[u]) * mpk;
        }
        rows[s.z + r] = out;
        rowsum[s.z + r] = sum;
        for (int k = 0; k < 3; ++k) used[(size_t)k * nr + s.z + r] = 0;
    }
    // cleared for the kernels that count into it
    if (isp == 0)
        for (int i = threadIdx.x; i < nsmall; i += blockDim.x) small[i] = 0u;
    const int npp = A_.nprim * npb;
    const bool same = s.x == s.y;
    const int ncA = ncart_d(lA), ncB = ncart_d(lB);
    const int ncp = same ? ncA * (ncA + 1) / 2 : ncA * ncB;
    const int cp0 = sp_cp[isp];
    __syncthreads();
    // terms and their bounds
    for (int t = threadIdx.x; t < ncp * npp; t += blockDim.x) {
        const int c = t / npp, pp = t - c * npp;
        int c1, c2;
        cp_decode(c, same, ncB, c1, c2);
        const int* pA = kCartD[lA][c1];
        const int* pB = kCartD[lB][c2];
        int rr[3];
        double bd = 1.0;
        for (int ax = 0; ax < 3; ++ax) {
            rr[ax] = s.z + pp * 3 * ncls + ax * ncls + pA[ax] * (lB + 1) + pB[ax];
            bd *= rowsum[rr[ax]];
        }
        trow[s.w + t] = make_int4(rr[0], rr[1], rr[2], cp0 + c);
        tbound[s.w + t] = bd;
    }
    __syncthreads();
    // component pairs: the sum of their term bounds; packed weights, component
    // pairs fastest (neighbours of one state share T's cache lines)
    for (int c = threadIdx.x; c < ncp; c += blockDim.x) {
        double b = 0.0;
        for (int pp = 0; pp < npp; ++pp) b += tbound[s.w + c * npp + pp];
        bsum[cp0 + c] = b;
    }
    for (int i = threadIdx.x; i < ncp * ns; i += blockDim.x) {
        const int st = i / ncp, c = i - st * ncp;
        int c1, c2;
        cp_decode(c, same, ncB, c1, c2);
        const int mu = bf0[s.x] + c1, nu = bf0[s.y] + c2;
        const double* Ts = T + (size_t)st * nbf * nbf;
        const double v = mu == nu ? Ts[(size_t)mu * nbf + mu] : Ts[(size_t)mu * nbf + nu] + Ts[(size_t)nu * nbf + mu];
        tp64[(size_t)(cp0 + c) * ns + st] = v * (cnorm[mu] * cnorm[nu] * spin);
    }
    __syncthreads();
    // per shell pair partial of sum_t |Tp(s)| bound(t), fixed order
    for (int st = threadIdx.x; st < ns; st += blockDim.x) {
        double acc = 0.0;
        for (int c = 0; c < ncp; ++c) acc += fabs(tp64[(size_t)(cp0 + c) * ns + st]) * bsum[cp0 + c];
        part[(size_t)isp * ns + st] = acc;
    }
}

__global__ __launch_bounds__(1024) void tot_kernel(const double* __restrict__ part, int nsp, int ns, double* __restrict__ tot) {
    // one block of 1024 threads per state: fixed-order strided partial sums,
    // then a fixed-shape tree (deterministic)
    __shared__ double red[1024];
    for (int st = blockIdx.x; st < ns; st += gridDim.x) {
        double a = 0.0;
        for (int i = threadIdx.x; i < nsp; i += blockDim.x) a += part[(size_t)i * ns + st];
        red[threadIdx.x] = a;
        __syncthreads();
        for (int w = blockDim.x / 2; w > 0; w >>= 1) {
            if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
            __syncthreads();
        }
        if (threadIdx.x == 0) tot[st] = red[0];
        __syncthreads();
    }
}

// per component pair: m_k = max_s |Tp(s,k)| / tot_s
__global__ void pairmax_kernel(const double* __restrict__ tp64, const double* __restrict__ tot, int ns, int ncp,
                               double* __restrict__ mk) {
    for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < ncp; k += gridDim.x * blockDim.x) {
        double m = 0.0;
        for (int st = 0; st < ns; ++st)
            if (tot[st] > 0.0) m = fmax(m, fabs(tp64[(size_t)k * ns + st]) / tot[st]);
        mk[k] = m;
    }
}

__global__ void weight_kernel(const int4* __restrict__ trow, const double* __restrict__ tbound,
                              const double* __restrict__ mk, long long nterms, double* __restrict__ w,
                              unsigned int* __restrict__ hist) {
    // the workgroup counts its terms' exponents in LDS (most terms share a
    // few bins, so global atomics per term would serialise) and adds its
    // non-empty bins to the global histogram once
    __shared__ unsigned int lh[kHistBins];
    for (int b = threadIdx.x; b < kHistBins; b += blockDim.x) lh[b] = 0u;
    __syncthreads();
    for (long long t = blockIdx.x * (long long)blockDim.x + threadIdx.x; t < nterms;
         t += (long long)gridDim.x * blockDim.x) {
        const double x = mk[trow[t].w] * tbound[t];
        w[t] = x;
        if (x > 0.0) {
            int e;
            frexp(x, &e);    // x in [2^(e-1), 2^e)
            e = min(max(e + kHistBias, 0), kHistBins - 1);
            atomicAdd(&lh[e], 1u);
        }
    }
    __syncthreads();
    for (int b = threadIdx.x; b < kHistBins; b += blockDim.x)
        if (lh[b]) atomicAdd(&hist[b], lh[b]);
}

__global__ void thresh_kernel(const unsigned int* __restrict__ hist, double eps, double* __restrict__ thr) {
    // one wave: per-bin upper bounds in LDS, then the largest bin `best` such
    // that the bounds of all bins <= best sum to at most eps.  The bins are
    // scanned as 64 runs of consecutive bins (one run per lane): each lane sums
    // its run, a scan over the lanes finds the run in which the total would pass
    // eps, and lane 0 walks that run bin by bin (a fixed order, so the result is
    // deterministic)
    constexpr int kRun = (kHistBins + 63) / 64;
    __shared__ double pre[kHistBins];
    __shared__ double run[64];
    const int lane = threadIdx.x;
    for (int b = lane; b < kHistBins; b += blockDim.x) pre[b] = (double)hist[b] * ldexp(1.0, b - kHistBias);
    __syncthreads();
    if (lane < 64) {
        double sr = 0.0;
        for (int b = lane * kRun; b < min((lane + 1) * kRun, kHistBins); ++b) sr += pre[b];
        run[lane] = sr;
    }
    __syncthreads();
    // sums of the runs up to and including each (a fixed-shape scan); the runs
    // that fit whole are the first r
    double incl = run[lane];
    for (int h = 1; h < 64; h <<= 1) {
        const double o = __shfl_up(incl, h);
        if (lane >= h) incl += o;
    }
    const int r = __popcll(__ballot(incl <= eps));   // non-decreasing: a prefix of the lanes
    double sum = __shfl(incl, max(r - 1, 0));
    if (lane == 0) {
        if (!(eps > 0.0)) {
            thr[0] = -1.0;   // no screening: keep every term, zero or not
            return;
        }
        if (r == 0) sum = 0.0;
        int best = r * kRun - 1;   // every bin of the runs before r is dropped
        if (r < 64) {
            for (int b = r * kRun; b < min((r + 1) * kRun, kHistBins); ++b) {
                if (sum + pre[b] > eps) break;
                sum += pre[b];
                best = b;
            }
        }
        best = min(best, kHistBins - 1);
        // w < 2^(best - bias) exactly when its frexp exponent bin is <= best
        thr[0] = best < 0 ? 0.0 : ldexp(1.0, best - kHistBias);
    }
}

__device__ __forceinline__ bool term_kept(double w, double thr) {
    return thr < 0.0 || (w > 0.0 && w >= thr);
}

// Virtual pairs of a component pair with n kept terms: ceil(n / 9), of lengths
// (n - pos) / (left) as vkeys_kernel cuts them.  stats: pairs with a term,
// terms; hist: virtual pairs per length.
__global__ __launch_bounds__(256) void stats_kernel(const int* __restrict__ cp_first, const int* __restrict__ cp_nterms,
                                                    const double* __restrict__ w, const double* __restrict__ thr,
                                                    int ncp, unsigned long long* __restrict__ stats,
                                                    int* __restrict__ hist) {
    __shared__ int lh[16], lp;
    __shared__ unsigned long long lt;
    if (threadIdx.x < 16) lh[threadIdx.x] = 0;
    if (threadIdx.x == 0) {
        lp = 0;
        lt = 0ull;
    }
    __syncthreads();
    const double th = thr[0];
    for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < ncp; k += gridDim.x * blockDim.x) {
        int n = 0;
        for (int t = 0; t < cp_nterms[k]; ++t) n += term_kept(w[cp_first[k] + t], th) ? 1 : 0;
        if (n == 0) continue;
        atomicAdd(&lp, 1);
        atomicAdd(&lt, (unsigned long long)n);
        const int m = (n + kMaxTermsPerPair - 1) / kMaxTermsPerPair;
        int pos = 0;
        for (int v = 0; v < m; ++v) {
            const int take = (n - pos) / (m - v);
            atomicAdd(&lh[take], 1);
            pos += take;
        }
    }
    __syncthreads();
    if (threadIdx.x < 16 && lh[threadIdx.x]) atomicAdd(&hist[threadIdx.x], lh[threadIdx.x]);
    if (threadIdx.x == 0 && lp) {
        atomicAdd(&stats[0], (unsigned long long)lp);
        atomicAdd(&stats[1], lt);
    }
}

__global__ void count_kernel(const int* __restrict__ cp_first, const int* __restrict__ cp_nterms,
                             const double* __restrict__ w, const double* __restrict__ thr, int ncp,
                             int* __restrict__ nk, int* __restrict__ nv) {
    for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < ncp; k += gridDim.x * blockDim.x) {
        const double th = thr[0];
        int n = 0;
        for (int t = 0; t < cp_nterms[k]; ++t) n += term_kept(w[cp_first[k] + t], th) ? 1 : 0;
        nk[k] = n;
        nv[k] = (n + kMaxTermsPerPair - 1) / kMaxTermsPerPair;
    }
}

__global__ void vkeys_kernel(const int* __restrict__ nk, const int* __restrict__ nv,
                             const int* __restrict__ vbase, int ncp, unsigned int* __restrict__ key,
                             int* __restrict__ val, int4* __restrict__ vinfo) {
    for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < ncp; k += gridDim.x * blockDim.x) {
        const int n = nk[k], m = nv[k];
        int pos = 0;
        for (int v = 0; v < m; ++v) {
            const int take = (n - pos) / (m - v);
            const int id = vbase[k] + v;
            key[id] = (unsigned)(kMaxTermsPerPair - take);   // longest first
            val[id] = id;
            vinfo[id] = make_int4(k, pos, take, 0);
            pos += take;
        }
    }
}

__global__ void unit_kernel(const int* __restrict__ order, const int4* __restrict__ vinfo, int nv,
                            int n_chunks, int* __restrict__ cnpp, int* __restrict__ csize) {
    for (int c = blockIdx.x * blockDim.x + threadIdx.x; c < n_chunks; c += gridDim.x * blockDim.x) {
        const int o = c * kChunk;
        const int npp = o < nv ? max(1, vinfo[order[o]].z) : 1;
        cnpp[c] = npp;
        csize[c] = kChunk * npp;
    }
}

__global__ void layout_kernel(const int* __restrict__ order, const int4* __restrict__ vinfo, int nv,
                              int n_vpairs, const int* __restrict__ cnpp, const int* __restrict__ coff,
                              const int* __restrict__ cp_first, const int* __restrict__ cp_nterms,
                              const int4* __restrict__ trow, const double* __restrict__ w,
                              const double* __restrict__ thr, const double* __restrict__ tp64, int ns,
                              int SW, const int* __restrict__ newid, int nr, int4* __restrict__ slots,
                              float* __restrict__ tp32) {
    for (int o = blockIdx.x * blockDim.x + threadIdx.x; o < n_vpairs; o += gridDim.x * blockDim.x) {
        const int c = o / kChunk, j = o - c * kChunk;
        const int npp = cnpp[c];
        int4* dst = slots + coff[c] + j * npp;
        int len = 0, k = -1;
        if (o < nv) {
            const int4 vi = vinfo[order[o]];
            k = vi.x;
            len = vi.z;
            const double th = thr[0];
            int seen = 0, q = 0;
            for (int t = 0; t < cp_nterms[k] && q < len; ++t) {
                const int ti = cp_first[k] + t;
                if (!term_kept(w[ti], th)) continue;
                if (seen++ < vi.y) continue;
                const int4 tr = trow[ti];
                dst[q++] = make_int4(1 + newid[tr.x], 1 + newid[(size_t)nr + tr.y], 1 + newid[(size_t)2 * nr + tr.z], 1);
            }
        }
        for (int q = len; q < npp; ++q) dst[q] = make_int4(0, 0, 0, 0);   // the zero row
        for (int st = 0; st < SW; ++st) {
            tp32[(size_t)o * SW + st] = (k >= 0 && st < ns) ? (float)tp64[(size_t)k * ns + st] : 0.0f;
        }
    }
}

// Component pairs of a shell pair by the powers (i, j) of an axis, in
// component order: for every axis and (lA, lB, same shell), class i (lB + 1) + j ->
// count and component pairs.
struct ZClasses {
    unsigned char n[54][9], c[54][9][kZTerms];
};
constexpr ZClasses make_zclasses() {
    constexpr int cart[3][3][6] = {{{0}, {1, 0, 0}, {2, 1, 1, 0, 0, 0}},
                                   {{0}, {0, 1, 0}, {0, 1, 0, 2, 1, 0}},
                                   {{0}, {0, 0, 1}, {0, 0, 1, 0, 1, 2}}};
    ZClasses t{};
    for (int ak = 0; ak < 54; ++ak) {
        const int(&cz)[3][6] = cart[ak / 18];
        const int k = ak % 18;
        const int lA = k / 6, lB = k / 2 % 3, same = k & 1;
        const int ncA = (lA + 1) * (lA + 2) / 2, ncB = (lB + 1) * (lB + 2) / 2;
        if (same && lA != lB) continue;
        int c = 0;
        for (int c1 = 0; c1 < ncA; ++c1)
            for (int c2 = same ? c1 : 0; c2 < ncB; ++c2, ++c) {
                const int cls = cz[lA][c1] * (lB + 1) + cz[lB][c2];
                t.c[ak][cls][t.n[ak][cls]++] = (unsigned char)c;
            }
    }
    return t;
}
__device__ __constant__ ZClasses kZClasses = make_zclasses();

// Scale of a z row: V 2^e with |V| <= bound < 2^(14 - e).
__device__ __forceinline__ int z_exponent(double bound) {
    return bound > 0.0 && bound < 1e300 ? max(-900, min(900, 13 - ilogb(bound))) : 0;
}

__device__ __forceinline__ int term_row(const int4& t, int axis) { return axis == 0 ? t.x : axis == 1 ? t.y : t.z; }

// Per z row (id = row offset / 3 + pp ncls + class): kept terms n, one-hot flags
// of 9 - n behind the row flags (used + 3 nr, 9 segments of all z rows, so that
// the one scan that numbers the rows also sorts the z rows, most terms first),
// and (shell pair, pp ncls + class).  mx: per state the largest sum of |Tp| x bound
// x y bound over a row's terms, divided by the row's scale, as the bits of a
// non-negative double (which order like the values); a maximum does not depend
// on the order of the atomics.  tail: per state and exponent of p the largest
// |Tp| x bound of an s-s term.
__global__ __launch_bounds__(128) void zcount_kernel(const PrepShell* __restrict__ sh, const int4* __restrict__ sp,
                                                    const int4* __restrict__ trow, const double* __restrict__ rowsum,
                                                    const double* __restrict__ w, const double* __restrict__ thr,
                                                    const double* __restrict__ tp64, int ns, int nr,
                                                    int nz_all, int axis, int* __restrict__ used, int* __restrict__ zn,
                                                    int2* __restrict__ zinfo, unsigned long long* __restrict__ gmx,
                                                    unsigned long long* __restrict__ gtail,
                                                    const VRowDev* __restrict__ rows) {
    __shared__ unsigned long long mx[kMaxStates], tail[kMaxStates * kTailBins];
    const int isp = blockIdx.x;
    const int4 s = sp[isp];
    const int lA = sh[s.x].l, lB = sh[s.y].l, npp = sh[s.x].nprim * sh[s.y].nprim;
    const bool same = s.x == s.y;
    const int ncls = (lA + 1) * (lB + 1);
    const double th = thr[0];
    const bool ss = lA + lB == 0;
    if (threadIdx.x < kMaxStates) mx[threadIdx.x] = 0ull;
    if (ss)
        for (int i = threadIdx.x; i < ns * kTailBins; i += blockDim.x) tail[i] = 0ull;
    __syncthreads();
    const int kc = 18 * axis + lA * 6 + lB * 2 + (same ? 1 : 0), nz = npp * ncls;
    const int la = axis == 0 ? 1 : 0, lb = axis == 2 ? 1 : 2;   // the line axes
    for (int z = threadIdx.x; z < nz; z += blockDim.x) {
        const int pp = z / ncls, cls = z - pp * ncls;
        int n = 0;
        for (int k = 0; k < kZClasses.n[kc][cls]; ++k) {
            const int t = s.w + kZClasses.c[kc][cls][k] * npp + pp;
            if (!term_kept(w[t], th)) continue;
            const int4 tr = trow[t];
            used[(size_t)la * nr + term_row(tr, la)] = 1;
            used[(size_t)lb * nr + term_row(tr, lb)] = 1;
            ++n;
        }
        const int id = s.z / 3 + z;
        zn[id] = n;
        zinfo[id] = make_int2(isp, z);
        for (int k = 0; k < kZTerms; ++k) used[(size_t)3 * nr + (size_t)k * nz_all + id] = n == kZTerms - k;
        if (n) used[(size_t)axis * nr + s.z + pp * 3 * ncls + axis * ncls + cls] = 1;
    }
    for (int i = threadIdx.x; i < nz * ns; i += blockDim.x) {
        const int z = i / ns, st = i - z * ns;
        const int pp = z / ncls, cls = z - pp * ncls;
        double b = 0.0;
        for (int k = 0; k < kZClasses.n[kc][cls]; ++k) {
            const int t = s.w + kZClasses.c[kc][cls][k] * npp + pp;
            if (!term_kept(w[t], th)) continue;
            const int4 tr = trow[t];
            b += fabs(tp64[(size_t)tr.w * ns + st]) * rowsum[term_row(tr, la)] * rowsum[term_row(tr, lb)];
        }
        const int rz = s.z + pp * 3 * ncls + axis * ncls + cls;
        if (ss) {   // one term, of magnitude b times its Gaussian
            const double t = b * rowsum[rz];
            const int e = ilogb(0.25 / rows[rz].inv4p) - kTailMin;
            if (t > 0.0 && t < 1e300)
                atomicMax(&tail[st * kTailBins + max(0, min(e, kTailBins - 1))], (unsigned long long)__double_as_longlong(t));
        }
        b *= ldexp(1.0, -z_exponent(rowsum[rz]));
        // non-negative doubles order like their bit patterns; NaN and infinity are left out
        if (b > 0.0 && b < 1e300) atomicMax(&mx[st], (unsigned long long)__double_as_longlong(b));
    }
    __syncthreads();
    for (int st = threadIdx.x; st < ns; st += blockDim.x)
        if (mx[st] > __hip_atomic_load(&gmx[st], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(&gmx[st], mx[st]);
    if (ss)
        for (int i = threadIdx.x; i < ns * kTailBins; i += blockDim.x)
            if (tail[i] && tail[i] > __hip_atomic_load(&gtail[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
                atomicMax(&gtail[i], tail[i]);
}

// Per state: its largest z-row bound, as the exponent ks with bound 2^ks <
// 2^15 (weights are scaled by 2^ks) and the factor 2^-ks of the results.  Then
// what the host needs: the first numbers of the y rows, the z rows and the nine
// segments of sorted z rows, and their end (meta[12], all numbers of one scan).
__global__ __launch_bounds__(64) void zmeta_kernel(const unsigned long long* __restrict__ mx, int ns,
                                                   const int* __restrict__ newid, const int* __restrict__ used, int nr,
                                                   int nz_all, int* __restrict__ ks, double* __restrict__ sinv,
                                                   int* __restrict__ meta) {
    const int i = threadIdx.x;
    if (i < ns) {
        const double b = __longlong_as_double((long long)mx[i]);
        const int k = b > 0.0 ? max(-900, min(900, 14 - ilogb(b))) : 0;
        ks[i] = k;
        sinv[i] = ldexp(1.0, -k);
    }
    const size_t end = (size_t)3 * nr + (size_t)kZTerms * nz_all;
    if (i < 2) meta[i] = newid[(size_t)(i + 1) * nr];
    else if (i < 2 + kZTerms) meta[i] = newid[(size_t)3 * nr + (size_t)(i - 2) * nz_all];
    else if (i == 2 + kZTerms) meta[i] = newid[end - 1] + used[end - 1];
}

// Rows compacted (blocks from nbz on), and one thread per (z row, state): its
// term records, weights T 2^(ks - e) and (thread of state 0) its z slot (row, e) at
// its sorted place p; then the places past the last row.
__global__ __launch_bounds__(256) void zlayout_kernel(const PrepShell* __restrict__ sh, const int4* __restrict__ sp,
                                                      const int4* __restrict__ trow, const double* __restrict__ rowsum,
                                                      const double* __restrict__ w, const double* __restrict__ thr,
                                                      const double* __restrict__ tp64, int ns, int nr,
                                                      const int* __restrict__ newid, const int* __restrict__ znum,
                                                      const int2* __restrict__ zinfo, int nz, int nzpad, int nz_all,
                                                      int axis, KSteps steps, const int* __restrict__ ks,
                                                      int2* __restrict__ zslots, int2* __restrict__ terms,
                                                      float* __restrict__ Tw, int nbz, const VRowDev* __restrict__ rows,
                                                      const int* __restrict__ used, VRowDev* __restrict__ out) {
    if ((int)blockIdx.x >= nbz) {
        const long long all = 3LL * nr;
        for (long long r = (blockIdx.x - nbz) * (long long)blockDim.x + threadIdx.x; r < all;
             r += (long long)(gridDim.x - nbz) * blockDim.x) {
            if (r == 0) {
                VRowDev z{};
                z.inv4p = 1.0;
                out[0] = z;
            }
            if (used[r]) out[1 + newid[r]] = rows[r % nr];
        }
        return;
    }
    const int la = axis == 0 ? 1 : 0, lb = axis == 2 ? 1 : 2;   // the line axes
    const long long tot = (long long)(nz_all + nzpad - nz) * ns;
    for (long long gi = blockIdx.x * (long long)blockDim.x + threadIdx.x; gi < tot; gi += (long long)nbz * blockDim.x) {
        const int id = (int)(gi / ns), st = (int)(gi - (long long)id * ns);
        int p = nz + id - nz_all;
        if (id < nz_all) {
            const int m = znum[id];
            if (m == 0) continue;
            const size_t seg = (size_t)3 * nr;
            p = newid[seg + (size_t)(kZTerms - m) * nz_all + id] - newid[seg];
        }
        const int zn = ksteps_terms(steps, p / kZStep), zc = ksteps_first(steps, p / kZStep);
        // record t of the row at rec[32 t], weight t at tw[grid_term_weights t]
        const int zl = p % kZStep;
        int2* rec = terms + zc * kZStep + zl;
        float* tw = Tw + (size_t)zc * grid_term_weights(ns) + ((zl >> 3) * ns + st) * 12 + (zl & 7);
        const int tstep = grid_term_weights(ns);
        int n = 0;
        if (id < nz_all) {
            const int2 zi = zinfo[id];
            const int4 s = sp[zi.x];
            const int lA = sh[s.x].l, lB = sh[s.y].l, npp = sh[s.x].nprim * sh[s.y].nprim;
            const int ncls = (lA + 1) * (lB + 1), pp = zi.y / ncls, cls = zi.y - pp * ncls;
            const int rz = s.z + pp * 3 * ncls + axis * ncls + cls;
            const int e = z_exponent(rowsum[rz]);
            const double th = thr[0], sc = ldexp(1.0, ks[st] - e);
            const int kc = 18 * axis + lA * 6 + lB * 2 + (s.x == s.y ? 1 : 0);
            for (int k = 0; k < kZClasses.n[kc][cls]; ++k) {
                const int t = s.w + kZClasses.c[kc][cls][k] * npp + pp;
                if (!term_kept(w[t], th)) continue;
                const int4 tr = trow[t];
                // rows of the line axes' tables, whose row 0 is the zero row
                if (st == 0)
                    rec[kZStep * n] = make_int2(1 + newid[(size_t)la * nr + term_row(tr, la)] - newid[(size_t)la * nr],
                                                1 + newid[(size_t)lb * nr + term_row(tr, lb)] - newid[(size_t)lb * nr]);
                const double tp = tp64[(size_t)tr.w * ns + st];
                float v = (float)(tp * sc);
                // finite weights stay finite (a row bound that underflows)
                if (isinf(v) && !isinf(tp)) v = copysignf(3e38f, v);
                tw[n * tstep] = v;
                ++n;
            }
            if (st == 0) zslots[p] = make_int2(1 + newid[(size_t)axis * nr + rz], e);
        } else if (st == 0) {
            zslots[p] = make_int2(0, 0);
        }
        for (; n < zn; ++n) {   // padding: the zero row, weight zero
            if (st == 0) rec[kZStep * n] = make_int2(0, 0);
            tw[n * tstep] = 0.f;
        }
    }
}

__global__ __launch_bounds__(256) void clear_kernel(unsigned* __restrict__ p, int n) {
    for (int i = threadIdx.x; i < n; i += 256) p[i] = 0u;
}

// ------------------------------------------------------------------ host driver

namespace {

int blocks_for(long long n, int bs) {
    long long b = (n + bs - 1) / bs;
    if (b < 1) b = 1;
    if (b > 65536) b = 65536;
    return (int)b;
}

}  // namespace

#define CK(x)                                  \
    do {                                       \
        if ((e = (x)) != hipSuccess) return e; \
    } while (0)

// Runs the precompute and the grid kernel's layout on `st`.  Buffers in `w` are (re)allocated through
// `alloc`, which enforces the caller's memory budget.  Returns hipSuccess or
// the first HIP error; sizes and statistics are written to `res`.
hipError_t run_prep(const PrepInputs& in, PrepWork& w, PrepResult& res, int axis, hipStream_t st,
                    const std::function<hipError_t(DeviceBuffer&, size_t)>& alloc) {
    hipError_t e;
    const long long NR = in.n_rows_all, NT = in.n_terms_all;
    const int NCP = in.n_cp, NSP = in.n_sp, ns = in.n_states;
    const int NZ = (int)(NR / 3);   // rows per axis
    CK(alloc(w.rows_all, (size_t)NR * sizeof(VRowDev)));
    CK(alloc(w.rowsum, (size_t)NR * sizeof(double)));
    CK(alloc(w.trow, (size_t)NT * sizeof(int4)));
    CK(alloc(w.tbound, std::max((size_t)NT * sizeof(double), (size_t)NZ * 12)));
    CK(alloc(w.wt, (size_t)NT * sizeof(double)));
    CK(alloc(w.tp64, (size_t)NCP * ns * sizeof(double)));
    CK(alloc(w.bsum, (size_t)NCP * sizeof(double)));
    CK(alloc(w.part, (size_t)NSP * ns * sizeof(double)));
    static_assert(kSmallHist + kHistBins * sizeof(unsigned) <= kSmallMeta, "histogram overlaps what the host reads");
    CK(alloc(w.small, kSmallBytes));
    // flags: rows used per axis, then the z rows' one-hot term counts
    const long long NF = 3 * NR + (long long)kZTerms * NZ;
    CK(alloc(w.row_used, (size_t)NF * sizeof(int)));
    CK(alloc(w.newid, (size_t)NF * sizeof(int)));
    double* tot = (double*)w.small.p;                                    // [<= 32]
    double* thr = tot + 64;                                              // [1]
    unsigned* hist = (unsigned*)((char*)w.small.p + kSmallHist);         // [kHistBins]

    const int nsmall = (int)(kSmallBytes / sizeof(unsigned));
    hipLaunchKernelGGL(rows_terms_kernel, dim3(NSP), dim3(128), 0, st, in.shells, in.sp, in.xyz, in.exps, in.coefs, in.n1d,
                       (int)NR, in.sp_cp, in.bf0, in.cnorm, in.T, in.nbf, ns, in.spin, (VRowDev*)w.rows_all.p,
                       (double*)w.rowsum.p, (int*)w.row_used.p, (unsigned*)w.small.p, nsmall, (int4*)w.trow.p,
                       (double*)w.tbound.p, (double*)w.tp64.p, (double*)w.bsum.p, (double*)w.part.p);
    CK(hipGetLastError());
    hipLaunchKernelGGL(tot_kernel, dim3(ns), dim3(1024), 0, st, (const double*)w.part.p, NSP, ns, tot);
    CK(hipGetLastError());
    hipLaunchKernelGGL(pairmax_kernel, dim3(blocks_for(NCP, 256)), dim3(256), 0, st, (const double*)w.tp64.p,
                       (const double*)tot, ns, NCP, (double*)w.bsum.p);
    CK(hipGetLastError());
    hipLaunchKernelGGL(weight_kernel, dim3(std::min(blocks_for(NT, 256), 512)), dim3(256), 0, st, (const int4*)w.trow.p,
                       (const double*)w.tbound.p, (const double*)w.bsum.p, NT, (double*)w.wt.p, hist);
    CK(hipGetLastError());
    hipLaunchKernelGGL(thresh_kernel, dim3(1), dim3(64), 0, st, (const unsigned*)hist, in.eps, thr);
    CK(hipGetLastError());
    return run_prep_layout(in, w, res, axis, true, st, alloc);
}

// The grid kernel's layout by one axis, after the rest of the precompute (first),
// or again by another axis.
hipError_t run_prep_layout(const PrepInputs& in, PrepWork& w, PrepResult& res, int axis, bool first, hipStream_t st,
                           const std::function<hipError_t(DeviceBuffer&, size_t)>& alloc) {
    hipError_t e;
    const long long NR = in.n_rows_all, NF = 3 * NR + (long long)kZTerms * (NR / 3);
    const int NZ = (int)(NR / 3), NSP = in.n_sp, ns = in.n_states;
    const double* thr = (const double*)w.small.p + 64;
    double* sinv = (double*)((char*)w.small.p + kSmallSinv);             // [<= 32]
    int* ks = (int*)((char*)w.small.p + kSmallKs);                       // [<= 32]
    int* meta = (int*)((char*)w.small.p + kSmallMeta);                   // [12]
    unsigned long long* zmx = (unsigned long long*)((char*)w.small.p + kSmallZmax);   // [<= 32]
    unsigned long long* tail = (unsigned long long*)((char*)w.small.p + kSmallTail);  // [ns][kTailBins]
    if (axis < 0 || axis > 2) return hipErrorInvalidValue;
    if (!first) {
        hipLaunchKernelGGL(clear_kernel, dim3(1), dim3(256), 0, st, (unsigned*)zmx,
                           (int)((kSmallBytes - kSmallZmax) / sizeof(unsigned)));
        CK(hipGetLastError());
    }
    // the term bounds were last read by weight_kernel: their buffer holds the
    // z rows' places and term counts from here on
    int2* zinfo = (int2*)w.tbound.p;
    int* zn = (int*)(zinfo + NZ);
    hipLaunchKernelGGL(zcount_kernel, dim3(NSP), dim3(128), 0, st, in.shells, in.sp, (const int4*)w.trow.p,
                       (const double*)w.rowsum.p, (const double*)w.wt.p, (const double*)thr, (const double*)w.tp64.p, ns,
                       (int)NR, NZ, axis, (int*)w.row_used.p, zn, zinfo, zmx, tail, (const VRowDev*)w.rows_all.p);
    CK(hipGetLastError());
    size_t tmp_bytes = 0;
    CK(hipcub::DeviceScan::ExclusiveSum(nullptr, tmp_bytes, (int*)w.row_used.p, (int*)w.newid.p, (size_t)NF, st));
    CK(alloc(w.tmp4, tmp_bytes + 256));
    CK(hipcub::DeviceScan::ExclusiveSum(w.tmp4.p, tmp_bytes, (int*)w.row_used.p, (int*)w.newid.p, (size_t)NF, st));
    hipLaunchKernelGGL(zmeta_kernel, dim3(1), dim3(64), 0, st, (const unsigned long long*)zmx, ns,
                       (const int*)w.newid.p, (const int*)w.row_used.p, (int)NR, NZ, ks, sinv, meta);
    CK(hipGetLastError());
    // the one readback lands in the context's pinned host memory when it has
    // some (a DMA; pageable destinations are staged by the runtime)
    const size_t rbytes = kSmallTail - kSmallMeta + (size_t)ns * kTailBins * sizeof(double);
    alignas(16) unsigned char local_rb[kSmallBytes - kSmallMeta];
    unsigned char* rbuf = w.pinned ? (unsigned char*)w.pinned : local_rb;
    const int* rb = (const int*)rbuf;
    CK(hipMemcpyAsync(rbuf, meta, rbytes, hipMemcpyDeviceToHost, st));
    CK(hipStreamSynchronize(st));
    const int nrows_used = rb[2];   // the numbers of the z rows' segments start after the rows'
    // k-steps of kZStep sorted z rows; every row is padded to the count of the
    // k-step's first (a single k-step of zero rows if nothing is kept)
    KSteps steps{};
    int nz = 0;
    for (int n = kZTerms; n >= 1; --n) {
        nz += rb[2 + kZTerms - n + 1] - rb[2 + kZTerms - n];
        steps.kend[n] = (nz + kZStep - 1) / kZStep;
    }
    if (nz == 0) steps.kend[1] = 1;
    const int n_ksteps = steps.kend[1], nzpad = n_ksteps * kZStep;
    long long nc = 0;
    for (int n = 1; n <= kZTerms; ++n) nc += steps.kend[n];
    const long long nterm = nc * kZStep, nw = nc * grid_term_weights(ns);
    if (nz > nrows_used || nterm > INT32_MAX) return hipErrorUnknown;
    CK(alloc(w.zslots, (size_t)nzpad * sizeof(int2)));
    CK(alloc(w.zterms, (size_t)nterm * sizeof(int2)));
    CK(alloc(w.zw, (size_t)nw * sizeof(float)));
    CK(alloc(w.rows, (size_t)(nrows_used + 1) * sizeof(VRowDev)));
    const int nbz = blocks_for((long long)(NZ + nzpad - nz) * ns, 256);
    hipLaunchKernelGGL(zlayout_kernel, dim3(nbz + blocks_for(3 * NR, 256)), dim3(256), 0, st, in.shells, in.sp,
                       (const int4*)w.trow.p, (const double*)w.rowsum.p, (const double*)w.wt.p, (const double*)thr,
                       (const double*)w.tp64.p, ns, (int)NR, (const int*)w.newid.p, (const int*)zn, (const int2*)zinfo, nz,
                       nzpad, NZ, axis, steps, (const int*)ks, (int2*)w.zslots.p, (int2*)w.zterms.p, (float*)w.zw.p, nbz,
                       (const VRowDev*)w.rows_all.p, (const int*)w.row_used.p, (VRowDev*)w.rows.p);
    CK(hipGetLastError());
    res.axis = axis;
    res.n_rows = nrows_used + 1;
    res.n_axis[0] = rb[0];
    res.n_axis[1] = rb[1] - rb[0];
    res.n_axis[2] = rb[2] - rb[1];
    std::memcpy(res.zmax, rbuf + kSmallZmax - kSmallMeta, ns * sizeof(double));
    std::memcpy(res.tail, rbuf + kSmallTail - kSmallMeta, ns * sizeof(res.tail[0]));
    res.n_ksteps = n_ksteps;
    res.ksteps = steps;
    res.n_zterms = nterm;
    res.n_zweights = nw;
    res.state_blocks = (ns + kStateBlock - 1) / kStateBlock;
    return hipSuccess;
}

// Pairs and terms kept, and the sizes of the layout by component pairs.
hipError_t run_prep_stats(const PrepInputs& in, PrepWork& w, PrepResult& res, hipStream_t st) {
    hipError_t e;
    const double* thr = (const double*)w.small.p + 64;
    unsigned long long* stats = (unsigned long long*)((char*)w.small.p + kSmallStats);   // [2], then int [16]
    constexpr size_t nb = 2 * sizeof(unsigned long long) + 16 * sizeof(int);
    CK(hipMemsetAsync(stats, 0, nb, st));
    hipLaunchKernelGGL(stats_kernel, dim3(std::min(blocks_for(in.n_cp, 256), 256)), dim3(256), 0, st, in.cp_first,
                       in.cp_nterms, (const double*)w.wt.p, thr, in.n_cp, stats, (int*)(stats + 2));
    CK(hipGetLastError());
    alignas(16) unsigned char local_rb[nb];
    unsigned char* rb = w.pinned ? (unsigned char*)w.pinned : local_rb;
    CK(hipMemcpyAsync(rb, stats, nb, hipMemcpyDeviceToHost, st));
    CK(hipStreamSynchronize(st));
    const unsigned long long* kr = (const unsigned long long*)rb;
    const int* hist = (const int*)(kr + 2);
    res.pairs_kept = (long long)kr[0];
    res.terms_kept = (long long)kr[1];
    // virtual pairs sorted longest first, in units of kChunk padded to their
    // first pair's length; chunks are runs of units of equal length, at most
    // kMaxUnitsPerChunk units and kMaxChunkTerms terms
    int units[16] = {};
    long long nv = 0, slots = 0;
    for (int v = kMaxTermsPerPair; v >= 1; --v) {
        const long long u0 = (nv + kChunk - 1) / kChunk, u1 = (nv + hist[v] + kChunk - 1) / kChunk;
        units[v] = (int)(u1 - u0);
        nv += hist[v];
    }
    res.n_virtual = (int)nv;
    if (nv == 0) units[1] = 1;   // one padded unit
    res.n_units = res.n_chunks = 0;
    for (int v = kMaxTermsPerPair; v >= 1; --v) {
        const int um = std::min(kMaxUnitsPerChunk, kMaxChunkTerms / (kChunk * v));
        res.n_units += units[v];
        res.n_chunks += (units[v] + um - 1) / um;
        slots += (long long)units[v] * kChunk * v;
    }
    res.n_slots = slots;
    res.n_vpairs = res.n_units * kChunk;
    return hipSuccess;
}

// The layout by component pairs (units of packed weights and term slots) of
// the paths other than the grid kernel, after run_prep and run_prep_stats on
// the same inputs.
hipError_t run_prep_pairs(const PrepInputs& in, PrepWork& w, const PrepResult& res, hipStream_t st,
                          const std::function<hipError_t(DeviceBuffer&, size_t)>& alloc) {
    hipError_t e;
    const int NCP = in.n_cp, ns = in.n_states;
    const long long NR = in.n_rows_all;
    const int SW = kStateBlock * ((ns + kStateBlock - 1) / kStateBlock);
    const double* thr = (const double*)w.small.p + 64;
    const int NV = res.n_virtual, NVA = NV > 0 ? NV : 1;
    const int n_vpairs = res.n_vpairs, n_units = res.n_units;
    CK(alloc(w.nk, (size_t)NCP * sizeof(int)));
    CK(alloc(w.nv, (size_t)NCP * sizeof(int)));
    CK(alloc(w.vbase, (size_t)NCP * sizeof(int)));
    CK(alloc(w.key, (size_t)NVA * sizeof(unsigned) * 2));
    CK(alloc(w.val, (size_t)NVA * sizeof(int) * 2));
    CK(alloc(w.vinfo, (size_t)NVA * sizeof(int4)));
    CK(alloc(w.cnpp, (size_t)n_units * sizeof(int)));
    CK(alloc(w.csize, (size_t)n_units * sizeof(int)));
    CK(alloc(w.coff, (size_t)n_units * sizeof(int)));
    CK(alloc(w.slots, (size_t)res.n_slots * sizeof(int4)));
    CK(alloc(w.tp32, (size_t)n_vpairs * SW * sizeof(float)));
    hipLaunchKernelGGL(count_kernel, dim3(blocks_for(NCP, 256)), dim3(256), 0, st, in.cp_first,
                       in.cp_nterms, (const double*)w.wt.p, (const double*)thr, NCP, (int*)w.nk.p, (int*)w.nv.p);
    CK(hipGetLastError());
    // exclusive scan of virtual pairs per component pair
    size_t tmp_bytes = 0;
    CK(hipcub::DeviceScan::ExclusiveSum(nullptr, tmp_bytes, (int*)w.nv.p, (int*)w.vbase.p, NCP, st));
    CK(alloc(w.tmp, tmp_bytes + 256));
    CK(hipcub::DeviceScan::ExclusiveSum(w.tmp.p, tmp_bytes, (int*)w.nv.p, (int*)w.vbase.p, NCP, st));
    unsigned* key_in = (unsigned*)w.key.p;
    unsigned* key_out = key_in + NVA;
    int* val_in = (int*)w.val.p;
    int* val_out = val_in + NVA;
    if (NV > 0) {
        hipLaunchKernelGGL(vkeys_kernel, dim3(blocks_for(NCP, 256)), dim3(256), 0, st, (const int*)w.nk.p,
                           (const int*)w.nv.p, (const int*)w.vbase.p, NCP, key_in, val_in, (int4*)w.vinfo.p);
        CK(hipGetLastError());
        size_t sort_bytes = 0;
        CK(hipcub::DeviceRadixSort::SortPairs(nullptr, sort_bytes, key_in, key_out, val_in, val_out, NV, 0, 4, st));
        CK(alloc(w.tmp2, sort_bytes + 256));
        CK(hipcub::DeviceRadixSort::SortPairs(w.tmp2.p, sort_bytes, key_in, key_out, val_in, val_out, NV, 0, 4, st));
    }
    // units of kChunk sorted virtual pairs, each padded to its first pair's term count
    hipLaunchKernelGGL(unit_kernel, dim3(blocks_for(n_units, 256)), dim3(256), 0, st, (const int*)val_out,
                       (const int4*)w.vinfo.p, NV, n_units, (int*)w.cnpp.p, (int*)w.csize.p);
    CK(hipGetLastError());
    size_t tmp3 = 0;
    CK(hipcub::DeviceScan::ExclusiveSum(nullptr, tmp3, (int*)w.csize.p, (int*)w.coff.p, n_units, st));
    CK(alloc(w.tmp3, tmp3 + 256));
    CK(hipcub::DeviceScan::ExclusiveSum(w.tmp3.p, tmp3, (int*)w.csize.p, (int*)w.coff.p, n_units, st));
    hipLaunchKernelGGL(layout_kernel, dim3(blocks_for(n_vpairs, 128)), dim3(128), 0, st, (const int*)val_out,
                       (const int4*)w.vinfo.p, NV, n_vpairs, (const int*)w.cnpp.p, (const int*)w.coff.p,
                       in.cp_first, in.cp_nterms, (const int4*)w.trow.p, (const double*)w.wt.p,
                       (const double*)thr, (const double*)w.tp64.p, ns, SW, (const int*)w.newid.p, (int)NR,
                       (int4*)w.slots.p, (float*)w.tp32.p);
    CK(hipGetLastError());
    return hipSuccess;
}

#undef CK

}  // namespace scff
