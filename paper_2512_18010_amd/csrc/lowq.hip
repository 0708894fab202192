// FP64 device kernels on the precompute's 1D V-tensor rows, with cost linear
// in the grid axes instead of their product (paper Sec. 5.3, separable
// integrals from the 1D V-tensors; Sec. 6, the low-momentum limit):
//
//  * separable integral  I_s = sum_{ix,iy,iz} wx[ix] wy[iy] wz[iz] f_s(q)
//      = sum_t Tp_s(t) (sum_ix wx V^x_t) (sum_iy wy V^y_t) (sum_iz wz V^z_t):
//    one weighted row sum per 1D row, then one complex triple product per
//    kept term, then the transition-weighted sum over component pairs;
//  * transition dipole  mu_s = grad_q Im f_s at q = 0: each row's value and
//    first derivative at q = 0 are V(0) = e_0 and V'(0) = i (P e_0 + e_1), so
//    d f_s / d q_x (0) = i sum_t Tp_s(t) (P e_0 + e_1)^x e_0^y e_0^z.
//
// All sums run in FP64 with the FP64 weights tp64[component pair][s], straight
// from the precompute's rows and terms; the reductions use a fixed order
// (deterministic).  The layout by packed pairs that these sums read before cost a
// context's first call 200 us and is not needed any more; the pair sums and
// their reduction are one kernel (dipole 41 us, separable 24 us, for 30 heavy
// atoms and 24 states; 10 + 29 us each before, from that layout).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "engine.h"
#include "vrow.h"

namespace scff {

namespace {

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
    return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

// S[r] = sum_i w_a[i] V_r(q_a[i]) for the axis a of row r (w: x, y, z weights
// concatenated).  Eight lanes per row: lane l takes the values i = l, l + 8, ...,
// then a fixed butterfly sums the eight.  On an axis symmetric about 0 (bit a of
// sym) V(-q) = V(q)* gives the value n - 1 - i with i.  Bound by FP64 issue, an
// exponential, a sine and a cosine per value: 30 heavy atoms and 96 values per axis
// 69 us on symmetric axes, 116 on others.  (Moving the
// phase from one value of a lane to the next by a complex product took 80 us, but
// carries the rounding of the first value's phase to all that follow, up to four
// times the error where q is small.  Four rows per eight lanes, sharing the factors where they
// belong to one primitive pair: 122 us, since some row of a wave always starts a new
// one.)
__global__ __launch_bounds__(256) void sep_rows_kernel(const VRowDev* __restrict__ rows, int nrows,
                                                       const double2* __restrict__ w, int3 n, int sym, double3 qmin,
                                                       double3 dq, double2* __restrict__ S) {
    const int l8 = threadIdx.x & 7;
    const int r = blockIdx.x * 32 + (threadIdx.x >> 3);
    const bool ok = r < nrows;
    const VRowDev row = rows[ok ? r : 0];
    const int a = row.axis;
    const int na = ok ? (a == 0 ? n.x : (a == 1 ? n.y : n.z)) : 0;
    const int off = a == 0 ? 0 : (a == 1 ? n.x : n.x + n.y);
    const double q0 = a == 0 ? qmin.x : (a == 1 ? qmin.y : qmin.z);
    const double d = a == 0 ? dq.x : (a == 1 ? dq.y : dq.z);
    const bool half = sym >> a & 1;
    double sr = 0.0, si = 0.0;
    for (int i = l8; i < (half ? (na + 1) / 2 : na); i += 8) {
        const double2 v = eval_row_fp64(row, q0 + d * (double)i);
        double2 wi = w[off + i];
        sr += wi.x * v.x - wi.y * v.y;
        si += wi.x * v.y + wi.y * v.x;
        if (half && na - 1 - i > i) {
            wi = w[off + na - 1 - i];
            sr += wi.x * v.x + wi.y * v.y;
            si += wi.y * v.x - wi.x * v.y;
        }
    }
    for (int o = 1; o < 8; o <<= 1) {
        sr += __shfl_xor(sr, o);
        si += __shfl_xor(si, o);
    }
    if (ok && l8 == 0) S[r] = make_double2(sr, si);
}

// Per chunk of 64 component pairs: G = sum over the kept terms (DIP: four real
// sums, the value at q = 0 and the derivatives / i along x, y, z; else Sx Sy Sz,
// complex), four lanes per pair (the loads of a term depend on one another),
// into LDS, then for every (state, component) the sum of tp64 G over the
// chunk, eight slices of 8 added in order.  part[(state ncomp + comp) nparts +
// block], a block's chunks added in order.
template <bool DIP>
__global__ __launch_bounds__(256) void sep_pairs_kernel(LowqPrep p, const double2* __restrict__ S, int ncp, int ns,
                                                        double2* __restrict__ part) {
    constexpr int NC = DIP ? 4 : 1;
    __shared__ double2 G[64][NC];
    __shared__ double2 red[8][kMaxStates * NC];
    const int tid = threadIdx.x, nsc = ns * NC;
    const double thr = p.thr[0];
    double2 acc = make_double2(0.0, 0.0);   // of (state, component) tid
    for (int k0 = blockIdx.x * 64; k0 < ncp; k0 += gridDim.x * 64) {
        const int k = k0 + (tid >> 2);
        double2 g[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) g[c] = make_double2(0.0, 0.0);
        if (k < ncp) {
            const int t0 = p.cp_first[k], t1 = t0 + p.cp_nterms[k];
            for (int t = t0 + (tid & 3); t < t1; t += 4) {
                const double w = p.wt[t];
                const int4 tr = p.trow[t];
                if (!(thr < 0.0 || (w > 0.0 && w >= thr))) continue;
                if constexpr (DIP) {
                    const VRowDev &X = p.rows[tr.x], &Y = p.rows[tr.y], &Z = p.rows[tr.z];
                    const double x = X.e[0], y = Y.e[0], z = Z.e[0];
                    const double dx = fma(X.P, x, X.e[1]), dy = fma(Y.P, y, Y.e[1]), dz = fma(Z.P, z, Z.e[1]);
                    g[0].x += x * y * z;
                    g[1].x += dx * y * z;
                    g[2].x += x * dy * z;
                    g[3].x += x * y * dz;
                } else {
                    const double2 v = cmul(cmul(S[p.newid[tr.x]], S[p.newid[(size_t)p.nr + tr.y]]), S[p.newid[(size_t)2 * p.nr + tr.z]]);
                    g[0].x += v.x;
                    g[0].y += v.y;
                }
            }
        }
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            for (int o = 1; o < 4; o <<= 1) {
                g[c].x += __shfl_xor(g[c].x, o);
                if (!DIP) g[c].y += __shfl_xor(g[c].y, o);
            }
            if ((tid & 3) == 0) G[tid >> 2][c] = g[c];
        }
        __syncthreads();
        const int nk = min(64, ncp - k0);
        for (int i = tid; i < 8 * nsc; i += 256) {
            const int sl = i / nsc, sc = i - sl * nsc, s = sc / NC, c = sc - s * NC;
            double2 a = make_double2(0.0, 0.0);
            for (int j = 8 * sl; j < min(8 * sl + 8, nk); ++j) {
                const double t = p.tp64[(size_t)(k0 + j) * ns + s];
                a.x = fma(t, G[j][c].x, a.x);
                if (!DIP) a.y = fma(t, G[j][c].y, a.y);
            }
            red[sl][sc] = a;
        }
        __syncthreads();
        if (tid < nsc)
            for (int sl = 0; sl < 8; ++sl) {
                acc.x += red[sl][tid].x;
                acc.y += red[sl][tid].y;
            }
    }
    if (tid < nsc) part[(size_t)tid * gridDim.x + blockIdx.x] = acc;
}

// One wave per (state, component): strided sums, then a fixed tree.
__global__ __launch_bounds__(64) void sep_final_kernel(const double2* __restrict__ part, int nparts,
                                                       double2* __restrict__ out) {
    double2 a = make_double2(0.0, 0.0);
    for (int b = threadIdx.x; b < nparts; b += 64) {
        a.x += part[(size_t)blockIdx.x * nparts + b].x;
        a.y += part[(size_t)blockIdx.x * nparts + b].y;
    }
    for (int h = 32; h > 0; h >>= 1) {
        a.x += __shfl_xor(a.x, h);
        a.y += __shfl_xor(a.y, h);
    }
    if (threadIdx.x == 0) out[blockIdx.x] = a;
}

}  // namespace

// Workgroups (and partial sums per state and component) of the pair sums.
int sep_parts(int ncp) { return std::max(1, std::min(1024, (ncp + 63) / 64)); }

hipError_t launch_separable(const LowqPrep& p, const VRowDev* rows, int nrows, int ncp, int ns, const double2* w,
                            const int n[3], int sym, const double qmin[3], const double dq[3], double2* S, double2* part,
                            double2* out, hipStream_t st) {
    if (ns < 1 || ns > kMaxStates || ncp < 1) return hipErrorInvalidValue;
    hipError_t e;
    if (nrows > 1) {   // row 0 is the zero row
        hipLaunchKernelGGL(sep_rows_kernel, dim3((nrows - 1 + 31) / 32), dim3(256), 0, st, rows + 1, nrows - 1, w,
                           make_int3(n[0], n[1], n[2]), sym, make_double3(qmin[0], qmin[1], qmin[2]),
                           make_double3(dq[0], dq[1], dq[2]), S);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    hipLaunchKernelGGL(sep_pairs_kernel<false>, dim3(sep_parts(ncp)), dim3(256), 0, st, p, (const double2*)S, ncp, ns,
                       part);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(sep_final_kernel, dim3(ns), dim3(64), 0, st, (const double2*)part, sep_parts(ncp), out);
    return hipGetLastError();
}

hipError_t launch_dipole(const LowqPrep& p, int ncp, int ns, double2* part, double2* out, hipStream_t st) {
    if (ns < 1 || ns > kMaxStates || ncp < 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL(sep_pairs_kernel<true>, dim3(sep_parts(ncp)), dim3(256), 0, st, p, (const double2*)nullptr, ncp,
                       ns, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(sep_final_kernel, dim3(4 * ns), dim3(64), 0, st, (const double2*)part, sep_parts(ncp), out);
    return hipGetLastError();
}

}  // namespace scff
