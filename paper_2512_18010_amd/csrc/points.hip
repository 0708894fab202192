// f_s and |f_s|^2 at arbitrary points (gfx950 / CDNA4): the engine's point
// evaluation and the fit of the averaged |f|^2.
//
// One lane per point, one wave per (64 points, share of the shell pairs).  Per
// shell pair the component pairs' G = sum over kept primitive pairs of
// Vx Vy Vz are held in registers: the three axes of a primitive pair share one
// exponential and one phase (the product of the axes' Gaussians and of their
// phases), the axes' polynomials are shared by the component pairs, and
// everything that does not depend on the point is wave-uniform (scalar loads).
// Then f_s += sum_c Tp(s, c) G_c, eight states at a time, into LDS totals.  All
// in FP64, whose vector rate is half of FP32's here.  Shares of the shell pairs
// are summed in a fixed order by points_reduce_kernel.
//
// The kernel before walked all pairs in every lane (1000 points: 16 waves in
// all), evaluating an exponential, a sine and a cosine per term and axis: 54.4
// ms for 1000 points of a molecule with 10 heavy atoms and 12 states (its FP64
// twin 24.9 ms for the fit's 576 points, 4 heavy atoms, 3 states); now 276 and
// 111 us, sums included.  Bound now: FP64 issue and the scalar loads' latency
// at two waves per SIMD (registers: 36 complex G; one wave without spills: 478
// against 345 us per call).  Splitting a shell pair's primitive pairs over
// waves too repeats the contraction with the states: 407 us for two, 534 for
// four.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "engine.h"

namespace scff {

namespace {

__host__ __device__ constexpr int pt_cart(int l, int c, int ax) {   // powers in component order
    constexpr int t[3][6][3] = {
        {{0, 0, 0}},
        {{1, 0, 0}, {0, 1, 0}, {0, 0, 1}},
        {{2, 0, 0}, {1, 1, 0}, {1, 0, 1}, {0, 2, 0}, {0, 1, 1}, {0, 0, 2}},
    };
    return t[l][c][ax];
}

// What does not depend on the point is read through the constant address
// space: scalar loads (no kernel writes it while this one runs).
template <typename T>
using PtConst = const __attribute__((address_space(4))) T*;
template <typename T>
__device__ __forceinline__ PtConst<T> pt_const(const T* p) { return (PtConst<T>)(uintptr_t)p; }

// complex value whose imaginary part may be known to be zero
struct PtC {
    double r, i;
    bool real;
};
__device__ __forceinline__ PtC pt_mul(PtC a, PtC b) {
    if (a.real && b.real) return {a.r * b.r, 0.0, true};
    if (a.real) return {a.r * b.r, a.r * b.i, false};
    if (b.real) return {a.r * b.r, a.i * b.r, false};
    return {fma(-a.i, b.i, a.r * b.r), fma(a.i, b.r, a.r * b.i), false};
}

// sum_u e_u (i q)^u of degree D
template <int D>
__device__ __forceinline__ PtC pt_poly(PtConst<VRowDev> r, double q, double q2) {
    if constexpr (D == 0) return {r->e[0], 0.0, true};
    if constexpr (D == 1) return {r->e[0], q * r->e[1], false};
    double re = fma(-r->e[2], q2, r->e[0]), im = r->e[1];
    if constexpr (D >= 4) re = fma(r->e[4], q2 * q2, re);
    if constexpr (D >= 3) im = fma(-r->e[3], q2, im);
    return {re, q * im, false};
}

template <int NB, int NCP>
__device__ __forceinline__ void pt_states(PtConst<double> tp, int ns, const double (&gr)[NCP],
                                          const double (&gi)[NCP], double2* fl) {
    double ar[NB], ai[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j) ar[j] = ai[j] = 0.0;
#pragma unroll
    for (int c = 0; c < NCP; ++c)
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            const double t = tp[c * ns + j];
            ar[j] = fma(t, gr[c], ar[j]);
            ai[j] = fma(t, gi[c], ai[j]);
        }
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        double2 v = fl[64 * j];
        v.x += ar[j];
        v.y += ai[j];
        fl[64 * j] = v;
    }
}

// One shell pair: rows from s.z, terms from s.w, component pairs from cp0.
template <int LA, int LB, bool SAME>
__device__ __forceinline__ void pt_shell_pair(const PointArgs& a, int4 s, int cp0, int npp, double qx, double qy,
                                              double qz, double thr, double2* fl) {
    constexpr int NA = (LA + 1) * (LA + 2) / 2, NB = (LB + 1) * (LB + 2) / 2, NCLS = (LA + 1) * (LB + 1);
    constexpr int NCP = SAME ? NA * (NA + 1) / 2 : NA * NB;
    const int lane = threadIdx.x;
    const double q2x = qx * qx, q2y = qy * qy, q2z = qz * qz, q2 = q2x + q2y + q2z;
    double gr[NCP], gi[NCP];
#pragma unroll
    for (int c = 0; c < NCP; ++c) gr[c] = gi[c] = 0.0;
    bool any = false;
    // lane c holds the weight of component pair c's term: the kept ones as a mask
    const double* w = a.wt + s.w + (lane < NCP ? lane : 0) * npp;
    double wc = w[0];
    for (int pp = 0; pp < npp; ++pp) {
        const unsigned long long kept = __ballot(lane < NCP && (thr < 0.0 || (wc > 0.0 && wc >= thr)));
        wc = w[min(pp + 1, npp - 1)];
        if (!kept) continue;
        any = true;
        const PtConst<VRowDev> r = pt_const(a.rows) + s.z + pp * 3 * NCLS;
        const double rev =
            fma(qx, r[0].P, fma(qy, r[NCLS].P, qz * r[2 * NCLS].P)) * 0.15915494309189535;   // 1 / (2 pi)
        double sn, cs;
        sincospi(2.0 * (rev - rint(rev)), &sn, &cs);
        const double g = exp(-q2 * r[0].inv4p);
        const PtC ph{g * cs, g * sn, false};
        PtC X[NCLS], Y[NCLS], Z[NCLS];
        auto axis = [&](PtC(&o)[NCLS], PtConst<VRowDev> ra, double q, double qq) {
#pragma unroll
            for (int i = 0; i <= LA; ++i)
#pragma unroll
                for (int j = 0; j <= LB; ++j) {
                    const int k = i * (LB + 1) + j;
                    o[k] = i + j == 0   ? pt_poly<0>(ra + k, q, qq)
                           : i + j == 1 ? pt_poly<1>(ra + k, q, qq)
                           : i + j == 2 ? pt_poly<2>(ra + k, q, qq)
                           : i + j == 3 ? pt_poly<3>(ra + k, q, qq)
                                        : pt_poly<4>(ra + k, q, qq);
                }
        };
        axis(X, r, qx, q2x);
        axis(Y, r + NCLS, qy, q2y);
        axis(Z, r + 2 * NCLS, qz, q2z);
#pragma unroll
        for (int k = 0; k < NCLS; ++k) X[k] = pt_mul(X[k], ph);
        auto terms = [&](bool all) {
#pragma unroll
            for (int c1 = 0; c1 < NA; ++c1)
#pragma unroll
                for (int c2 = SAME ? c1 : 0; c2 < NB; ++c2) {
                    const int c = SAME ? c1 * NB - c1 * (c1 - 1) / 2 + (c2 - c1) : c1 * NB + c2;
                    const int kx = pt_cart(LA, c1, 0) * (LB + 1) + pt_cart(LB, c2, 0);
                    const int ky = pt_cart(LA, c1, 1) * (LB + 1) + pt_cart(LB, c2, 1);
                    const int kz = pt_cart(LA, c1, 2) * (LB + 1) + pt_cart(LB, c2, 2);
                    if (all || (kept >> c & 1)) {
                        const PtC v = pt_mul(X[kx], Y[ky]), z = Z[kz];
                        gr[c] = fma(v.r, z.r, gr[c]);
                        gi[c] = fma(v.i, z.r, gi[c]);
                        if (!z.real) {
                            gr[c] = fma(-v.i, z.i, gr[c]);
                            gi[c] = fma(v.r, z.i, gi[c]);
                        }
                    }
                }
        };
        if (kept == (NCP == 64 ? ~0ull : (1ull << NCP) - 1)) terms(true);
        else terms(false);
    }
    if (!any) return;
    const PtConst<double> tp = pt_const(a.tp64) + (size_t)cp0 * a.ns;
    int st = 0;
    for (; st + 8 <= a.ns; st += 8) pt_states<8, NCP>(tp + st, a.ns, gr, gi, fl + 64 * st);
    for (; st + 4 <= a.ns; st += 4) pt_states<4, NCP>(tp + st, a.ns, gr, gi, fl + 64 * st);
    for (; st < a.ns; ++st) pt_states<1, NCP>(tp + st, a.ns, gr, gi, fl + 64 * st);
}

__device__ __forceinline__ void pt_store(const PointArgs& a, int s, int iq, double re, double im) {
    const size_t o = (size_t)s * a.nq + iq;
    if (a.f) a.f[o] = make_float2((float)re, (float)im);
    if (a.f2) a.f2[o] = (float)(re * re + im * im);
    if (a.f2d) a.f2d[o] = re * re + im * im;
}

}  // namespace

__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2, 2))) void points_kernel(PointArgs a) {
    extern __shared__ __align__(16) double2 pt_lds[];   // [states][64 points]
    const int lane = threadIdx.x;
    double2* fl = pt_lds + lane;
    for (int s = 0; s < a.ns; ++s) fl[64 * s] = make_double2(0.0, 0.0);
    const int iq = blockIdx.x * 64 + lane, ic = min(iq, a.nq - 1);
    const double qx = a.q[3 * (size_t)ic], qy = a.q[3 * (size_t)ic + 1], qz = a.q[3 * (size_t)ic + 2];
    const double thr = pt_const(a.thr)[0];
    for (int isp = blockIdx.y; isp < a.n_sp; isp += gridDim.y) {
        const PtConst<int> e = pt_const((const int*)(a.sp + isp));
        const int4 s = make_int4(e[0], e[1], e[2], e[3]);
        const PtConst<PrepShell> A = pt_const(a.shells) + s.x, B = pt_const(a.shells) + s.y;
        const int npp = A->nprim * B->nprim, cp0 = pt_const(a.sp_cp)[isp];
#define PT_CASE(la, lb) \
    case (la) * 6 + (lb) * 2: pt_shell_pair<la, lb, false>(a, s, cp0, npp, qx, qy, qz, thr, fl); break;
#define PT_SAME(l) \
    case (l) * 8 + 1: pt_shell_pair<l, l, true>(a, s, cp0, npp, qx, qy, qz, thr, fl); break;
        switch (A->l * 6 + B->l * 2 + (s.x == s.y ? 1 : 0)) {
            PT_CASE(0, 0) PT_CASE(0, 1) PT_CASE(0, 2)
            PT_CASE(1, 0) PT_CASE(1, 1) PT_CASE(1, 2)
            PT_CASE(2, 0) PT_CASE(2, 1) PT_CASE(2, 2)
            PT_SAME(0) PT_SAME(1) PT_SAME(2)
        }
#undef PT_CASE
#undef PT_SAME
    }
    if (iq >= a.nq) return;
    for (int s = 0; s < a.ns; ++s) {
        const double2 v = fl[64 * s];
        if (a.part) a.part[((size_t)blockIdx.y * a.ns + s) * a.nq + iq] = v;
        else pt_store(a, s, iq, v.x, v.y);
    }
}

// Sums the shares: 4 quarters of them per (state, point), then the quarters.
__global__ __launch_bounds__(256) void points_reduce_kernel(PointArgs a, int n_split) {
    __shared__ double2 red[4][64];
    const int lane = threadIdx.x & 63, h = threadIdx.x >> 6;
    const size_t tot = (size_t)a.ns * a.nq, i = blockIdx.x * (size_t)64 + lane;
    double2 v = make_double2(0.0, 0.0);
    if (i < tot)
        for (int j = n_split * h / 4; j < n_split * (h + 1) / 4; ++j) {
            const double2 p = a.part[j * tot + i];
            v.x += p.x;
            v.y += p.y;
        }
    red[h][lane] = v;
    __syncthreads();
    if (h || i >= tot) return;
    for (int k = 1; k < 4; ++k) {
        v.x += red[k][lane].x;
        v.y += red[k][lane].y;
    }
    pt_store(a, (int)(i / a.nq), (int)(i % a.nq), v.x, v.y);
}

// Shares of the shell pairs: enough for 4096 waves (two rounds of the device's
// resident ones, so that uneven shares level out), at most 256 and as many as
// the partial sums' 64 MB hold.
int points_split(int nq, int ns, int n_sp) {
    const long long blocks = (nq + 63) / 64, bytes = (long long)nq * ns * (long long)sizeof(double2);
    const long long s = std::min<long long>({4096 / blocks, 256, n_sp, (64LL << 20) / bytes});
    return (int)std::max<long long>(1, s);
}

hipError_t launch_points(const PointArgs& a, int n_split, hipStream_t st) {
    if (a.nq < 1 || a.ns < 1 || a.ns > kMaxStates || a.n_sp < 1 || n_split < 1 || n_split > 65535 ||
        (n_split > 1) != (a.part != nullptr))
        return hipErrorInvalidValue;
    hipLaunchKernelGGL(points_kernel, dim3((a.nq + 63) / 64, n_split), dim3(64), (size_t)a.ns * 64 * sizeof(double2), st,
                       a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || n_split == 1) return e;
    const size_t blocks = ((size_t)a.ns * a.nq + 63) / 64;
    if (blocks > 0x7fffffff) return hipErrorInvalidValue;
    hipLaunchKernelGGL(points_reduce_kernel, dim3((unsigned)blocks), dim3(256), 0, st, a, n_split);
    return hipGetLastError();
}

}  // namespace scff
