// The FFT method (paper Sec. 3 and Sec. 5.2) on the device:
//
//   1. fft_pack_kernel      transition weights as MFMA A operands:
//                           s_f c_mu c_nu (T_{mu nu} + T_{nu mu}) per unordered
//                           component pair (T_{mu mu} on the diagonal), split
//                           into three BF16 parts (FP32 precision) or two;
//   2. fft_density_kernel   the transition density (eq. PhiTDM, AO form)
//                             Phi_s(r) = sum_mu phi_mu(r) sum_{nu >= mu} Tp_s(mu,nu) phi_nu(r)
//                           on a tile of up to 64 real-space points: the AO
//                           values of the tile are formed in LDS (FP64,
//                           rounded once and split into three BF16 parts; or FP32
//                           and split into two), Y_s(mu, r) = sum_nu Tp_s(mu,nu) phi_nu(r)
//                           runs on the matrix cores (rows mu of one state,
//                           k = nu, columns = points), and sum_mu phi_mu Y_s(mu)
//                           is folded per 16 rows.  Two states share one
//                           complex array (Phi_2b + i Phi_2b+1), so each FFT
//                           carries two.
//   3. fft_lines_kernel     radix-2 transforms of all lines of one axis of the
//                           complex arrays, a line group staged in LDS (eq.
//                           Falbega as three 1D passes);
//   4. fft_finish_kernel    separates the two states of each array
//                           (F_a = (Z_k + Z*_{-k})/2, F_b = (Z_k - Z*_{-k})/2i),
//                           orders the frequencies most negative first and
//                           applies the pixel volume and the corner phase:
//                           f_s(q) = V_pix e^{+i q.x_min} conj(F_s) (eq.
//                           fftABC for the conjugate array, eq. qabc);
//   5. fft_sum_kernel       the two sides of Parseval's identity (Sec. 7) from
//                           per-wave FP64 partial sums, in a fixed order.
#include <hip/hip_runtime.h>

#include "engine.h"

namespace scff {

typedef float fft_floatx4 __attribute__((ext_vector_type(4)));
typedef float fft_floatx2 __attribute__((ext_vector_type(2)));
typedef unsigned int fft_uintx4 __attribute__((ext_vector_type(4)));
typedef __bf16 fft_bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 fft_bf16x8 __attribute__((ext_vector_type(8)));

// Split-BF16 of one value: hi = RNE(v), lo = RNE(v - hi), each in the low
// half of a dword whose high half is zero.  v - hi is exact in FP32, so the
// BF16 dot product hi . (-1, -0) + v gives it in one instruction (-0, not +0:
// the compiler would encode (-1, +0) as the inline constant -1.0, which the
// instruction reads as the BF16 pair (+0, -1)).
__device__ inline void fft_split(float v, uint32_t& hi, uint32_t& lo) {
    const fft_bf16x2 h = __builtin_convertvector(fft_floatx2{v, 0.f}, fft_bf16x2);
    const float r = __builtin_amdgcn_fdot2_f32_bf16(h, fft_bf16x2{(__bf16)-1.0f, (__bf16)-0.0f}, v, false);
    hi = __builtin_bit_cast(uint32_t, h);
    lo = __builtin_bit_cast(uint32_t, __builtin_convertvector(fft_floatx2{r, 0.f}, fft_bf16x2));
}
// The three BF16 parts of two values (the second's in the high halves), each the
// rest of the one before: FP32's 24 bits over its exponent range.
__device__ inline void fft_split3(float v0, float v1, uint32_t (&part)[3]) {
    const fft_bf16x2 first{(__bf16)-1.0f, (__bf16)-0.0f}, second{(__bf16)-0.0f, (__bf16)-1.0f};
#pragma unroll
    for (int p = 0; p < 3; ++p) {
        const fft_bf16x2 h = __builtin_convertvector(fft_floatx2{v0, v1}, fft_bf16x2);
        part[p] = __builtin_bit_cast(uint32_t, h);
        if (p < 2) {
            v0 = __builtin_amdgcn_fdot2_f32_bf16(h, first, v0, false);
            v1 = __builtin_amdgcn_fdot2_f32_bf16(h, second, v1, false);
        }
    }
}
// Primitives whose exponent argument alpha r^2 exceeds this are skipped (the
// paper's thresholding of negligible primitives): e^{-103} is below the
// smallest FP32 subnormal, so the rounded AO value is unchanged.
constexpr double kExpCut = 103.0;

namespace {

__device__ __forceinline__ double fft_weight(const double* Ts, const double* cnorm, int nbf, double spin, int mu,
                                             int nu) {
    const double t = mu == nu ? Ts[(size_t)mu * nbf + mu] : Ts[(size_t)mu * nbf + nu] + Ts[(size_t)nu * nbf + mu];
    return spin * cnorm[mu] * cnorm[nu] * t;
}

// First function group of row block rb in the A operands of a state (groups
// rb .. RB - 1 of every row block).
__device__ __forceinline__ int fft_group0(int rb, int RB) { return rb * RB - rb * (rb - 1) / 2; }

// A operands.  Function group g holds nu = 16 g .. 16 g + 15; lane (row = lane %
// 16, kk = lane / 16) carries nu_j = 16 g + 4 kk + j, j < 4, as the words of the
// first and of the second parts in Ap[((s groups + group0(rb) + g - rb) 64 + lane],
// g >= rb, and (FP32 precision) of the third parts in Ar.
template <bool BF>
__global__ void fft_pack_kernel(const double* __restrict__ T, const double* __restrict__ cnorm, int nbf, int ns, int RB,
                                double spin, uint4* __restrict__ Ap, uint2* __restrict__ Ar) {
    const int per = RB * (RB + 1) / 2;
    const long long total = (long long)ns * per * 64;
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < total;
         i += (long long)gridDim.x * blockDim.x) {
        const int lane = (int)(i & 63);
        const long long r = i >> 6;
        const int s = (int)(r / per), k = (int)(r - (long long)s * per);
        int rb = 0;
        while (fft_group0(rb + 1, RB) <= k) ++rb;
        const int g = rb + k - fft_group0(rb, RB);
        const int mu = 16 * rb + (lane & 15);
        const double* Ts = T + (size_t)s * nbf * nbf;
        float v[4];
        for (int j = 0; j < 4; ++j) {
            const int nu = 16 * g + 4 * (lane >> 4) + j;
            v[j] = mu < nbf && nu < nbf && mu <= nu ? (float)fft_weight(Ts, cnorm, nbf, spin, mu, nu) : 0.f;
        }
        uint32_t a[3], b[3];
        fft_split3(v[0], v[1], a);
        fft_split3(v[2], v[3], b);
        Ap[i] = make_uint4(a[0], b[0], a[1], b[1]);
        if (!BF) Ar[i] = make_uint2(a[2], b[2]);
    }
}

// e^{-x} for 0 <= x <= kExpCut in FP64, accurate to ~5e-9 relative (the
// value is rounded to FP32 afterwards): x = n ln2 + r with |r| <= ln2 / 2
// (ln2 in two parts, so r is exact to ~1e-16), e^{-r} by its Taylor
// polynomial of degree 7 (remainder r^8 / 8! < 5.2e-9), scaled by 2^{-n}.
__device__ __forceinline__ double fft_exp_neg(double x) {
    const double n = __builtin_rint(x * 1.4426950408889634);
    const double r = fma(n, 1.9082149292705877e-10, fma(n, 0.6931471803691238, -x));   // -(x - n ln2)
    double p = 1.0 / 5040.0;
    p = fma(p, r, 1.0 / 720.0);
    p = fma(p, r, 1.0 / 120.0);
    p = fma(p, r, 1.0 / 24.0);
    p = fma(p, r, 1.0 / 6.0);
    p = fma(p, r, 0.5);
    p = fma(p, r, 1.0);
    p = fma(p, r, 1.0);
    return __builtin_ldexp(p, -(int)n);
}

// AO values of one shell at one point before the contracted normalisation
// (c_mu is folded into the packed weights), handed to put(row, value) for
// each Cartesian component (row = bf0 + c).  F is double (the FP32
// contraction: values rounded once to FP32) or float (the split-BF16
// contraction, whose operands keep 16 significant bits: the offsets from the
// centre are formed in FP64 and rounded, the rest runs in FP32 with the
// hardware 2^x).
template <typename F, typename Put>
__device__ __forceinline__ void shell_values(const FftMol& m, int sh, double x, double y, double z, Put put) {
    const PrepShell S = m.shells[sh];
    const double* A = m.xyz + 3 * S.atom;
    const F dx = (F)(x - A[0]), dy = (F)(y - A[1]), dz = (F)(z - A[2]);
    const F r2 = dx * dx + dy * dy + dz * dz;
    // radial sums: sum_k d_k (product of 1D norms for the power pattern) e^{-alpha_k r^2}
    F ra = 0, rb = 0;   // l = 2: ra for xx-type, rb for xy-type; l < 2: ra only
    for (int k = 0; k < S.nprim; ++k) {
        const int o = S.off + k;
        const F ar = (F)m.exps[o] * r2;
        if (ar > (F)kExpCut) continue;
        F e;
        if constexpr (sizeof(F) == 8)
            e = (F)m.coefs[o] * fft_exp_neg(ar);
        else
            e = (F)m.coefs[o] * __builtin_amdgcn_exp2f(ar * -1.44269504f);
        const F n0 = (F)m.n1d[3 * o], n1 = (F)m.n1d[3 * o + 1], n2 = (F)m.n1d[3 * o + 2];
        if (S.l == 0) {
            ra += e * (n0 * n0 * n0);
        } else if (S.l == 1) {
            ra += e * (n1 * n0 * n0);
        } else {
            ra += e * (n2 * n0 * n0);
            rb += e * (n1 * n1 * n0);
        }
    }
    const int b0 = m.bf0[sh];
    if (S.l == 0) {
        put(b0, ra);
    } else if (S.l == 1) {
        put(b0, dx * ra);
        put(b0 + 1, dy * ra);
        put(b0 + 2, dz * ra);
    } else {
        put(b0, dx * dx * ra);
        put(b0 + 1, dx * dy * rb);
        put(b0 + 2, dx * dz * rb);
        put(b0 + 3, dy * dy * ra);
        put(b0 + 4, dy * dz * rb);
        put(b0 + 5, dz * dz * ra);
    }
}

// LDS bytes of a density workgroup of nw waves: the AO block of nbf_pad rows x 16
// CB points (two or three parts of 2 bytes per value) and two buffers of nw x 16 CB
// FP64 partial densities.
__host__ __device__ constexpr size_t fft_lds_bytes(bool bf, int nbf_pad, int cb, int nw) {
    return (size_t)cb * ((bf ? 64 : 96) * (size_t)nbf_pad + 256 * nw);
}

// One workgroup (NW waves) per tile of NP = 16 CB consecutive grid points
// (flattened [ix][iy][iz], z fastest; column c = 16 cb + col of the tile).
//
// AO phase: a lane evaluates one shell at one point (64 / NP shells per wave
// step; with NP = 64 every lane of a wave takes the same shell, so its data
// are scalar loads).  The values end in LDS as parts, the B operands of a
// 16x16x32 matrix instruction: the uint4 entry ((g 4 + kk) CB + cb) 16 + col holds
// the first and second BF16 parts of the rows r_j = 16 g + 4 kk + j (j < 4) of
// column c, as (h(r_0) | h(r_1) << 16, h(r_2) | h(r_3) << 16, m(r_0) | m(r_1) << 16,
// m(r_2) | m(r_3) << 16); FP32 precision: the uint2 entry of the same number behind
// them the third parts.  A lane (kk, col) takes an entry as the 8 k-items of one
// instruction (no operand copies), and the same entry holds the rows 16 rb + 4 kk +
// i that the lane folds after row block rb.
// Products per function group and column block: with W = (h, m, l) and phi = (h,
// m, l) the instructions (W_h, W_h) (phi_h, phi_m), (W_m, W_m) (phi_h, phi_m) and (W_l,
// W_h) (phi_h, phi_l): every product above 2^-24 of the whole.  BF (split-BF16): two
// parts each, the first instruction and (W_m, 0) (phi_h, phi_m).
//
// FP32 precision used FP32 matrix instructions, 2.7x the cycles of the split
// products: 8.9 ms a call for 190 functions, 12 states on 128^3 points, 74 % of it in
// the matrix cores; 6.3 ms now, bound by the vector unit (AO values and fold, FP64)
// and the matrix cores in equal parts, which overlap little at two waves per SIMD.
// f16 halves of the AO values, scaled per point, take 4 bytes instead of 6 and let
// three workgroups stay on a CU (4.75 ms), but a shell whose coefficients are given
// small (the contracted norm is in the weights) then falls below a point's smallest
// half: density error 1 for coefficients of 1e-12.  Error over 48 boxes of 80 to
// 420 functions, rms against the peak: 0.64 to 1.05e-8, FP32 matrix instructions
// 0.76 to 1.3e-8.
//
// Contraction: wave w takes row blocks rb of 16 functions in a snake order
// (0 1 .. NW - 1 NW - 1 .. 1 0 ...), which evens out the triangle's rows; per row block
// the k-steps from the diagonal block on, with the A operands of the next
// k-steps loaded while the current ones run and each A operand used by CB
// MFMAs.  The 16-row block is folded with its AO values, the waves'
// partial densities of a group of states are summed through LDS and wave 0
// writes the tile.
template <bool BF, int CB, int NW, int WPS>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(WPS))) void fft_density_kernel(FftMol m, const uint4* __restrict__ Av,
                                                          const uint2* __restrict__ Ar, int nbf_pad, int ns, int RB,
                                                          int3 n, double3 x0, double3 h,
                                                          long long npts, float* __restrict__ Z,
                                                          float* __restrict__ phi_out, double* __restrict__ psum) {
    extern __shared__ __align__(16) float fft_lds[];
    constexpr int NP = 16 * CB, NT = 64 * NW;
    // MFMA accumulator chains: per column block one, or (TWO; where the registers
    // hold them) one of the first products and one of the small ones, so that these
    // are not rounded to the whole sum each time
    constexpr bool TWO = CB == 1 || (!BF && !(CB == 4 && WPS > 2));
    constexpr int NCH = TWO ? 2 * CB : CB;
    const int tid = threadIdx.x, lane = tid & 63;
    // wave-uniform: the row-block loop and the A-operand addresses stay scalar
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const long long p0 = (long long)blockIdx.x * NP;
    uint32_t* pu = reinterpret_cast<uint32_t*>(fft_lds);
    unsigned short* ps16 = reinterpret_cast<unsigned short*>(fft_lds);
    constexpr int WV = BF ? 2 : 3;   // parts of a value
    uint2* const p3 = reinterpret_cast<uint2*>(ps16 + (size_t)2 * nbf_pad * NP);   // third parts
    double* red = reinterpret_cast<double*>(ps16 + (size_t)WV * nbf_pad * NP);

    for (int i = tid; i < nbf_pad * NP / 4; i += NT) reinterpret_cast<uint4*>(pu)[i] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    {
        constexpr int SPI = 64 / NP;   // shells per wave step
        const int p = lane % NP;
        const long long g = p0 + p;
        const int iz = (int)(g % n.z);
        const long long r1 = g / n.z;
        const int iy = (int)(r1 % n.y), ix = (int)(r1 / n.y);
        const double x = x0.x + ix * h.x, y = x0.y + iy * h.y, z = x0.z + iz * h.z;
        const int col = p & 15, cb = p >> 4;
        auto put = [&](int r, auto v) {
            const int i = r & 3;
            const int e0 = (((r >> 4) * 4 + ((r >> 2) & 3)) * CB + cb) * 16 + col;   // the entry
            if constexpr (BF) {
                uint32_t hi, lo;
                fft_split((float)v, hi, lo);
                ps16[8 * e0 + i] = (unsigned short)hi;
                ps16[8 * e0 + 4 + i] = (unsigned short)lo;
            } else {
                pu[4 * e0 + i] = __float_as_uint((float)v);
            }
        };
        for (int sh0 = wave * SPI; sh0 < m.n_shells; sh0 += NW * SPI) {
            const int sh = sh0 + lane / NP;
            if (sh < m.n_shells && g < npts) shell_values<std::conditional_t<BF, float, double>>(m, sh, x, y, z, put);
        }
    }

    if constexpr (!BF) {   // values to parts, in place (one LDS write a value before instead of three)
        __syncthreads();
        for (int i = tid; i < nbf_pad * NP / 4; i += NT) {
            uint4* const o = reinterpret_cast<uint4*>(pu) + i;
            const uint4 u = *o;
            uint32_t a[3], b[3];
            fft_split3(__uint_as_float(u.x), __uint_as_float(u.y), a);
            fft_split3(__uint_as_float(u.z), __uint_as_float(u.w), b);
            *o = make_uint4(a[0], b[0], a[1], b[1]);
            p3[i] = make_uint2(a[2], b[2]);
        }
    }

    const int kk = lane >> 4, col = lane & 15;
    // the AO values of rows 16 rb + 4 kk + i (i < 4) at this lane's CB columns,
    // v[i][cb]: the parts, summed in FP32 (exact for three parts; for two within
    // 2^-24 of the split value, far below the split's own 2^-16)
    using FV = std::conditional_t<BF, float, double>;
    auto phi_rows = [&](int rb, FV (&v)[4][CB]) {
#pragma unroll
        for (int q = 0; q < CB; ++q) {
            const uint4 e = reinterpret_cast<const uint4*>(pu)[((rb * 4 + kk) * CB + q) * 16 + col];
            float w[4] = {__uint_as_float(e.z << 16), __uint_as_float(e.z & 0xffff0000u), __uint_as_float(e.w << 16),
                          __uint_as_float(e.w & 0xffff0000u)};
            if constexpr (!BF) {
                const uint2 t = p3[((rb * 4 + kk) * CB + q) * 16 + col];
                w[0] += __uint_as_float(t.x << 16);
                w[1] += __uint_as_float(t.x & 0xffff0000u);
                w[2] += __uint_as_float(t.y << 16);
                w[3] += __uint_as_float(t.y & 0xffff0000u);
            }
            v[0][q] = __uint_as_float(e.x << 16) + w[0];
            v[1][q] = __uint_as_float(e.x & 0xffff0000u) + w[1];
            v[2][q] = __uint_as_float(e.y << 16) + w[2];
            v[3][q] = __uint_as_float(e.y & 0xffff0000u) + w[3];
        }
    };
    __syncthreads();

    // function group k (functions 16 k .. 16 k + 15) of row block rb for all CB
    // column blocks; the two products of a column block go to different chains
    // (CB = 1) or are CB instructions apart
    struct AOp {
        uint4 a;
        uint2 r;   // third parts (not BF)
    };
    auto kstep = [&](const AOp& o, int k, fft_floatx4 (&c)[NCH]) {
        const uint4 a = o.a;
        fft_uintx4 B[CB];
        uint2 Bl[CB];
#pragma unroll
        for (int q = 0; q < CB; ++q) {
            const int i = ((k * 4 + kk) * CB + q) * 16 + col;
            const uint4 e = reinterpret_cast<const uint4*>(pu)[i];
            B[q] = fft_uintx4{e.x, e.y, e.z, e.w};
            if constexpr (!BF) Bl[q] = p3[i];
        }
        auto mma = [](fft_uintx4 x, fft_uintx4 y, fft_floatx4 z) {
            return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(fft_bf16x8, x),
                                                           __builtin_bit_cast(fft_bf16x8, y), z, 0, 0, 0);
        };
        const fft_uintx4 A1{a.x, a.y, a.x, a.y}, A2{a.z, a.w, BF ? 0u : a.z, BF ? 0u : a.w};
        if constexpr (!BF) {
            const fft_uintx4 A3{o.r.x, o.r.y, a.x, a.y};
#pragma unroll
            for (int q = 0; q < CB; ++q)
                c[NCH - CB + q] = mma(A3, fft_uintx4{B[q][0], B[q][1], Bl[q].x, Bl[q].y}, c[NCH - CB + q]);
        }
#pragma unroll
        for (int q = 0; q < CB; ++q) c[NCH - CB + q] = mma(A2, B[q], c[NCH - CB + q]);
#pragma unroll
        for (int q = 0; q < CB; ++q) c[q] = mma(A1, B[q], c[q]);
    };

    // the k-steps k0 .. k0 + nk - 1 of one row block (nk >= 1).  The main loop runs whole blocks of 2 PD k-steps with no exit
    // inside, the A operands of the next PD k-steps loaded while the current
    // PD run (an exit between a load and its use lets the compiler sink the
    // load to the use, which then waits for it); the last 0 .. 2 PD - 1
    // k-steps run in a guarded tail.  Loads past the row block read the next
    // block or the array's slack and are not used.
    constexpr int PD = BF ? 4 : 2;   // k-steps per register set (prefetch depth)
    auto run_row = [&](size_t a0, int k0, int nk, fft_floatx4 (&c)[NCH]) {
        AOp A0[PD], A1[PD];
        auto load = [&](int k) {
            AOp o;
            o.a = Av[a0 + (size_t)k * 64 + lane];
            o.r = BF ? make_uint2(0, 0) : Ar[a0 + (size_t)k * 64 + lane];
            return o;
        };
#pragma unroll
        for (int j = 0; j < PD; ++j) A0[j] = load(j);
        int t = 0;
        for (; t + 2 * PD <= nk; t += 2 * PD) {
#pragma unroll
            for (int j = 0; j < PD; ++j) A1[j] = load(t + PD + j);
#pragma unroll
            for (int j = 0; j < PD; ++j) kstep(A0[j], k0 + t + j, c);
#pragma unroll
            for (int j = 0; j < PD; ++j) A0[j] = load(t + 2 * PD + j);
#pragma unroll
            for (int j = 0; j < PD; ++j) kstep(A1[j], k0 + t + PD + j, c);
        }
        const int r = nk - t;   // wave-uniform
        if (r > 0) {
#pragma unroll
            for (int j = 0; j < PD; ++j) A1[j] = load(t + PD + j);
#pragma unroll
            for (int j = 0; j < PD; ++j) {
                if (j >= r) return;
                kstep(A0[j], k0 + t + j, c);
            }
#pragma unroll
            for (int j = 0; j < PD; ++j) {
                if (PD + j >= r) return;
                kstep(A1[j], k0 + t + PD + j, c);
            }
        }
    };

    // States in groups of SG: the AO values of a row block are formed once per
    // group, and the waves' partial densities of the group meet in one
    // LDS slot (two barriers per group).  The fold over a wave's row blocks is
    // FP64 for the FP32 contraction and FP32 for split-BF16 (whose products
    // carry 16 significant bits); the slot holds SG x 4 x NP of them, within
    // the 64 NP bytes set aside.
    constexpr int SG = 2;
    FV* rd = reinterpret_cast<FV*>(red);
    for (int s0 = 0; s0 < ns; s0 += SG) {
        FV acc[SG][CB];
#pragma unroll
        for (int si = 0; si < SG; ++si)
#pragma unroll
            for (int q = 0; q < CB; ++q) acc[si][q] = 0;
        for (int i0 = 0, odd = 0; i0 < RB; i0 += NW, odd ^= 1) {
            // snake order: blocks i0 .. i0 + NW - 1 go to waves 0 .. NW - 1, then back
            const int rb = i0 + (odd ? NW - 1 - wave : wave);
            if (rb >= RB) continue;
            // lane (kk, col) holds rows 16 rb + 4 kk + i of its columns
            FV v[4][CB];
            phi_rows(rb, v);
#pragma unroll
            for (int si = 0; si < SG; ++si) {
                const int s = s0 + si;
                if (s >= ns) break;
                fft_floatx4 c[NCH];
#pragma unroll
                for (int q = 0; q < NCH; ++q) c[q] = fft_floatx4{0.f, 0.f, 0.f, 0.f};
                run_row(((size_t)s * (RB * (RB + 1) / 2) + fft_group0(rb, RB)) * 64, rb, RB - rb, c);
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int q = 0; q < CB; ++q) {
                        const float y = TWO ? c[q][i] + c[NCH - CB + q][i] : c[q][i];
                        acc[si][q] += v[i][q] * (FV)y;
                    }
            }
        }
#pragma unroll
        for (int si = 0; si < SG; ++si)
#pragma unroll
            for (int q = 0; q < CB; ++q) {
                FV a = acc[si][q];
                a += __shfl_xor(a, 16);
                a += __shfl_xor(a, 32);
                if (lane < 16) rd[(si * NW + wave) * NP + q * 16 + lane] = a;
            }
        __syncthreads();
        if (wave == 0) {
            const long long g = p0 + lane;
            const bool valid = lane < NP && g < npts;
#pragma unroll
            for (int si = 0; si < SG; ++si) {
                const int s = s0 + si;
                if (s >= ns) break;
                const FV* rw = rd + si * NW * NP;
                double d = 0.0;
                if (lane < NP)
#pragma unroll
                    for (int w = 0; w < NW; ++w) d += (double)rw[w * NP + lane];
                if (valid) {
                    const float v = (float)d;
                    float* zp = Z + ((size_t)(s >> 1) * npts + g) * 2;
                    zp[s & 1] = v;
                    if ((ns & 1) && s == ns - 1) zp[1] = 0.f;
                    if (phi_out) phi_out[(size_t)s * npts + g] = v;
                }
                double q = valid ? d * d : 0.0;
#pragma unroll
                for (int o = 1; o < 64; o <<= 1) q += __shfl_xor(q, o);
                if (psum && lane == 0) psum[(size_t)s * gridDim.x + blockIdx.x] = q;
            }
        }
        __syncthreads();
    }
}

// Lines of one axis of the complex arrays Z[nb][nx][ny][nz]: a workgroup
// transforms M lines of length N in LDS (radix-2, decimation in time on
// bit-reversed input), with twiddles e^{-2 pi i k / N} built in FP64 and
// rounded.  Along z the M lines are consecutive rows; along y and x they are
// M consecutive z, so every load and store touches contiguous runs.
__global__ __launch_bounds__(256) void fft_lines_kernel(float2* __restrict__ Z, int axis, int3 n, int nb, int M,
                                                        long long lines) {
    extern __shared__ __align__(16) float fft_lds[];
    const int N = axis == 0 ? n.x : axis == 1 ? n.y : n.z;
    const int logN = 31 - __clz(N);
    float2* buf = reinterpret_cast<float2*>(fft_lds);
    float2* tw = buf + (size_t)M * N;
    for (int k = threadIdx.x; k < N / 2; k += blockDim.x) {
        double sn, cs;
        sincospi(-2.0 * k / N, &sn, &cs);
        tw[k] = make_float2((float)cs, (float)sn);
    }
    const long long plane = (long long)n.y * n.z, vol = (long long)n.x * plane;
    const long long gidx = blockIdx.x;
    long long base, es, ls;
    int mcount = M;
    if (axis == 2) {
        base = gidx * M * N;
        es = 1;
        ls = N;
        const long long left = lines - gidx * M;
        if (left < M) mcount = (int)left;
    } else {
        const int zb = n.z / M;
        const int z0 = (int)(gidx % zb) * M;
        const long long r = gidx / zb;
        if (axis == 1) {
            const int x = (int)(r % n.x);
            const long long b = r / n.x;
            base = b * vol + (long long)x * plane + z0;
            es = n.z;
        } else {
            const int y = (int)(r % n.y);
            const long long b = r / n.y;
            base = b * vol + (long long)y * n.z + z0;
            es = plane;
        }
        ls = 1;
    }
    (void)nb;
    const int tot = mcount * N;
    for (int i = threadIdx.x; i < tot; i += blockDim.x) {
        int mm, k;
        if (axis == 2) {
            mm = i / N;
            k = i - mm * N;
        } else {
            k = i / mcount;
            mm = i - k * mcount;
        }
        const float2 v = Z[base + mm * ls + k * es];
        buf[mm * N + (int)(__brev((unsigned)k) >> (32 - logN))] = v;
    }
    __syncthreads();
    const int hN = N / 2;
    for (int len = 2; len <= N; len <<= 1) {
        const int half = len >> 1, tstep = N / len;
        for (int j = threadIdx.x; j < mcount * hN; j += blockDim.x) {
            const int mm = j / hN, r = j - mm * hN;
            const int grp = r / half, pos = r - grp * half;
            const int i0 = mm * N + grp * len + pos, i1 = i0 + half;
            const float2 w = tw[pos * tstep];
            const float2 a = buf[i0], b = buf[i1];
            const float tr = w.x * b.x - w.y * b.y, ti = w.x * b.y + w.y * b.x;
            buf[i0] = make_float2(a.x + tr, a.y + ti);
            buf[i1] = make_float2(a.x - tr, a.y - ti);
        }
        __syncthreads();
    }
    for (int i = threadIdx.x; i < tot; i += blockDim.x) {
        int mm, k;
        if (axis == 2) {
            mm = i / N;
            k = i - mm * N;
        } else {
            k = i / mcount;
            mm = i - k * mcount;
        }
        Z[base + mm * ls + k * es] = buf[mm * N + k];
    }
}

// One thread per output point (i, j, k) of every state: q_a = 2 pi (i_a - n_a/2) / L_a.
__global__ __launch_bounds__(256) void fft_finish_kernel(const float2* __restrict__ Z, int3 n, int ns, double vpix,
                                                         double3 u, long long npts, float2* __restrict__ f,
                                                         float* __restrict__ f2, double* __restrict__ psum) {
    const long long idx = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    const bool valid = idx < npts;
    const int lane = threadIdx.x & 63;
    const long long wv = idx >> 6;   // global wave index
    const long long nwv = (npts + 63) >> 6;
    long long src = 0, mir = 0;
    double cs = 1.0, sn = 0.0;
    if (valid) {
        const int k = (int)(idx % n.z);
        const long long r1 = idx / n.z;
        const int j = (int)(r1 % n.y), i = (int)(r1 / n.y);
        const int ai = i - n.x / 2, aj = j - n.y / 2, ak = k - n.z / 2;
        const int si = (i + n.x / 2) & (n.x - 1), sj = (j + n.y / 2) & (n.y - 1), sk = (k + n.z / 2) & (n.z - 1);
        const int mi = (n.x - si) & (n.x - 1), mj = (n.y - sj) & (n.y - 1), mk = (n.z - sk) & (n.z - 1);
        src = ((long long)si * n.y + sj) * n.z + sk;
        mir = ((long long)mi * n.y + mj) * n.z + mk;
        // q.x_min / (2 pi) in turns, reduced to [-1/2, 1/2], in FP64
        double t = ai * u.x + aj * u.y + ak * u.z;
        t -= rint(t);
        sincospi(2.0 * t, &sn, &cs);
    }
    for (int s = 0; s < ns; ++s) {
        double a2 = 0.0;
        if (valid) {
            const float2 zs = Z[(size_t)(s >> 1) * npts + src];
            const float2 zm = Z[(size_t)(s >> 1) * npts + mir];
            double fr, fi;   // F_s
            if ((s & 1) == 0) {
                fr = 0.5 * ((double)zs.x + (double)zm.x);
                fi = 0.5 * ((double)zs.y - (double)zm.y);
            } else {
                fr = 0.5 * ((double)zs.y + (double)zm.y);
                fi = -0.5 * ((double)zs.x - (double)zm.x);
            }
            // f = V_pix e^{i theta} conj(F)
            const double vr = vpix * (cs * fr + sn * fi), vi = vpix * (sn * fr - cs * fi);
            a2 = vr * vr + vi * vi;
            const size_t o = (size_t)s * npts + idx;
            if (f) f[o] = make_float2((float)vr, (float)vi);
            if (f2) f2[o] = (float)a2;
        }
        if (psum) {
            for (int d = 1; d < 64; d <<= 1) a2 += __shfl_xor(a2, d);
            if (lane == 0 && wv < nwv) psum[(size_t)s * nwv + wv] = a2;
        }
    }
}

// out[s * stride] = sum of part[s][0..n) in a fixed order (one workgroup per state).
__global__ __launch_bounds__(256) void fft_sum_kernel(const double* __restrict__ part, long long n, double scale,
                                                      double* __restrict__ out, int stride) {
    __shared__ double sm[256];
    const int s = blockIdx.x;
    double a = 0.0;
    for (long long i = threadIdx.x; i < n; i += 256) a += part[(size_t)s * n + i];
    sm[threadIdx.x] = a;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) sm[threadIdx.x] += sm[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[(size_t)s * stride] = scale * sm[0];
}

}  // namespace

// Bytes of the A operands: the upper triangle of function groups per state and
// what the density kernel loads past a row block (up to 7 groups, unused); FP32
// precision (up to 3): the same of the third parts.
static size_t fft_groups(int nbf_pad, int ns) {
    const size_t RB = nbf_pad / 16;
    return (size_t)ns * (RB * (RB + 1) / 2);
}
struct FftPack {
    size_t ar, total;   // offset of the third parts
};
static FftPack fft_pack_layout(int precision, int nbf_pad, int ns) {
    const size_t g = fft_groups(nbf_pad, ns);
    FftPack p;
    if (precision == SCFF_BF16X3) {
        p.ar = p.total = (g + 7) * 64 * sizeof(uint4);
    } else {
        p.ar = (g + 3) * 64 * sizeof(uint4);
        p.total = p.ar + (g + 3) * 64 * sizeof(uint2);
    }
    return p;
}
size_t fft_pack_bytes(int precision, int nbf_pad, int ns) { return fft_pack_layout(precision, nbf_pad, ns).total; }

hipError_t launch_fft_pack(int precision, const double* T, const double* cnorm, int nbf, int nbf_pad, int ns,
                           double spin, void* Ap, hipStream_t st) {
    const int RB = nbf_pad / 16;
    const FftPack p = fft_pack_layout(precision, nbf_pad, ns);
    uint2* ar = (uint2*)((char*)Ap + p.ar);
    const long long total = (long long)fft_groups(nbf_pad, ns) * 64;
    const int blocks = (int)std::min<long long>((total + 255) / 256, 65536);
    if (precision == SCFF_BF16X3)
        hipLaunchKernelGGL(fft_pack_kernel<true>, dim3(blocks), dim3(256), 0, st, T, cnorm, nbf, ns, RB, spin, (uint4*)Ap,
                           ar);
    else
        hipLaunchKernelGGL(fft_pack_kernel<false>, dim3(blocks), dim3(256), 0, st, T, cnorm, nbf, ns, RB, spin,
                           (uint4*)Ap, ar);
    return hipGetLastError();
}

// Waves per workgroup: four; eight in FP32 precision for tiles of 16 and 32 points,
// whose registers allow four waves per SIMD where the LDS holds two workgroups (380
// functions, 12 states, 64^3: 3.87 -> 2.74 ms a call; 265 functions 1.85 -> 1.53).
static int fft_density_nw(bool bf, int cb) { return bf || cb == 4 ? 4 : 8; }

int fft_density_cb(int precision, int nbf_pad, size_t lds_limit) {
    // the widest tile whose block lets two workgroups stay on a CU (split-BF16: within
    // 64 KiB); 16-point tiles up to the device limit for the largest bases.  FP32
    // precision, 190 functions, 12 states, 128^3: 64 points 6.4 ms, 32 points 7.0
    const bool bf = precision == SCFF_BF16X3;
    for (int cb : {4, 2})
        if (fft_lds_bytes(bf, nbf_pad, cb, fft_density_nw(bf, cb)) <= std::min<size_t>(lds_limit, bf ? 64u << 10 : 80u << 10))
            return cb;
    return fft_lds_bytes(bf, nbf_pad, 1, fft_density_nw(bf, 1)) <= lds_limit ? 1 : 0;
}

hipError_t launch_fft_density(int precision, const FftMol& m, const void* Ap, int nbf_pad, int ns, const int n[3],
                              const double x0[3], const double h[3], float* Z, float* phi, double* psum,
                              size_t lds_limit, long long* n_part, hipStream_t st) {
    const long long npts = (long long)n[0] * n[1] * n[2];
    const int cb = fft_density_cb(precision, nbf_pad, lds_limit);
    if (cb == 0 || nbf_pad % 16) return hipErrorInvalidValue;
    const FftPack p = fft_pack_layout(precision, nbf_pad, ns);
    const uint2* ar = (const uint2*)((const char*)Ap + p.ar);
    const bool bf = precision == SCFF_BF16X3;
    const int nw = fft_density_nw(bf, cb);
    const size_t lds = fft_lds_bytes(bf, nbf_pad, cb, nw);
    const long long tiles = (npts + 16 * cb - 1) / (16 * cb);
    if (tiles > 0x7fffffffLL) return hipErrorInvalidValue;
    *n_part = tiles;
    const int3 nn = make_int3(n[0], n[1], n[2]);
    const double3 xx = make_double3(x0[0], x0[1], x0[2]), hh = make_double3(h[0], h[1], h[2]);
    const auto launch = [&](auto kernel) {
        if (lds > 65536) {   // dynamic LDS beyond 64 KiB per workgroup must be allowed explicitly
            const hipError_t e =
                hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            if (e != hipSuccess) return e;
        }
        hipLaunchKernelGGL(kernel, dim3((unsigned)tiles), dim3(64 * nw), lds, st, m, (const uint4*)Ap, ar, nbf_pad, ns,
                           nbf_pad / 16, nn, xx, hh, npts, Z, phi, psum);
        return hipGetLastError();
    };
    if (bf)
        return cb == 4   ? launch(fft_density_kernel<true, 4, 4, 3>)
               : cb == 2 ? launch(fft_density_kernel<true, 2, 4, 3>)
                         : launch(fft_density_kernel<true, 1, 4, 3>);
    if (cb == 4)   // three workgroups per CU, or two
        return 3 * lds <= (160u << 10) ? launch(fft_density_kernel<false, 4, 4, 3>)
                                       : launch(fft_density_kernel<false, 4, 4, 2>);
    return cb == 2 ? launch(fft_density_kernel<false, 2, 8, 4>) : launch(fft_density_kernel<false, 1, 8, 4>);
}

hipError_t launch_fft_lines(float2* Z, int nb, const int n[3], hipStream_t st) {
    const int3 nn = make_int3(n[0], n[1], n[2]);
    for (int axis = 2; axis >= 0; --axis) {
        const int N = n[axis];
        if (N < 2) continue;
        long long lines;
        int M;
        long long groups;
        if (axis == 2) {
            lines = (long long)nb * n[0] * n[1];
            M = std::max(1, 4096 / N);
            groups = (lines + M - 1) / M;
        } else {
            M = std::min(std::min(16, n[2]), std::max(1, 4096 / N));
            lines = (long long)nb * n[0] * n[1] * n[2] / N;
            groups = lines / M;
        }
        if (groups > 0x7fffffffLL) return hipErrorInvalidValue;
        const size_t lds = ((size_t)M * N + N / 2) * sizeof(float2);
        hipLaunchKernelGGL(fft_lines_kernel, dim3((unsigned)groups), dim3(256), lds, st, Z, axis, nn, nb, M, lines);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_fft_finish(const float2* Z, const int n[3], int ns, double vpix, const double u[3], float2* f,
                             float* f2, double* psum, long long* n_part, hipStream_t st) {
    const long long npts = (long long)n[0] * n[1] * n[2];
    const long long blocks = (npts + 255) / 256;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    *n_part = (npts + 63) / 64;
    hipLaunchKernelGGL(fft_finish_kernel, dim3((unsigned)blocks), dim3(256), 0, st, Z, make_int3(n[0], n[1], n[2]),
                       ns, vpix, make_double3(u[0], u[1], u[2]), npts, f, f2, psum);
    return hipGetLastError();
}

hipError_t launch_fft_sum(const double* part, int ns, long long n, double scale, double* out, int stride,
                          hipStream_t st) {
    hipLaunchKernelGGL(fft_sum_kernel, dim3(ns), dim3(256), 0, st, part, n, scale, out, stride);
    return hipGetLastError();
}

}  // namespace scff
