// Device kernels of the Cartesian form-factor engine (gfx950 / CDNA4).
//
// Hot path (paper Sec. 4 eq. CartesianMethod, Sec. 5.3):
//
//   f_s(qx,qy,qz) = sum_k Tp(s,k) G(k,q),
//   G(k,q)        = sum_{t in terms(k)} Vx_t(qx) Vy_t(qy) Vz_t(qz),
//
// where k runs over unique component pairs (mu <= nu), t over their kept
// primitive-pair terms, and V_t^a are the 1D V-tensors of eq.
// CartesianVector in monomial form (eq. Ccoefficients).
//
//  * vtable_kernel: the 1D tables V[row][n] for every grid value of each
//    axis.  They are evaluated in FP64 (phase q*P with range reduction,
//    Gaussian, polynomial) and rounded once to FP32: the polynomial can
//    cancel, and FP32 evaluation would leave errors proportional to its bound
//    rather than to its value.  Exported only; the grid kernel reads
//    tables_kernel's layouts of the same values.
//  * grid_kernel: the sum contracted over z rows on the matrix cores (FP32
//    accumulation; FP32 precision: three BF16 parts per operand, folded into
//    FP64 totals; split precision: two f16 halves, or BF16 parts); the operand is
//    formed on the VALU.  grid_batch_kernel: the same tiles popped
//    from a queue of several requests.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstdint>
#include <type_traits>

#include "engine.h"
#include "vrow.h"

namespace scff {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef unsigned int uintx4 __attribute__((ext_vector_type(4)));
typedef _Float16 halfx2 __attribute__((ext_vector_type(2)));
typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// ---------------------------------------------------------------- 1D tables

__device__ __forceinline__ float2 eval_row(const VRowDev& r, double q) {
    const double2 v = eval_row_fp64(r, q);
    return make_float2((float)v.x, (float)v.y);
}

__global__ void vtable_kernel(const VRowDev* __restrict__ rows, int nrows, int vstride,
                              int3 n, double3 qmin, double3 dq, float2* __restrict__ V) {
    const long long tot = (long long)nrows * vstride;
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < tot;
         i += (long long)gridDim.x * blockDim.x) {
        const int r = (int)(i / vstride);
        const int j = (int)(i - (long long)r * vstride);
        const VRowDev row = rows[r];
        const int ax = row.axis;
        const int na = ax == 0 ? n.x : (ax == 1 ? n.y : n.z);
        if (j >= na) {
            V[i] = make_float2(0.f, 0.f);
            continue;
        }
        const double q0 = ax == 0 ? qmin.x : (ax == 1 ? qmin.y : qmin.z);
        const double d = ax == 0 ? dq.x : (ax == 1 ? dq.y : dq.z);
        V[i] = eval_row(row, q0 + d * (double)j);
    }
}

// The tables of the grid kernel's line axes, "x" and "y".  x: value-major
// V[qx][row], so that the rows of neighbouring terms (which neighbour each other)
// share cache lines; y: blocks of 8 values, V[qy / 8][row][8], so that a tile's
// lines read whole 64-byte runs.  Table row r is the zero row rows[0] or
// rows[seg + r]; nxr and nyr count the zero row too.
__device__ __forceinline__ void xytable(const VRowDev* __restrict__ rows, int nxr, int nyr, int2 seg, int nx, int ny, double2 qmin,
                                        double2 dq, float2* __restrict__ X, float2* __restrict__ Y, long long i0,
                                        long long step) {
    const long long tx = (long long)nx * nxr, tot = tx + (long long)((ny + 7) & ~7) * nyr;
    for (long long i = i0; i < tot; i += step) {
        if (i < tx) {
            const int q = (int)(i / nxr), r = (int)(i - (long long)q * nxr);
            X[i] = eval_row(rows[r ? seg.x + r : 0], qmin.x + dq.x * (double)q);
        } else {
            const long long o = i - tx;
            const int v = (int)(o & 7);
            const long long br = o >> 3;
            const int b = (int)(br / nyr), r = (int)(br - (long long)b * nyr), q = 8 * b + v;
            Y[o] = q < ny ? eval_row(rows[r ? seg.y + r : 0], qmin.y + dq.y * (double)q) : make_float2(0.f, 0.f);
        }
    }
}

// V block of the contracted axis in the grid kernel's operand order: fragment
// ((k-step * ncg + column group) * planes + plane) of 64 lanes x 16 bytes, lane
// (g, n) = z rows 8 g .. 8 g + 7 of the k-step at column n, planes re then im,
// each part of the row (scaled by its power of two) in turn: three BF16 parts
// (FP32 precision) or two f16 halves, every part the FP64 value's rest rounded
// to nearest.  One thread per (8 z rows, column).
template <typename H, int PARTS>
__device__ __forceinline__ void ztable(const VRowDev* __restrict__ rows, const int2* __restrict__ zslots, int n_oct,
                                       int ncg, int ncol, int iz0, double qmin, double dq, uint4* __restrict__ Bt,
                                       long long i0, long long step) {
    typedef H hx8 __attribute__((ext_vector_type(8)));
    const long long tot = (long long)n_oct * ncg * 16;
    for (long long i = i0; i < tot; i += step) {
        const int oct = (int)(i / (ncg * 16)), col = (int)(i - (long long)oct * ncg * 16);
        hx8 pl[2 * PARTS];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            double2 v = make_double2(0.0, 0.0);
            if (col < ncol) {
                const int2 zs = zslots[oct * 8 + j];
                v = eval_row_fp64(rows[zs.x], qmin + dq * (double)(iz0 + col));
                v.x = ldexp(v.x, zs.y);
                v.y = ldexp(v.y, zs.y);
            }
#pragma unroll
            for (int p = 0; p < PARTS; ++p) {
                const H re = (H)(float)v.x, im = (H)(float)v.y;
                pl[p][j] = re;
                pl[PARTS + p][j] = im;
                v.x -= (double)(float)re;
                v.y -= (double)(float)im;
            }
        }
        uint4* o = Bt + (((size_t)(oct >> 2) * ncg + (col >> 4)) * (2 * PARTS)) * 64 + (oct & 3) * 16 + (col & 15);
#pragma unroll
        for (int p = 0; p < 2 * PARTS; ++p) o[p * 64] = __builtin_bit_cast(uint4, pl[p]);
    }
}

// All of them in one launch: the contracted axis' blocks (eight values per
// thread, the longest) first.  nx, ny and the members of qmin and dq: line axes
// 0 and 1, contracted axis.
template <typename H, int PARTS>
__global__ __launch_bounds__(256) void tables_kernel(const VRowDev* __restrict__ rows, int nxr, int nyr, int2 seg, int nx,
                                                     int ny, double3 qmin, double3 dq, float2* __restrict__ X,
                                                     float2* __restrict__ Y, const int2* __restrict__ zslots, int n_oct,
                                                     int ncg, int ncol, int iz0, uint4* __restrict__ Bt, int nbz) {
    if ((int)blockIdx.x < nbz)
        ztable<H, PARTS>(rows, zslots, n_oct, ncg, ncol, iz0, qmin.z, dq.z, Bt, blockIdx.x * 256LL + threadIdx.x,
                         nbz * 256LL);
    else
        xytable(rows, nxr, nyr, seg, nx, ny, make_double2(qmin.x, qmin.y), make_double2(dq.x, dq.y), X, Y,
                (blockIdx.x - nbz) * 256LL + threadIdx.x, (gridDim.x - nbz) * 256LL);
}

// ---------------------------------------------------------------- grid kernel
//
// The pair sum is contracted in the order
//   U_s(z, line) = sum_{t with z row z} T'_s(t) Vx_t(qx) Vy_t(qy)     (VALU)
//   f_s(line, qz) = sum_z U_s(z, line) Vz(z, qz)                      (matrix cores)
// z runs over the distinct 1D rows of the z axis (one per primitive pair and
// power pair; about half as many as terms), line over the (qx, qy) pairs.  "z" is
// the contracted axis, of the three the one of the least cost (choose_axis,
// runtime.cpp), "x" and "y" the other two.
// The second sum is a real matrix product of [Re U; Im U] (rows: state, line)
// with [Re V | Im V] (columns: qz), K = z rows, whose four blocks
//   P = Ur Vr, Q = Ui Vi, R = Ur Vi, S = Ui Vr
// give f = (P - Q) + i (R + S).  V(-q) = V(q)* for every 1D row, so on an axis
// with qmin_z = -qmax_z the columns are the upper half of the axis only and
// the mirror value is (P + Q) + i (S - R): the same products serve both.  On other
// axes P - Q and R + S are the sums (half the registers per column, so that a tile
// may be twice as wide and U is formed once for up to 96 columns): 30 heavy atoms,
// 24 states, 96^3 off centre on every axis 110 -> 88 ms in FP32 precision, 62 -> 46
// in split precision, where the kernel by pairs took 100 and 50.
//
// FOLD (FP32 precision): U and V as three BF16 parts each, which hold FP32's 24
// bits over FP32's whole exponent range, and the six products above 2^-24 of the
// whole; the FP32 sums of two k-steps go to FP64 totals (the sum over z cancels).
// Split precision: f16 halves hi + lo (22 significant bits and more), hi hi + hi
// lo + lo hi, FP32 sums throughout; where a half's range is too short for the
// grid (grid_kind, runtime.cpp), the BF16 parts without totals.  Exact powers of two bring V's rows to |V| <
// 2^14 and U to |U| < 2^15 (prep.hip, from q-independent bounds), so the f16
// halves keep their bits and nothing overflows; the epilogue removes them.
//
// FP32 precision on f16 halves as well took 37.6 ms where the BF16 parts take 54.3
// (30 heavy atoms, 24 states, 96^3; 10 heavy atoms, 12 states, 64^3: 1.63 and
// 2.10), but an f16 half ends at 2^-24: in the tail of a diffuse basis, where
// every value of U and V lies far below its bound, nothing was left (relative
// error 4e-4 where |f| is 3e-15 of the peak; 2e-7 down to 1e-33 now).
//
// A workgroup is 4 waves; its tile 64 rows (row = line * states + state, lines
// padded to pairs per qx) by 16 CG columns.  Each wave forms its own 16 rows'
// operand: lane (g, m) holds U of row m for the z rows 8 g .. 8 g + 7 of a k-step
// of 32, i.e. exactly its share of a 16x16x32 A operand, so U goes from registers
// to the matrix cores.  The products W = Vx Vy, which the states of a line
// share, are formed once per workgroup, two lines per gather (a pair's y values
// are 16 adjacent bytes), and pass through LDS; the V block of a k-step (stored
// in operand order by tables_kernel) and the weights come to LDS by DMA.  All of
// it goes out one step (one or two terms of a k-step) ahead, one barrier a step.
//
// Why: the kernel before formed G = sum_t Vx Vy Vz per (pair, q) on the VALU (4
// FMAs per term and q) and contracted with FP32 matrix instructions; here the
// VALU's part does not depend on the number of columns.  It pays where there are
// more columns than about two thirds of the states: with 24 states and 48 columns
// off centre it is 0.8 to 0.9 of the kernel before, the worst case.  A version whose
// waves formed W each for itself was bound by its gathers (64 cache lines per
// instruction): 46.8 ms on a 30-heavy-atom molecule with 24 states on 96^3; sharing
// W: 40.2 ms (both with f16 halves).  What bounds it now: the products.  96^3 with 24
// states issues 3.6e9 matrix instructions in FP32 precision and half of that in split
// precision, 52 and 26 ms at the rate that a large BF16 product reaches on this card
// (1130 TFLOP/s), of 57 to 61 and 31 to 32 ms.  The operand's LDS reads do not:
// broadcasting W between lanes by DPP instead of reading it per lane was 3 to 15 %
// slower (FP32 55.9 -> 59.9 ms).  Three waves per SIMD at CG = 2 with totals and mirror
// values spill (2.05 -> 2.47 ms).

constexpr int kGridWaves = 4;
// Waves per SIMD, by the registers of the sums: 48 per column group with FP64 totals
// (four sums), 24 without the mirror values (two sums), a third of both without totals.
constexpr int grid_waves(int cg, bool fold, bool refl) { return fold && cg * (refl ? 2 : 1) > 2 ? 2 : 3; }
// Buffers of V blocks: tiles of four groups and more have one, so that two or three
// workgroups fit a CU's LDS (96 columns off centre, 24 states: the other workgroups
// cover the wait).
constexpr int grid_vbufs(int cg, bool refl) { return refl || cg < 4 ? 2 : 1; }
// k-steps per FP64 fold.  Two sums take twice the products each, so they are folded
// twice as often (at the same cost per product).
constexpr int fold_steps(bool refl) { return refl ? 2 : 1; }

typedef __attribute__((address_space(3))) void lds_void_t;

template <typename T>
__device__ __forceinline__ uint32_t lds_addr(T* p) { return (uint32_t)(uintptr_t)(lds_void_t*)p; }

// 16 bytes per lane from sbase + voff (sbase wave-uniform, voff per lane) to
// LDS at lds_byte + 16 * lane (lds_byte wave-uniform).  Issued as inline
// assembly so that the compiler does not treat every later LDS read as a
// possible alias of the in-flight copy (it would then wait for all outstanding
// vector-memory operations before each of them); completion is awaited
// explicitly by barrier_dma.
__device__ __forceinline__ void dma_b128(uint32_t voff, const void* sbase, uint32_t lds_byte) {
    const uint32_t m0 = __builtin_amdgcn_readfirstlane(lds_byte);
    // the base is wave-uniform; say so, so that it lives in scalar registers
    // also where it was loaded from memory (the batch kernel's descriptors)
    // (readfirstlane returns a signed int: each half is widened through
    // uint32_t, never sign-extended into the other half)
    const uint64_t b = (uint64_t)(uintptr_t)sbase;
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)b);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
    const uint64_t bu = ((uint64_t)hi << 32) | (uint64_t)lo;
    // s_nop 4: five wait states between a VALU write of the base or M0
    // (v_readfirstlane) and their read by the VMEM instruction, which the
    // compiler cannot see inside the asm; also covers the M0 write (one)
    asm volatile("s_nop 4\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(bu), "{m0}"(m0) : "memory");
}


// Barrier with this wave's LDS accesses and DMA into LDS complete.  The wait
// is the compiler's own s_waitcnt (vmcnt(0) lgkmcnt(0)), so it knows that
// every earlier vector-memory load is complete here.
__device__ __forceinline__ void barrier_dma() {
    __builtin_amdgcn_s_waitcnt(0x0070);
    asm volatile("s_barrier" ::: "memory");
}

// Split of two FP32 values into f16 halves: hi = RNE(v), lo = RNE(v - hi)
// (v - hi is exact in FP32), two values per dword.  The mixed-precision FMA
// forms v - hi in one instruction without unpacking hi.
__device__ __forceinline__ void split_f16(float v0, float v1, uint32_t& hi, uint32_t& lo) {
    const uint32_t h = __builtin_bit_cast(uint32_t, __builtin_convertvector(floatx2{v0, v1}, halfx2));
    float r0, r1;
    asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel_hi:[1,0,0]" : "=v"(r0) : "v"(h), "v"(v0));
    asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(r1) : "v"(h), "v"(v1));
    hi = h;
    lo = __builtin_bit_cast(uint32_t, __builtin_convertvector(floatx2{r0, r1}, halfx2));
}

// Split of two FP32 values into three BF16 parts, each the rest rounded to
// nearest: 24 bits, so the sum of the parts is the value (parts below the BF16
// subnormals aside).  A BF16 dot product with (-1, -0) or (-0, -1) forms a rest
// in one instruction without unpacking the part (-0, not +0: (-1, +0) would be
// sent as the inline constant -1.0, which the instruction reads as (+0, -1)).
__device__ __forceinline__ void split_bf16(float v0, float v1, uint32_t (&part)[3]) {
    const bf16x2 first{(__bf16)-1.0f, (__bf16)-0.0f}, second{(__bf16)-0.0f, (__bf16)-1.0f};
#pragma unroll
    for (int p = 0; p < 3; ++p) {
        const bf16x2 h = __builtin_convertvector(floatx2{v0, v1}, bf16x2);
        part[p] = __builtin_bit_cast(uint32_t, h);
        if (p < 2) {
            v0 = __builtin_amdgcn_fdot2_f32_bf16(h, first, v0, false);
            v1 = __builtin_amdgcn_fdot2_f32_bf16(h, second, v1, false);
        }
    }
}

// Operand parts, planes of a V block (re and im of every part) and, smallest
// products first, the parts of U and V that are multiplied.
template <bool BF>
struct Operands {   // three BF16 parts; left out: products below 2^-24 of the whole
    typedef bf16x8 frag;
    static constexpr int parts = 3, planes = 6, products = 6;
    static constexpr int u[products] = {1, 0, 2, 0, 1, 0}, v[products] = {1, 2, 0, 1, 0, 0};
};
template <>
struct Operands<false> {   // f16 halves
    typedef halfx8 frag;
    static constexpr int parts = 2, planes = 4, products = 3;
    static constexpr int u[products] = {1, 0, 0}, v[products] = {0, 1, 0};
};
__device__ __forceinline__ floatx4 mma(bf16x8 a, bf16x8 b, floatx4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ floatx4 mma(halfx8 a, halfx8 b, floatx4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}

// One tile of one evaluation (blk = (split * row tiles + row tile) * column
// tiles + column tile).  Shared by the single-request kernel (one tile per
// workgroup) and the persistent batch kernel (tiles of several requests popped
// from a queue), so a tile's values do not depend on which of the two computed
// it; nor do they depend on the tile a row falls into.
//
// LDS (floats): V blocks [1 or 2][CG planes 256], weights [2][tcm 48 ns],
// W [2][tcm][2 np lines][kWLine].
template <int CG, bool FOLD, bool BF, bool REFL>
__device__ __forceinline__ void grid_tile(const GridDesc& d, int blk, float* lds) {
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, m = lane & 15;
    const int ns = d.n_states, tcm = d.tcm;           // tcm: 1 or 2
    using Op = Operands<BF>;
    using frag = typename Op::frag;
    constexpr int PL = Op::planes, BW = CG * PL * 256;   // floats of a V block
    const int TW = tcm * 48 * ns;                     // floats of a weight buffer
    const int WT = 2 * d.np * kWLine;                 // floats of W, one term
    constexpr int VB = grid_vbufs(CG, REFL);
    float* const Tl = lds + VB * BW;
    float* const Wl = Tl + 2 * TW;

    const int ct = blk % d.ntc;
    const int bl = blk / d.ntc;
    const int split = bl / d.ntl, lt = bl - split * d.ntl;
    const int k_lo = d.sp.lo[split], k_hi = d.sp.lo[split + 1];

    // the tile's line pairs; the lane's row (clamped into the problem)
    const int nlines = d.n1 * d.nyp, nrows = nlines * ns;
    const int row0 = lt * kGridWaves * 16;
    const int pair0 = row0 / ns >> 1;
    const int npair = (min(row0 + kGridWaves * 16, nrows) - 1) / ns / 2 - pair0 + 1;
    const int row = min(row0 + 16 * wave + m, nrows - 1);
    const int line = row / ns, st = row - line * ns;
    const float* const tl = Tl + (g * ns + st) * 12;
    const float* const wl = Wl + (line - 2 * pair0) * kWLine + g * 20;

    // W items: (pair, term, z row); a lane's term and z row are fixed, its pairs
    // come ppass apart
    const int lt2 = tcm == 2 ? 6 : 5;
    const int wz = tid & 31, wt = (tid & ((1 << lt2) - 1)) >> 5, wp = tid >> lt2, ppass = kGridWaves * 64 >> lt2;
    auto offsets = [&](int pair, uint32_t& ox, uint32_t& oy) {
        const int l = 2 * (pair0 + min(pair, npair - 1));
        const int qx = l / d.nyp, qy = l - qx * d.nyp;
        ox = 8u * (uint32_t)qx * (uint32_t)d.nxr;
        oy = d.ybase + 64u * (uint32_t)(qy >> 3) * (uint32_t)d.nyr + 8u * (uint32_t)(qy & 7);
    };
    uint32_t ox[kWPasses], oy[kWPasses];
#pragma unroll
    for (int i = 0; i < kWPasses; ++i) offsets(wp + i * ppass, ox[i], oy[i]);
    const char* const Vb = reinterpret_cast<const char*>(d.V);
    float* const wst = Wl + wt * WT + 2 * wp * kWLine + (wz >> 3) * 20 + (wz & 7) * 2;

    // a step: terms t0 .. t0 + tc - 1 of the n terms of k-step k, which start at c
    // (in terms per z row); the k-steps before kn have n terms
    struct Pos {
        int k, t0, n, c, kn;
    };
    auto next = [&](const Pos& p) {   // past the last k-step: stays on its last step
        Pos q = p;
        if (p.t0 + tcm < p.n) {
            q.t0 += tcm;
        } else if (p.k + 1 < k_hi) {
            q.c += p.n;
            q.t0 = 0;
            ++q.k;
            while (q.k >= q.kn) q.kn = d.steps.kend[--q.n];
        }
        return q;
    };
    auto terms_of = [&](const Pos& p) { return min(tcm, p.n - p.t0); };
    auto dma_w = [&](const Pos& p, int buf) {
        const float* src = d.Tw + (size_t)(p.c + p.t0) * (size_t)(48 * ns);
        const uint32_t dst = lds_addr(Tl + buf * TW);
        const int units = terms_of(p) * 12 * ns;   // 16 bytes each
        for (int u = 64 * wave; u < units; u += 64 * kGridWaves)
            if (u + lane < units) dma_b128(16u * (u + lane), src, dst + 16u * u);
    };
    auto dma_v = [&](int k) {
        const uint4* src = d.Bt + ((size_t)k * d.ncg + ct * CG) * (64 * PL);
        const uint32_t dst = lds_addr(lds + (k & (VB - 1)) * BW);
#pragma unroll
        for (int i = 0; i < CG * PL; i += kGridWaves)   // a wave copies a plane of 1 KB at a time
            if (CG * PL % kGridWaves == 0 || i + wave < CG * PL)
                dma_b128(16u * (64 * (i + wave) + lane), src, dst + 1024u * (i + wave));
    };
    // term record (x row, y row) of the lane's item
    auto load_rec = [&](const Pos& p) { return d.terms[(p.c + p.t0 + min(wt, terms_of(p) - 1)) * 32 + wz]; };
    auto load_xy = [&](int2 rec, uint32_t px, uint32_t py, float2& x, float4& y) {
        x = *reinterpret_cast<const float2*>(Vb + (size_t)(px + 8u * (uint32_t)rec.x));
        y = *reinterpret_cast<const float4*>(Vb + (size_t)(py + 64u * (uint32_t)rec.y));
    };
    float2 vx[kWPasses];
    float4 vy[kWPasses];
    auto gather = [&](int tc, int2 rec) {
#pragma unroll
        for (int i = 0; i < kWPasses; ++i)
            if (wt < tc && wp + i * ppass < npair) load_xy(rec, ox[i], oy[i], vx[i], vy[i]);
    };
    auto put_w = [&](float2 x, float4 y, float* dst) {   // the pair's two lines
        *reinterpret_cast<float2*>(dst) = make_float2(fmaf(-x.y, y.y, x.x * y.x), fmaf(x.y, y.x, x.x * y.y));
        *reinterpret_cast<float2*>(dst + kWLine) =
            make_float2(fmaf(-x.y, y.w, x.x * y.z), fmaf(x.y, y.z, x.x * y.w));
    };
    auto write_w = [&](int tc, int2 rec, int buf) {
        float* const w = wst + buf * tcm * WT;
#pragma unroll
        for (int i = 0; i < kWPasses; ++i)
            if (wt < tc && wp + i * ppass < npair) put_w(vx[i], vy[i], w + i * 2 * ppass * kWLine);
        for (int p = wp + kWPasses * ppass; p < npair; p += ppass) {   // tiles of many lines (few states)
            if (wt >= tc) break;
            uint32_t px, py;
            offsets(p, px, py);
            float2 x;
            float4 y;
            load_xy(rec, px, py, x, y);
            put_w(x, y, w + 2 * (p - wp) * kWLine);
        }
    };

    // sums of a column group: [2 a + b] of part a of U (re, im) and b of V, or
    // (where no mirror value is wanted) the real and the imaginary part of f
    constexpr int NS = REFL ? 4 : 2;
    floatx4 acc[CG][NS];
    double tot[FOLD ? CG : 1][NS][4];
#pragma unroll
    for (int q = 0; q < CG; ++q)
#pragma unroll
        for (int a = 0; a < NS; ++a) {
            acc[q][a] = floatx4{0.f, 0.f, 0.f, 0.f};
            if constexpr (FOLD)
#pragma unroll
                for (int i = 0; i < 4; ++i) tot[q][a][i] = 0.0;
        }
    float ur[8], ui[8];

    if (k_hi > k_lo) {
        const int n0 = ksteps_terms(d.steps, k_lo);
        Pos p0{k_lo, 0, n0, ksteps_first(d.steps, k_lo), d.steps.kend[n0]}, p1 = next(p0);
        if constexpr (VB == 2) dma_v(k_lo);
        dma_w(p0, 0);
        int2 rec = load_rec(p0);
        gather(terms_of(p0), rec);
        write_w(terms_of(p0), rec, 0);
        rec = load_rec(p1);
        barrier_dma();
        for (int i = 0;; i ^= 1) {
            const int tc = terms_of(p0), tc1 = terms_of(p1);
            const bool last_term = p0.t0 + tc >= p0.n, last = last_term && p0.k + 1 >= k_hi;
            const Pos p2 = next(p1);
            int2 rec2 = rec;
            // the next step's loads and copies go out first
            if constexpr (VB == 1)
                if (p0.t0 == 0) dma_v(p0.k);
            if (!last) {
                gather(tc1, rec);
                rec2 = load_rec(p2);
                dma_w(p1, i ^ 1);
                if (VB == 2 && last_term) dma_v(p1.k);
            }
            // U of the lane's row: eight z rows
            auto add = [&](int t, bool first) {
                const float* T = tl + i * TW + t * 48 * ns;
                const float* w = wl + (i * tcm + t) * WT;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const floatx4 tv = *reinterpret_cast<const floatx4*>(T + 4 * h);
                    const floatx4 ab[2] = {*reinterpret_cast<const floatx4*>(w + 8 * h),
                                           *reinterpret_cast<const floatx4*>(w + 8 * h + 4)};
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const float wr = ab[j >> 1][2 * (j & 1)], wi = ab[j >> 1][2 * (j & 1) + 1];
                        ur[4 * h + j] = first ? tv[j] * wr : fmaf(tv[j], wr, ur[4 * h + j]);
                        ui[4 * h + j] = first ? tv[j] * wi : fmaf(tv[j], wi, ui[4 * h + j]);
                    }
                }
            };
            // vector work beside another wave's matrix instructions issues at half its
            // rate, while they keep theirs: priority from here to the products (96^3,
            // 24 states, FP32 41.8 -> 40.0 ms per call, 64^3, 12 states 1.93 -> 1.89; with
            // the fold or the loads and W included it is slower or the same)
            __builtin_amdgcn_s_setprio(1);
            if (p0.t0 == 0) add(0, true);
            else add(0, false);
            if (tc > 1) add(1, false);
            if (last_term) {
                frag A[2][Op::parts];   // [re/im][part]
#pragma unroll
                for (int a = 0; a < 2; ++a) {
                    const float(&u)[8] = a ? ui : ur;
                    uintx4 w[Op::parts];
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        uint32_t t[Op::parts];
                        if constexpr (BF) split_bf16(u[2 * j], u[2 * j + 1], t);
                        else split_f16(u[2 * j], u[2 * j + 1], t[0], t[1]);
#pragma unroll
                        for (int p = 0; p < Op::parts; ++p) w[p][j] = t[p];
                    }
#pragma unroll
                    for (int p = 0; p < Op::parts; ++p) A[a][p] = __builtin_bit_cast(frag, w[p]);
                }
                frag M[Op::parts];   // -im
                if constexpr (!REFL)
#pragma unroll
                    for (int p = 0; p < Op::parts; ++p)
                        M[p] = __builtin_bit_cast(frag, __builtin_bit_cast(uintx4, A[1][p]) ^ 0x80008000u);
                const uint4* B = reinterpret_cast<const uint4*>(lds + (p0.k & (VB - 1)) * BW) + lane;
                __builtin_amdgcn_s_setprio(0);
                // one V block: it was asked for in this step where the k-step has no other
                if constexpr (VB == 1)
                    if (p0.t0 == 0) barrier_dma();
#pragma unroll
                for (int q = 0; q < CG; ++q) {
                    frag V[2][Op::parts];
#pragma unroll
                    for (int b = 0; b < PL; ++b)
                        V[b / Op::parts][b % Op::parts] = __builtin_bit_cast(frag, B[(q * PL + b) * 64]);
#pragma unroll
                    for (int pr = 0; pr < Op::products; ++pr) {
                        const int u = Op::u[pr], v = Op::v[pr];
                        if constexpr (REFL) {
#pragma unroll
                            for (int a = 0; a < 2; ++a)
#pragma unroll
                                for (int b = 0; b < 2; ++b) acc[q][2 * a + b] = mma(A[a][u], V[b][v], acc[q][2 * a + b]);
                        } else {
                            acc[q][0] = mma(A[0][u], V[0][v], acc[q][0]);
                            acc[q][1] = mma(A[0][u], V[1][v], acc[q][1]);
                            acc[q][0] = mma(M[u], V[1][v], acc[q][0]);
                            acc[q][1] = mma(A[1][u], V[0][v], acc[q][1]);
                        }
                    }
                }
                if (FOLD && ((p0.k - k_lo) % fold_steps(REFL) == fold_steps(REFL) - 1 || last)) {
#pragma unroll
                    for (int q = 0; q < (FOLD ? CG : 0); ++q)
#pragma unroll
                        for (int a = 0; a < NS; ++a) {
#pragma unroll
                            for (int e = 0; e < 4; ++e) tot[q][a][e] += (double)acc[q][a][e];
                            acc[q][a] = floatx4{0.f, 0.f, 0.f, 0.f};
                        }
                }
            }
            if (last) break;
            write_w(tc1, rec, i ^ 1);
            barrier_dma();
            p0 = p1;
            p1 = p2;
            rec = rec2;
        }
    }

    // epilogue: lane (g, m) holds rows 4 g + i, column m of its quads
    const int rw = row0 + 16 * wave + 4 * g;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int ln = (rw + i) / ns, s = rw + i - ln * ns;
        const int qx = ln / d.nyp, qy = ln - qx * d.nyp;
        if (rw + i >= nrows || qy >= d.nl) continue;
        const double sc = d.sinv[s];
        const size_t base = (size_t)s * d.npts + (size_t)qx * d.sx + (size_t)qy * d.sy;
#pragma unroll
        for (int q = 0; q < CG; ++q) {
            const int col = (ct * CG + q) * 16 + m;
            if (col >= d.ncol) continue;
            double v[NS];
#pragma unroll
            for (int a = 0; a < NS; ++a) v[a] = sc * (FOLD ? tot[FOLD ? q : 0][a][i] : (double)acc[q][a][i]);
            auto put = [&](int iz, double re, double im) {
                const size_t o = base + (size_t)iz * d.sz;
                if (d.partial) {   // split pair sum: FP64 partial, summed by reduce_kernel
                    d.partial[(size_t)split * d.part_stride + o] = make_double2(re, im);
                } else {
                    if (d.f) d.f[o] = make_float2((float)re, (float)im);
                    if (d.f2) d.f2[o] = (float)(re * re + im * im);
                }
            };
            if constexpr (REFL) {
                const int iz = d.iz0 + col, im = d.nc - 1 - iz;
                put(iz, v[0] - v[3], v[1] + v[2]);
                if (im != iz) put(im, v[0] + v[3], v[2] - v[1]);
            } else {
                put(col, v[0], v[1]);
            }
        }
    }
}

#define SCFF_GRID_BOUNDS                    \
    __launch_bounds__(kGridWaves * 64)      \
        __attribute__((amdgpu_waves_per_eu(grid_waves(CG, FOLD, REFL), grid_waves(CG, FOLD, REFL))))
template <int CG, bool FOLD, bool BF, bool REFL>
__global__ SCFF_GRID_BOUNDS void grid_kernel(GridDesc d) {
    extern __shared__ __align__(16) float grid_lds[];
    grid_tile<CG, FOLD, BF, REFL>(d, blockIdx.x, grid_lds);
}

// Persistent batch kernel: every workgroup pops (request, tile) items from a
// device queue (items[i] = (descriptor index, tile of that request's launch))
// through an atomic counter until the queue is exhausted, so the tiles of
// several requests share one launch.  Every workgroup leaves the loop once
// the counter passes n_items; the counter must be 0 at launch.  The launch's
// LDS holds the largest of its requests' needs after the 16 bytes of the queue.
template <int CG, bool FOLD, bool BF, bool REFL>
__global__ SCFF_GRID_BOUNDS void grid_batch_kernel(
    const GridDesc* __restrict__ descs, const int2* __restrict__ items, int n_items, int* __restrict__ counter) {
    extern __shared__ __align__(16) float grid_lds[];
    int* s_item = reinterpret_cast<int*>(grid_lds);
    for (;;) {
        __syncthreads();   // the previous tile's LDS use is over
        if (threadIdx.x == 0) s_item[0] = atomicAdd(counter, 1);
        __syncthreads();
        const int it = __builtin_amdgcn_readfirstlane(s_item[0]);
        if (it >= n_items) break;
        const int2 w = items[it];
        grid_tile<CG, FOLD, BF, REFL>(descs[w.x], w.y, grid_lds + 4);
    }
}

// Zeroes the batch queue counters (a kernel rather than a memset, so a
// captured graph replays it faithfully).
__global__ void zero_counters_kernel(int* __restrict__ c, int n) {
    if ((int)threadIdx.x < n) c[threadIdx.x] = 0;
}

// ---------------------------------------------------------------- split reduction
//
// Sum of the FP64 partial results of the k-step ranges (fixed order) for
// the evaluated planes ix < nx_eval, then f and |f|^2 as from the grid kernel.

__global__ void reduce_kernel(const double2* __restrict__ part, int n_split, long long stride, int3 n,
                              int nx_eval, int n_states, float2* __restrict__ f, float* __restrict__ f2) {
    const long long per_s = (long long)nx_eval * n.y * n.z;
    const long long tot = per_s * n_states;
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < tot;
         i += (long long)gridDim.x * blockDim.x) {
        const int s = (int)(i / per_s);
        long long r = i - (long long)s * per_s;
        const int iz = (int)(r % n.z);
        r /= n.z;
        const int iy = (int)(r % n.y);
        const int ix = (int)(r / n.y);
        const size_t o = (((size_t)s * n.x + ix) * n.y + iy) * n.z + iz;
        double re = 0.0, im = 0.0;
        for (int j = 0; j < n_split; ++j) {
            const double2 v = part[(size_t)j * stride + o];
            re += v.x;
            im += v.y;
        }
        if (f) f[o] = make_float2((float)re, (float)im);
        if (f2) f2[o] = (float)(re * re + im * im);
    }
}

// ---------------------------------------------------------------- mirror kernel
//
// For a real transition density the form factor obeys f(-q) = f(q)* (the
// integrand's phase e^{iq.r} is conjugated by q -> -q, everything else is
// real).  On a grid symmetric about q = 0 (q_min = -q_max on every axis) the
// point with indices (nx-1-ix, ny-1-iy, nz-1-iz) is -q of (ix, iy, iz), so
// the grid kernel need only evaluate the planes ix < nx_eval = ceil(nx/2) and this
// kernel writes the others as conjugates: f[s][ix][iy][iz] =
// conj(f[s][nx-1-ix][ny-1-iy][nz-1-iz]), |f|^2 copied.

__global__ void mirror_kernel(int3 n, int nx_eval, int n_states, float2* __restrict__ f, float* __restrict__ f2) {
    const long long per_s = (long long)(n.x - nx_eval) * n.y * n.z;
    const long long tot = per_s * n_states;
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < tot;
         i += (long long)gridDim.x * blockDim.x) {
        const int s = (int)(i / per_s);
        long long r = i - (long long)s * per_s;
        const int iz = (int)(r % n.z);
        r /= n.z;
        const int iy = (int)(r % n.y);
        const int ix = nx_eval + (int)(r / n.y);
        const size_t o = (((size_t)s * n.x + ix) * n.y + iy) * n.z + iz;
        const size_t m = (((size_t)s * n.x + (n.x - 1 - ix)) * n.y + (n.y - 1 - iy)) * n.z + (n.z - 1 - iz);
        if (f) {
            const float2 v = f[m];
            f[o] = make_float2(v.x, -v.y);
        }
        if (f2) f2[o] = f2[m];
    }
}

// ---------------------------------------------------------------- launchers

hipError_t launch_vtable(const VRowDev* rows, int nrows, int vstride, const int n[3],
                         const double qmin[3], const double dq[3], float2* V, hipStream_t st) {
    const long long tot = (long long)nrows * vstride;
    int blocks = (int)((tot + 255) / 256);
    if (blocks > 65536) blocks = 65536;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(vtable_kernel, dim3(blocks), dim3(256), 0, st, rows, nrows, vstride,
                       make_int3(n[0], n[1], n[2]), make_double3(qmin[0], qmin[1], qmin[2]),
                       make_double3(dq[0], dq[1], dq[2]), V);
    return hipGetLastError();
}

// Row stride of the x / y tables.
int vtable_stride(const int n[3]) {
    int m = n[0] > n[1] ? n[0] : n[1];
    m = m > n[2] ? m : n[2];
    return ((m + 15) / 16) * 16 + 16;
}

hipError_t launch_grid_tables(const PrepResult& p, const VRowDev* rows, const int2* zslots, const GridShape& g,
                              const int n[3], const double qmin[3], const double dq[3], float2* X, float2* Y, uint4* Bt,
                              hipStream_t st) {
    if (p.axis != g.axis) return hipErrorInvalidValue;
    const int n_oct = p.n_ksteps * (kZStep / 8);
    const int a = g.l[0], b = g.l[1], c = g.axis, nxr = p.n_axis[a] + 1, nyr = p.n_axis[b] + 1;
    const int2 seg = make_int2(p.seg(a), p.seg(b));
    const long long tz = (long long)n_oct * g.ncg * 16;
    const long long txy = (long long)n[a] * nxr + (long long)((n[b] + 7) & ~7) * nyr;
    const int nbz = (int)std::min<long long>((tz + 255) / 256, 32768);
    const int nbxy = (int)std::max<long long>(1, std::min<long long>((txy + 255) / 256, 32768));
    const double3 q0 = make_double3(qmin[a], qmin[b], qmin[c]), d = make_double3(dq[a], dq[b], dq[c]);
    if (g.planes == Operands<true>::planes)
        hipLaunchKernelGGL((tables_kernel<__bf16, Operands<true>::parts>), dim3(nbz + nbxy), dim3(256), 0, st, rows, nxr,
                           nyr, seg, n[a], n[b], q0, d, X, Y, zslots, n_oct, g.ncg, g.ncol, g.iz0, Bt, nbz);
    else
        hipLaunchKernelGGL((tables_kernel<_Float16, Operands<false>::parts>), dim3(nbz + nbxy), dim3(256), 0, st, rows, nxr,
                           nyr, seg, n[a], n[b], q0, d, X, Y, zslots, n_oct, g.ncg, g.ncol, g.iz0, Bt, nbz);
    return hipGetLastError();
}

// Tiling: column groups per tile (CG), chosen for the least time among those
// whose LDS fits.  A wave's k-step costs its products (and, in FP32, their
// fold) and forming U, which every column tile repeats: 30 + 31 CG in FP32
// precision, 30 + 10 CG and 30 + 22 CG in split precision on f16 halves and BF16
// parts (30 heavy atoms, 24 states, 96x96 lines, one and three column groups: 26.9
// and 54.3, 20.3 and 30.2, 26.1 and 48.2 ms).  Two terms per step where
// the LDS allows (one barrier for both), else one (one or two states: W has up to
// 64 lines).  With mirror values FP32 precision stops at three column groups: the totals of a fourth
// spill 34 registers of 256 (10 heavy atoms, 12 states, 128^3, whose 64 columns are
// then two tiles of two: 27.4 -> 21.6 ms; 48x48x256, 128 columns, three tiles of three:
// 8.9 -> 6.2 ms).  At most one group of padding: the z blocks then stay within
// rows x vtable_stride, by which a grid is accepted.
int max_cg(GridKind kind, bool refl) { return refl ? (kind == kGridFp32 ? 3 : 4) : 6; }

GridShape grid_shape(const int n[3], int axis, int nx_eval, int n_states, bool reflect, GridKind kind) {
    GridShape g{};
    g.axis = axis;
    g.l[0] = axis == 0 ? 1 : 0;
    g.l[1] = axis == 2 ? 1 : 2;
    g.n1 = g.l[0] == 0 ? nx_eval : n[1];
    const int nc = n[axis];
    g.reflect = reflect ? 1 : 0;
    g.kind = kind;
    g.planes = kind == kGridSplitF16 ? Operands<false>::planes : Operands<true>::planes;
    g.ncol = reflect ? (nc + 1) / 2 : nc;
    g.iz0 = reflect ? nc - g.ncol : 0;
    g.nyp = (n[g.l[1]] + 1) & ~1;   // lines in pairs of one value of l[0]
    const int ng = (g.ncol + 15) / 16, tr = 16 * kGridWaves;
    const long long nrows = (long long)g.n1 * g.nyp * n_states;
    g.ntl = (int)((nrows + tr - 1) / tr);
    // most line pairs that a tile's rows touch
    g.np = 1;
    for (long long r = 0; r < std::min(2LL * tr * n_states, nrows); r += tr) {
        const int p = (int)((r + tr - 1) / n_states / 2 - r / n_states / 2 + 1);
        g.np = std::max(g.np, p);
    }
    long long best = 0;
    for (int cg = 1; cg <= max_cg(kind, reflect); ++cg) {
        int tcm = 2;
        auto bytes = [&] { return 4 * (grid_vbufs(cg, reflect) * cg * g.planes * 256 + 2 * tcm * (48 * n_states + 2 * g.np * kWLine)); };
        if (bytes() > kGridLds) tcm = 1;
        if (bytes() > kGridLds) break;
        const int nt = (ng + cg - 1) / cg;
        if (nt * cg > ng + 1) continue;
        const long long cost = (long long)nt * (30 + (kind == kGridFp32 ? 31 : kind == kGridSplitF16 ? 10 : 22) * cg);
        if (!g.cg || cost < best) {
            best = cost;
            g.cg = cg;
            g.ntc = nt;
            g.tcm = tcm;
            g.lds = bytes();
        }
    }
    g.ncg = g.ntc * g.cg;
    g.cost = best * g.ntl;
    return g;
}

// The kernel's variant: kind, with or without mirror values, column groups; some
// numbers have no kernel (FP32 precision with four groups and mirror values).
int grid_class(const GridShape& g) { return 10 * g.kind + (g.reflect ? g.cg - 1 : 3 + g.cg); }

// Workgroups resident per CU: what the registers allow, and the 160 KB of LDS.
int grid_wgs_per_cu(int cls, int lds) {
    const bool fold = cls / 10 == kGridFp32, refl = cls % 10 < 4;
    return std::min(grid_waves(refl ? cls % 10 + 1 : cls % 10 - 3, fold, refl),
                    160 * 1024 / ((lds + 16 + kLdsGranule - 1) / kLdsGranule * kLdsGranule));
}

hipError_t grid_desc(const GridShape& g, const PrepResult& p, const float2* V, uint32_t ybase, const uint4* Bt,
                     const int2* terms, const float* Tw, const double* sinv, const ChunkSplit& sp, const int n[3],
                     int n_states, float2* f, float* f2, double2* part, GridDesc* d, long long* blocks) {
    const int nxr = p.n_axis[g.l[0]] + 1, nyr = p.n_axis[g.l[1]] + 1;
    if (p.axis != g.axis || (size_t)ybase < (size_t)n[g.l[0]] * nxr * sizeof(float2)) return hipErrorInvalidValue;
    if (g.n1 < 1 || g.n1 > n[g.l[0]] || n_states < 1 || n_states > kMaxStates) return hipErrorInvalidValue;
    if (g.cg < 1 || g.cg > 6 || g.ncg != g.cg * g.ntc || g.ncg * 16 < g.ncol || g.tcm < 1 || g.tcm > 2)
        return hipErrorInvalidValue;
    if ((long long)g.n1 * g.nyp * n_states > 0x7fffffff - 64) return hipErrorInvalidValue;   // at most 4096 4096 32
    if (sp.n < 1 || sp.n > kMaxSplit || sp.lo[0] != 0) return hipErrorInvalidValue;
    for (int j = 0; j < sp.n; ++j)
        if (sp.lo[j + 1] < sp.lo[j]) return hipErrorInvalidValue;
    if (sp.n > 1 && !part) return hipErrorInvalidValue;
    d->V = V;
    d->nxr = nxr;
    d->nyr = nyr;
    d->ybase = ybase;
    d->Bt = Bt;
    d->steps = p.ksteps;
    d->terms = terms;
    d->Tw = Tw;
    d->sinv = sinv;
    d->sp = sp;
    const int stride[3] = {n[1] * n[2], n[2], 1};
    d->sx = stride[g.l[0]];
    d->sy = stride[g.l[1]];
    d->sz = stride[g.axis];
    d->npts = (long long)n[0] * n[1] * n[2];
    d->nl = n[g.l[1]];
    d->nc = n[g.axis];
    d->n1 = g.n1;
    d->n_states = n_states;
    d->nyp = g.nyp;
    d->tcm = g.tcm;
    d->np = g.np;
    d->ntl = g.ntl;
    d->ntc = g.ntc;
    d->ncg = g.ncg;
    d->ncol = g.ncol;
    d->iz0 = g.iz0;
    d->f = f;
    d->f2 = f2;
    d->partial = sp.n > 1 ? part : nullptr;
    d->part_stride = n_states * d->npts;
    *blocks = (long long)g.ntl * g.ntc * sp.n;
    return hipSuccess;
}

#define SCFF_GRID_CASES(KERNEL, ...)                                                      \
    switch (cls) {                                                                        \
        case 0: SCFF_GRID_VARIANT((KERNEL<1, true, true, true>), __VA_ARGS__); break;     \
        case 1: SCFF_GRID_VARIANT((KERNEL<2, true, true, true>), __VA_ARGS__); break;     \
        case 2: SCFF_GRID_VARIANT((KERNEL<3, true, true, true>), __VA_ARGS__); break;     \
        case 4: SCFF_GRID_VARIANT((KERNEL<1, true, true, false>), __VA_ARGS__); break;    \
        case 5: SCFF_GRID_VARIANT((KERNEL<2, true, true, false>), __VA_ARGS__); break;    \
        case 6: SCFF_GRID_VARIANT((KERNEL<3, true, true, false>), __VA_ARGS__); break;    \
        case 7: SCFF_GRID_VARIANT((KERNEL<4, true, true, false>), __VA_ARGS__); break;    \
        case 8: SCFF_GRID_VARIANT((KERNEL<5, true, true, false>), __VA_ARGS__); break;    \
        case 9: SCFF_GRID_VARIANT((KERNEL<6, true, true, false>), __VA_ARGS__); break;    \
        case 10: SCFF_GRID_VARIANT((KERNEL<1, false, false, true>), __VA_ARGS__); break;  \
        case 11: SCFF_GRID_VARIANT((KERNEL<2, false, false, true>), __VA_ARGS__); break;  \
        case 12: SCFF_GRID_VARIANT((KERNEL<3, false, false, true>), __VA_ARGS__); break;  \
        case 13: SCFF_GRID_VARIANT((KERNEL<4, false, false, true>), __VA_ARGS__); break;  \
        case 14: SCFF_GRID_VARIANT((KERNEL<1, false, false, false>), __VA_ARGS__); break; \
        case 15: SCFF_GRID_VARIANT((KERNEL<2, false, false, false>), __VA_ARGS__); break; \
        case 16: SCFF_GRID_VARIANT((KERNEL<3, false, false, false>), __VA_ARGS__); break; \
        case 17: SCFF_GRID_VARIANT((KERNEL<4, false, false, false>), __VA_ARGS__); break; \
        case 18: SCFF_GRID_VARIANT((KERNEL<5, false, false, false>), __VA_ARGS__); break; \
        case 19: SCFF_GRID_VARIANT((KERNEL<6, false, false, false>), __VA_ARGS__); break; \
        case 20: SCFF_GRID_VARIANT((KERNEL<1, false, true, true>), __VA_ARGS__); break;   \
        case 21: SCFF_GRID_VARIANT((KERNEL<2, false, true, true>), __VA_ARGS__); break;   \
        case 22: SCFF_GRID_VARIANT((KERNEL<3, false, true, true>), __VA_ARGS__); break;   \
        case 23: SCFF_GRID_VARIANT((KERNEL<4, false, true, true>), __VA_ARGS__); break;   \
        case 24: SCFF_GRID_VARIANT((KERNEL<1, false, true, false>), __VA_ARGS__); break;  \
        case 25: SCFF_GRID_VARIANT((KERNEL<2, false, true, false>), __VA_ARGS__); break;  \
        case 26: SCFF_GRID_VARIANT((KERNEL<3, false, true, false>), __VA_ARGS__); break;  \
        case 27: SCFF_GRID_VARIANT((KERNEL<4, false, true, false>), __VA_ARGS__); break;  \
        case 28: SCFF_GRID_VARIANT((KERNEL<5, false, true, false>), __VA_ARGS__); break;  \
        case 29: SCFF_GRID_VARIANT((KERNEL<6, false, true, false>), __VA_ARGS__); break;  \
        default: return hipErrorInvalidValue;                                             \
    }

// Dynamic LDS beyond 64 KB must be allowed per kernel (on the current device; the
// same each time, so once is enough).
hipError_t grid_allow_lds(int device) {
    static std::atomic<uint64_t> allowed{0};   // devices
    const uint64_t bit = device < 64 ? 1ull << device : 0;
    if (allowed.load() & bit) return hipSuccess;
    hipError_t e = hipSuccess;
    auto allow = [&](const void* f) {
        if (e == hipSuccess) e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, kGridLds + 16);
    };
#define SCFF_GRID_VARIANT(K, ...) allow((const void*)(K))
    auto one = [&](int cls) {
        SCFF_GRID_CASES(grid_kernel)
        return hipSuccess;
    };
    auto batch = [&](int cls) {
        SCFF_GRID_CASES(grid_batch_kernel)
        return hipSuccess;
    };
#undef SCFF_GRID_VARIANT
    for (int cls = 0; cls < kGridClasses; ++cls) {
        (void)one(cls);   // (a class that does not exist allows nothing)
        (void)batch(cls);
    }
    if (e == hipSuccess) allowed |= bit;
    return e;
}

#define SCFF_GRID_VARIANT(K, ...) hipLaunchKernelGGL(K, __VA_ARGS__)
hipError_t launch_grid(int cls, const GridShape& g, const GridDesc& d, long long blocks, hipStream_t st) {
    if (blocks < 1 || blocks > 0x7fffffffLL || g.lds > kGridLds) return hipErrorInvalidValue;
    const dim3 grid((unsigned)blocks), block(kGridWaves * 64);
    SCFF_GRID_CASES(grid_kernel, grid, block, g.lds, st, d)
    return hipGetLastError();
}

// Persistent launch over a queue of (descriptor, tile) items of class cls:
// `wgs` workgroups (the device's resident capacity), each looping until the
// queue is exhausted; lds: the largest GridShape::lds of the requests.
// *counter must be 0 when the launch starts.
hipError_t launch_grid_batch(int cls, int lds, const GridDesc* descs, const int2* items, int n_items, int* counter,
                             int wgs, hipStream_t st) {
    if (n_items < 1 || wgs < 1 || lds > kGridLds) return hipErrorInvalidValue;
    const dim3 grid((unsigned)wgs), block(kGridWaves * 64);
    SCFF_GRID_CASES(grid_batch_kernel, grid, block, lds + 16, st, descs, items, n_items, counter)
    return hipGetLastError();
}

hipError_t launch_zero_counters(int* c, int n, hipStream_t st) {
    if (n < 1 || n > 256) return hipErrorInvalidValue;
    hipLaunchKernelGGL(zero_counters_kernel, dim3(1), dim3(256), 0, st, c, n);
    return hipGetLastError();
}

hipError_t launch_reduce(const double2* part, int n_split, const int n[3], int nx_eval, int n_states, float2* f,
                         float* f2, hipStream_t st) {
    if (n_split < 1 || nx_eval < 1 || nx_eval > n[0]) return hipErrorInvalidValue;
    const long long tot = (long long)nx_eval * n[1] * n[2] * n_states;
    int blocks = (int)((tot + 255) / 256);
    if (blocks > 16384) blocks = 16384;
    hipLaunchKernelGGL(reduce_kernel, dim3(blocks), dim3(256), 0, st, part, n_split,
                       (long long)n_states * n[0] * n[1] * n[2], make_int3(n[0], n[1], n[2]), nx_eval, n_states, f,
                       f2);
    return hipGetLastError();
}

hipError_t launch_mirror(const int n[3], int nx_eval, int n_states, float2* f, float* f2, hipStream_t st) {
    // planes ix >= nx_eval mirror planes nx-1-ix < nx - nx_eval <= nx_eval (computed)
    if (nx_eval < (n[0] + 1) / 2 || nx_eval > n[0]) return hipErrorInvalidValue;
    if (nx_eval == n[0]) return hipSuccess;
    const long long tot = (long long)(n[0] - nx_eval) * n[1] * n[2] * n_states;
    int blocks = (int)((tot + 255) / 256);
    if (blocks > 16384) blocks = 16384;
    hipLaunchKernelGGL(mirror_kernel, dim3(blocks), dim3(256), 0, st, make_int3(n[0], n[1], n[2]), nx_eval,
                       n_states, f, f2);
    return hipGetLastError();
}

}  // namespace scff
