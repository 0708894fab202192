// Internal declarations of the form-factor engine (host precompute, device
// kernels, runtime).  Not part of the public ABI; see include/scarff.h.
#pragma once

#include <array>
#include <cstddef>
#include <cstdint>
#include <functional>
#include <shared_mutex>
#include <string>
#include <vector>

#include <hip/hip_runtime.h>

#include "../../include/scarff.h"

namespace scff {

// Maximum primitive-pair terms per (virtual) component pair.  A component
// pair with more terms is split into several virtual pairs that share its
// packed transition weight, so any contraction length is supported.
constexpr int kMaxTermsPerPair = 9;
// Component pairs per unit: the layout granule of packed weights and term
// slots, and one pair of MFMA k-steps (4 pairs each) of the grid kernel.
constexpr int kChunk = 8;
// Chunks: runs of consecutive units that share a term count npp, at most
// kMaxUnitsPerChunk units and kMaxChunkTerms terms (reported by scff_query).
constexpr int kMaxUnitsPerChunk = 4;
constexpr int kMaxChunkTerms = kChunk * kMaxTermsPerPair;   // 72
// Grid kernel: z rows (distinct 1D rows of the contracted axis, "z" in all that
// follows; x or y of the grid where that is cheaper) come in k-steps of kZStep, sorted by their number of terms (at most kZTerms: the component
// pairs of one primitive pair that share its z powers).
constexpr int kZStep = 32;
constexpr int kZTerms = 9;
constexpr int kWPasses = 2;       // W items per lane whose loads go out a step ahead
constexpr int kGridLds = 81920 - 16;   // LDS bytes of a workgroup, at most: half a CU's (the batch kernel adds 16)
constexpr int kLdsGranule = 1280;      // a CU's 160 KB in 128 blocks
constexpr int kWLine = 84;        // floats of W per line: 4 groups of 8 z rows, padded apart in the banks
// Arithmetic of the grid kernel's products: FP32 precision; split precision on
// f16 halves, or on BF16 parts where the values fall out of the halves' range.
enum GridKind { kGridFp32, kGridSplitF16, kGridSplitBf16 };
constexpr int kGridClasses = 30;   // kernel variants: kind, mirror values or not, column groups per tile
// Bins of the s-s terms by binary exponent of p (PrepResult::tail): the first
// holds p < 2^(kTailMin + 1)
constexpr int kTailBins = 32, kTailMin = -12;
// Term counts of the k-steps, longest rows first: k-step k has the largest n
// with k < kend[n], so a k-step's position in the term arrays is closed form.
struct KSteps {
    int kend[kZTerms + 1];   // [n]: k-steps of n or more terms (n >= 1)
};
__host__ __device__ inline int ksteps_terms(const KSteps& s, int k) {
    int n = 0;
    for (int i = 1; i <= kZTerms; ++i) n += k < s.kend[i];
    return n;
}
__host__ __device__ inline int ksteps_first(const KSteps& s, int k) {   // terms per z row of the k-steps before k
    int c = 0;
    for (int i = 1; i <= kZTerms; ++i) c += k < s.kend[i] ? k : s.kend[i];
    return c;
}
// Floats of the weights of one term index of a k-step: [group of 8 z rows][state][8 + 4]
__host__ __device__ constexpr int grid_term_weights(int ns) { return 48 * ns; }
// The grid kernel may split a grid's k-steps into up to kMaxSplit ranges
// (one workgroup per tile and range, FP64 partial sums reduced afterwards)
// when the grid has too few tiles to fill the device.
constexpr int kMaxSplit = 32;
struct ChunkSplit {
    int n;                   // number of ranges (1 = no split)
    int lo[kMaxSplit + 1];   // range j is k-steps [lo[j], lo[j+1]); lo[0] = 0, lo[n] = n_ksteps
};
// Tiling of an evaluation: the contracted axis, whose values are the columns, and
// the line axes l[0], l[1] (the others, in order; lines are numbered with l[1]
// fastest); columns computed (the upper half of an axis symmetric about 0),
// column groups of 16 per tile (cg) and in all (ncg, padded to whole tiles), row
// and column tiles, lines per value of l[0] (padded to pairs), terms of a k-step
// handled between two barriers, most line pairs a tile touches, planes of a V
// block, LDS bytes of a workgroup; estimated cost (relative).
struct GridShape {
    GridKind kind;
    int axis, l[2], n1;   // n1: values of l[0] computed
    long long cost;
    int reflect, ncol, iz0, cg, ntc, ncg, ntl, nyp, tcm, np, planes, lds;
};
// Everything the fused grid kernel needs for one evaluation (one request of
// a batch): the x / y tables, the z axis' operand blocks, the k-steps with
// their terms and weights, the grid and its tiling, the split of the k-steps
// and the outputs.  Filled on the host; the batch kernel reads it from device
// memory.
struct GridDesc {
    const float2* V;          // table of line axis 0 ("x"), then (from byte ybase) of line axis 1 ("y")
    int nxr, nyr;             // their rows, the zero row included
    uint32_t ybase;
    const uint4* Bt;          // contracted axis ("z"), operand order
    const int2* terms;        // (x row, y row)
    const float* Tw;          // weights (grid_term_weights)
    const double* sinv;       // per state: the power of two that undoes the scaling
    ChunkSplit sp;
    int nl, nc;               // grid points of line axis 1 and of the contracted axis
    int sx, sy, sz;           // output strides of the line axes and the contracted one
    long long npts;           // grid points
    KSteps steps;
    int n1, n_states;         // values of line axis 0 computed
    int ntl, ntc, ncg, ncol, iz0, nyp, tcm, np;
    float2* f;                // outputs (NULL to skip), or
    float* f2;
    double2* partial;         // FP64 partial sums of a split (NULL: unsplit)
    long long part_stride;
};
// States per MFMA row block.
constexpr int kStateBlock = 16;
constexpr int kMaxStates = 32;
constexpr int kMaxPrim = 32;

// One 1D V-tensor row is a (primitive pair, axis, power pair) triple.  On a
// q value of its axis it evaluates
//   V(q) = exp(-q^2/(4p)) * exp(i q P) * sum_u e[u] (i q)^u ,
// where every q-independent factor of the pair (contraction coefficients,
// primitive normalisation on this axis, and on the x row the Gaussian
// product prefactor with (pi/p)^{3/2}) is folded into e[].
// Device copy of a row.  The 1D tables are built from it in FP64 and rounded
// once to FP32 (phase argument, range reduction, Gaussian and polynomial).
struct VRowDev {
    double P;
    double inv4p;    // 1/(4p)
    double e[5];
    int deg;
    int axis;
};

// A device allocation owned by a context.
struct DeviceBuffer {
    void* p = nullptr;
    size_t bytes = 0;
};

struct PrepShell {
    int atom, l, nprim, off;
};

// Host-side view of a loaded molecule: validated basis plus the integer
// tables that lay out rows, component pairs and terms (no arithmetic of the
// method beyond normalisation constants).
struct Basis {
    int n_atoms = 0, n_shells = 0, nbf = 0;
    std::vector<double> xyz;
    std::vector<int> sh_atom, sh_l, sh_nprim, sh_off, sh_bf0;
    std::vector<double> exps, coefs;
    std::vector<double> cnorm;   // contracted normalisation per AO
    std::vector<double> n1d;     // per primitive, 1D normalisation for powers 0..2
    bool normalise = true;
    // layout tables
    int n_sp = 0, n_cp = 0;
    long long n_rows = 0, n_terms = 0;
    std::vector<PrepShell> shells;
    std::vector<int> sp;          // 4 ints per shell pair: sA, sB, row_off, term_off
    std::vector<int> sp_cp;       // first component pair of each shell pair
    std::vector<int> cp_first;    // first term of each component pair
    std::vector<int> cp_nterms;   // primitive pairs of each component pair
};

// Device pointers the precompute reads.
struct PrepInputs {
    const PrepShell* shells;
    const int4* sp;
    const int* sp_cp;
    const int* bf0;
    const int* cp_first;
    const int* cp_nterms;
    const double* xyz;
    const double* exps;
    const double* coefs;
    const double* n1d;
    const double* cnorm;
    const double* T;
    int nbf, n_states, n_sp, n_cp;
    long long n_rows_all, n_terms_all;
    double eps, spin;
};

// What the separable-integral and dipole kernels (lowq.hip) read of the
// precompute; newid numbers the used rows from 0, at [axis nr + row].
struct LowqPrep {
    const int *cp_first, *cp_nterms;
    const VRowDev* rows;   // all rows, by shell pair
    const int4* trow;
    const double *wt, *thr, *tp64;
    const int* newid;
    int nr;
};

// Point evaluation (points.hip): the precompute's arrays, the points and what is
// written (f, |f|^2, |f|^2 in FP64; each may be null).  part: FP64 sums per
// share of the shell pairs, [n_split][state][point], null for one share.
struct PointArgs {
    const PrepShell* shells;
    const int4* sp;
    const int* sp_cp;
    const VRowDev* rows;   // all rows, by shell pair
    const double *wt, *thr, *tp64, *q;
    int n_sp, ns, nq;
    float2* f;
    float* f2;
    double* f2d;
    double2* part;
};

// Device buffers of the precompute.  What the grid kernel reads: rows, zslots,
// zterms, zw and the state factors in small; the layout by component
// pairs (made when the export first needs it): slots, tp32 and, per
// unit, cnpp (terms per pair) and coff (first slot).
struct PrepWork {
    DeviceBuffer rows_all, rowsum, trow, tbound, wt, tp64, bsum, part, small, nk, nv, vbase,
        tmp, key, val, vinfo, tmp2, cnpp, csize, coff, tmp3, slots, tp32, row_used, newid, tmp4,
        rows, zslots, zterms, zw;
    // pinned host memory of the context (kPinnedBytes, or NULL if it could
    // not be allocated): small readbacks and the molecule upload travel through
    // it by DMA; every use is complete before run_prep returns
    void* pinned = nullptr;
};

constexpr size_t kPinnedBytes = (size_t)4 << 20;
// byte offsets in the precompute's small buffer
constexpr size_t kSmallStats = 1024, kSmallSinv = 1280, kSmallKs = 1792, kSmallHist = 2048;   // kHistBins unsigned
// what the host reads back, together
constexpr size_t kSmallMeta = 7168, kSmallZmax = kSmallMeta + 64, kSmallTail = kSmallZmax + 8 * kMaxStates;
constexpr size_t kSmallBytes = kSmallTail + 8 * kMaxStates * kTailBins;
constexpr size_t kPinnedTables = 4096;   // byte offset of the molecule upload

struct PrepResult {
    int n_rows = 0, n_axis[3] = {};   // compacted rows: the zero row, then the rows of x, y and z
    int axis = 2;                     // contracted axis of the grid kernel's layout
    int seg(int a) const { return (a > 0 ? n_axis[0] : 0) + (a > 1 ? n_axis[1] : 0); }   // rows before axis a's, the zero row aside
    int n_ksteps = 0, state_blocks = 1;
    KSteps ksteps{};
    long long n_zterms = 0, n_zweights = 0;
    // per state: bound of its largest z row, and the largest |weight| x bound of its
    // s-s terms by exponent of p (a term of bin b falls off as e^{-q^2/4p}, p >=
    // 2^(kTailMin + b)); the range of f over a grid
    double zmax[kMaxStates] = {}, tail[kMaxStates][kTailBins] = {};
    // layout by component pairs (run_prep_stats)
    int n_virtual = 0, n_vpairs = 0, n_units = 0, n_chunks = 0;
    long long n_slots = 0, pairs_kept = 0, terms_kept = 0;
};

// ---- host side of the precompute (precompute.cpp) ----
std::string build_basis(Basis& b, int n_atoms, const double* xyz, int n_shells,
                        const int* shell_atom, const int* shell_l, const int* shell_nprim,
                        const double* exps, const double* coefs, int normalise);

// ---- device precompute (prep.hip) ----
// axis: contracted axis of the grid kernel's layout; run_prep_layout makes the
// layout of another one.
hipError_t run_prep(const PrepInputs& in, PrepWork& w, PrepResult& res, int axis, hipStream_t st,
                    const std::function<hipError_t(DeviceBuffer&, size_t)>& alloc);
hipError_t run_prep_layout(const PrepInputs& in, PrepWork& w, PrepResult& res, int axis, bool first, hipStream_t st,
                           const std::function<hipError_t(DeviceBuffer&, size_t)>& alloc);
hipError_t run_prep_stats(const PrepInputs& in, PrepWork& w, PrepResult& res, hipStream_t st);
hipError_t run_prep_pairs(const PrepInputs& in, PrepWork& w, const PrepResult& res, hipStream_t st,
                          const std::function<hipError_t(DeviceBuffer&, size_t)>& alloc);

// ---- static scratch (scratch.hip) ----
// Bytes of the per-device scratch array of scff_eval_grid_noalloc.
// kScratchBytes is the limit on a grid's tables of 8 bytes per (row, value);
// kScratchSlack covers the z axis' 12 bytes in FP32 precision (at most 9 of 19
// rows of a primitive pair are z rows, so 0.24 of the limit) and z rows padded
// to whole k-steps and column tiles when there are few of them.
constexpr size_t kScratchBytes = (size_t)256 << 20;
constexpr size_t kScratchSlack = (size_t)72 << 20;
// Device address of this device's array (device current; resolved once).
hipError_t scratch_address(int device, void** ptr);

// ---- FFT method (fft.hip) ----
// Molecule tables the transition-density kernel reads (device pointers).
struct FftMol {
    const PrepShell* shells;
    const int* bf0;
    const double* xyz;
    const double* exps;
    const double* coefs;
    const double* n1d;
    const double* cnorm;
    int n_shells;
};
// LDS a density workgroup may hold: its AO block grows with the basis, up to
// 1232 functions of 6 bytes a value in FP32 precision (4 in split-BF16).
constexpr size_t kFftLdsBytes = (size_t)120 << 10;
constexpr int kFftMaxPad = 1232;
// Column blocks of 16 points per density workgroup for nbf_pad basis rows
// (4, 2 or 1), 0 if the AO block does not fit lds_limit bytes of LDS.
int fft_density_cb(int precision, int nbf_pad, size_t lds_limit);
// precision: SCFF_FP32 (weights in three BF16 parts) or SCFF_BF16X3 (in two), as
// operands of 16x16x32 products.
size_t fft_pack_bytes(int precision, int nbf_pad, int ns);   // of the array that launch_fft_pack fills
hipError_t launch_fft_pack(int precision, const double* T, const double* cnorm, int nbf, int nbf_pad, int ns,
                           double spin, void* Ap, hipStream_t st);
hipError_t launch_fft_density(int precision, const FftMol& m, const void* Ap, int nbf_pad, int ns, const int n[3],
                              const double x0[3], const double h[3], float* Z, float* phi, double* psum,
                              size_t lds_limit, long long* n_part, hipStream_t st);
hipError_t launch_fft_lines(float2* Z, int nb, const int n[3], hipStream_t st);
hipError_t launch_fft_finish(const float2* Z, const int n[3], int ns, double vpix, const double u[3], float2* f,
                             float* f2, double* psum, long long* n_part, hipStream_t st);
hipError_t launch_fft_sum(const double* part, int ns, long long n, double scale, double* out, int stride,
                          hipStream_t st);

// ---- spherical method (sph_tables.cpp, sph.hip) ----
// Polynomial degree of one geometry's D tensor (l_A + l_B <= 4 for d shells).
constexpr int kSphMaxN = 4;
// Gaunt entries per (lam mu, l m): L = |l - lam| + 2 j, j < 5.
constexpr int kSphGauntJ = 5;
constexpr int kSphMaxL = 48;   // largest lmax accepted
struct SphIndex {
    std::vector<std::array<int, 3>> nlm;   // (n, lam, mu) of the W tensor, n <= 4, lam = n, n-2, ...
    std::vector<std::array<int, 3>> uvw;   // monomial powers with u + v + w <= 4
};
SphIndex sph_index();
// Theta[uvw][nlm] complex (re, im), zero unless u + v + w = n.
std::vector<double> sph_theta_table(const SphIndex& ix);
// Gaunt[(lam mu)][(l m)][j], (lmax + 1)^2 harmonics l m, real.
std::vector<double> sph_gaunt_table(int lmax);
// The same in real harmonics (S_lm = (-1)^m sqrt(2) Re Y_l^m, S_l,-m = (-1)^m
// sqrt(2) Im Y_l^m), whose coefficients are real.
std::vector<double> sph_theta_real(const SphIndex& ix);
// One geometry (shell pair, primitive pair) of the spherical method.
struct SphGeom {
    int pp;           // primitive pair within the shell pair
    int ncp, npp;     // component pairs and primitive pairs of the shell pair
    int term0;        // first term of the shell pair
    int lsum;         // l_A + l_B; geometries are sorted by it, largest first
};
// Geometries of l_A + l_B >= lam.
struct SphExt {
    int n[kSphMaxN + 1];
};
// Work item of the contraction: a row tile, a range of geometries, where the
// tile's second 16 rows end, the index of its partial sum (-1: the tile's only
// range).
struct SphItem {
    int tile, k0, k1, kb, part;
};
// Partial sums first[t] .. first[t + 1] - 1 belong to row tile t, t < n_split.
struct SphSegs {
    int n_split;
    int first[kMaxStates * (kSphMaxN + 1) * (kSphMaxN + 1) / 32 + 2];
};
inline int sph_geo_stride(int n_geo) { return (n_geo + 15) & ~15; }
void sph_plan(const SphExt& ext, int ns, int Lmax, int n_q, int n_cu, bool split, std::vector<SphItem>& items,
              SphSegs& segs);
hipError_t launch_sph_geom(const SphGeom* geo, int n_geo, const VRowDev* rows, const int4* trow, const double* tp64,
                           int ns, const double* theta, const int* uvw_idx, const int* nfirst, int n_nlm, int Lmax,
                           double4* gdat, double* Y, double* W, hipStream_t st);
// Bq: workspace of nqb radii x ns 25 rows x sph_geo_stride(n_geo) (the row
// operands of one batch of radii); P: partial sums, 32 rows x columns per
// (part, radius).
hipError_t launch_sph_q(const double4* gdat, const double* Y, const double* W, const SphExt& ext, int n_geo, int ns,
                        int Lmax, const int* nlm_of, const double* qs, int n_q, double* J, double* Bq, int nqb,
                        const SphItem* items, int n_items, const SphSegs& segs, double* Q, double* P, hipStream_t st);
hipError_t launch_sph_couple(const double* Q, const double* gaunt, int ns, int lmax, int Lmax, int n_q, double2* R,
                             hipStream_t st);
hipError_t launch_sph_grid(const double2* R, int ns, int lmax, int n_q, int n_theta, int n_phi, double2* F,
                           float2* f, float* f2, hipStream_t st);
hipError_t launch_sph_avg(const double2* R, int ns, int lmax, int n_q, double* avg, hipStream_t st);

// ---- runtime.cpp ----
// Gate between stream capture and device-wide runtime calls.  Allocation and
// release of device or pinned memory, event and stream creation and
// destruction, and device synchronisation take it shared; a thread that
// captures a stream into a graph holds it exclusively from the start to the
// end of the capture, so no such call (which the runtime may let touch or
// synchronise every stream, the capturing one included) runs meanwhile.
// Hold it only around the runtime call itself, never across another gated
// call.
std::shared_mutex& device_gate();
using GateShared = std::shared_lock<std::shared_mutex>;
// Thread-local message returned by scff_last_error().
void set_error(const std::string& msg);
// Pack and upload a context's problem for grid g on stream st and wait for
// it: when this returns, the precompute is complete in device memory, so an
// evaluation on any other stream may use it.  *bytes_needed receives the
// device bytes an evaluation on g in `precision` will hold in total.
int ctx_prepare(scff_ctx* c, const scff_grid* g, int precision, hipStream_t st, size_t* bytes_needed);
// Device bytes a context holds (its buffers are kept between calls).
size_t ctx_device_bytes(const scff_ctx* c);

// Two-phase evaluation of a prepared context for the server's batch runner:
// ctx_batch_reserve reserves every device buffer the evaluation needs (1D
// tables, device outputs, split partial sums) and fills the grid kernel's
// descriptor, without launching anything; ctx_batch_tables and
// ctx_batch_finish then only enqueue work (1D tables; split reduction and
// the copy of f / |f|^2 to host memory), so a batch's launches can be
// captured into a graph.
struct BatchEval {
    GridDesc desc;
    GridShape shape;
    int cls = 0;               // grid kernel variant, < kGridClasses
    long long blocks = 0;      // tiles x splits of the evaluation
    int n_split = 1, nx_eval = 0;
    size_t nout = 0;           // output values (n_states x grid points)
};
int ctx_batch_reserve(scff_ctx* c, const scff_grid* g, int precision, bool want_f, bool want_f2, BatchEval* be);
int ctx_batch_tables(scff_ctx* c, const scff_grid* g, const BatchEval& be, hipStream_t st);
int ctx_batch_finish(scff_ctx* c, const scff_grid* g, const BatchEval& be, float* host_f, float* host_f2,
                     hipStream_t st);
// After the batch's stream has been synchronised: the context has no
// asynchronous work pending.
void ctx_batch_done(scff_ctx* c);
// Grid kernel launchers (kernels.hip)
hipError_t grid_allow_lds(int device);   // the current device, before the first launch on it
int grid_wgs_per_cu(int cls, int lds);
hipError_t launch_grid_batch(int cls, int lds, const GridDesc* descs, const int2* items, int n_items, int* counter, int wgs,
                             hipStream_t st);
hipError_t launch_zero_counters(int* c, int n, hipStream_t st);
int ctx_n_cu(const scff_ctx* c);

}  // namespace scff
