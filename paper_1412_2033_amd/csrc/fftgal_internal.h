// Internal declarations shared by the host library (fftgal.cpp) and the HIP
// kernels (fftgal_kernels.hip).  Not part of the public C ABI.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

namespace fftgal {

constexpr int kThreads = 256;   // work-group size of every kernel
constexpr int kMaxStages = 16;  // radix-3/5/7 stages per FFT length

// Mixed-radix factorisation of one FFT length and where its twiddles live.
// Stage s has radix radix[s] and twiddles w(q, k) = exp(-2 pi i q k / (p r)),
// q = 1..r-1, k = 0..p-1 (p = product of the earlier radices), stored at
// twoff[s] + (q - 1) * p + k in the plan's twiddle tables.
// A length n that is not 3,5,7-smooth is transformed by Bluestein's chirp
// convolution: with c_m = exp(sg i pi m^2 / n), sum_j x_j exp(sg 2 pi i j k / n)
// = c_k sum_j (x_j c_j) conj(c_{k-j}), a circular convolution of length L >= 2n - 1
// (3,5,7-smooth) done with two transforms of length L; the stages then describe
// L, and the tables hold the chirp exp(i pi m^2 / n) (m < n) at choff and
// H = DFT_L^-(conj chirp, placed at m mod L for |m| < n) / L at hoff.
struct FftDesc {
    int n;
    int nst;
    int radix[kMaxStages];
    int twoff[kMaxStages];
    int L;      // transform buffer length in LDS: n, or the Bluestein length
    int blue;   // 1: Bluestein transform of length n through length L
    int choff;
    int hoff;
};

// Transform lengths with compile-time specialised kernels, and their radix
// schedules (composite radices are done in registers): every odd 3,5,7-smooth
// length from 9 to 2025, the lengths a double grid takes, and, for the plans
// whose transforms have the length of the order itself (GaNi, reduced Ga), 20
// odd lengths up to 385 with a factor 11 or 13 (those listed below; 275, 351 and
// 363 are not among them), which would otherwise run Bluestein's convolution of
// twice the length (3D GaNi of order 99 with its bounds, FP64: 121 -> 67 ms).
// The host builds the twiddle tables of these lengths with the same schedule,
// and the generic kernels run it too (radices 3, 5, 7, 9, 11, 13, 15, 25).  The schedules of the first six read the same forwards and
// backwards where the length allows: then the last stage of an inverse
// transform leaves each thread holding exactly the points that the first stage
// of a forward transform consumes.  The others get that from running the
// forward transform as the transpose of the inverse one (row_iso_pairs).
struct FastSched {
    int n;
    int nst;
    int r[4];
};
constexpr FastSched kFastSched[] = {
    {81, 2, {9, 9, 0, 0}},      {125, 2, {25, 5, 0, 0}},   {225, 2, {15, 15, 0, 0}},
    {245, 3, {7, 5, 7, 0}},     {729, 3, {9, 9, 9, 0}},    {2025, 3, {15, 9, 15, 0}},
    {9, 2, {3, 3, 0, 0}},       {15, 2, {5, 3, 0, 0}},     {21, 2, {3, 7, 0, 0}},
    {25, 2, {5, 5, 0, 0}},      {27, 2, {9, 3, 0, 0}},     {35, 2, {5, 7, 0, 0}},
    {45, 2, {5, 9, 0, 0}},      {49, 2, {7, 7, 0, 0}},     {63, 2, {9, 7, 0, 0}},
    {75, 2, {5, 15, 0, 0}},     {105, 2, {7, 15, 0, 0}},   {135, 2, {15, 9, 0, 0}},
    {147, 3, {7, 3, 7, 0}},     {175, 3, {5, 7, 5, 0}},    {189, 3, {9, 3, 7, 0}},
    {243, 3, {9, 3, 9, 0}},     {315, 3, {9, 5, 7, 0}},    {343, 3, {7, 7, 7, 0}},
    {375, 3, {5, 15, 5, 0}},    {405, 3, {9, 5, 9, 0}},    {441, 3, {7, 9, 7, 0}},
    {525, 3, {7, 5, 15, 0}},    {567, 3, {9, 7, 9, 0}},    {625, 3, {5, 25, 5, 0}},
    {675, 3, {9, 5, 15, 0}},    {735, 3, {7, 15, 7, 0}},   {875, 3, {5, 25, 7, 0}},
    {945, 3, {7, 9, 15, 0}},    {1029, 4, {7, 7, 3, 7}},   {1125, 3, {15, 5, 15, 0}},
    {1215, 3, {9, 15, 9, 0}},   {1225, 4, {7, 5, 5, 7}},   {1323, 4, {7, 9, 3, 7}},
    {1575, 3, {15, 7, 15, 0}},  {1701, 4, {9, 7, 3, 9}},   {1715, 4, {7, 5, 7, 7}},
    {1875, 4, {5, 15, 5, 5}},
    {11, 1, {11, 0, 0, 0}},     {13, 1, {13, 0, 0, 0}},    {33, 2, {11, 3, 0, 0}},
    {39, 2, {13, 3, 0, 0}},     {55, 2, {11, 5, 0, 0}},    {65, 2, {13, 5, 0, 0}},
    {77, 2, {11, 7, 0, 0}},     {91, 2, {13, 7, 0, 0}},    {99, 2, {11, 9, 0, 0}},
    {117, 2, {13, 9, 0, 0}},    {121, 2, {11, 11, 0, 0}},  {143, 2, {13, 11, 0, 0}},
    {165, 3, {5, 11, 3, 0}},    {169, 2, {13, 13, 0, 0}},  {195, 3, {5, 13, 3, 0}},
    {231, 3, {7, 11, 3, 0}},    {273, 3, {7, 13, 3, 0}},   {297, 3, {9, 11, 3, 0}},
    {325, 3, {5, 13, 5, 0}},    {385, 3, {7, 11, 5, 0}},
};
// The lengths FFTGAL_FAST_GRID chooses from (the first entries of kFastSched).
constexpr int kNumGridLengths = 6;
// 3D passes are compiled for lengths up to kMaxFast3 and for the first six.
constexpr int kMaxFast3 = 405;
constexpr int kNumFast = sizeof(kFastSched) / sizeof(kFastSched[0]);
constexpr int fast_index(int n) {
    for (int i = 0; i < kNumFast; ++i)
        if (kFastSched[i].n == n) return i;
    return -1;
}
constexpr bool fast_dim(int fi, int d) { return d == 2 || fi < kNumGridLengths || kFastSched[fi].n <= kMaxFast3; }

// Device-resident state of one CG solve (Remark CG), advanced by the scalar
// kernels; every kernel of an iteration returns at once when `done` is set.
struct CgStatus {
    double rr;       // (r_k, r_k)
    double rr0;      // (r_0, r_0)
    double pq;       // (p_k, K p_k)
    double alpha;    // rr / pq
    double beta;     // rr_{k+1} / rr_k (0 before the first step)
    double tol2;     // rtol^2
    double floor2;   // (floor * ||A_M E||)^2
    double load2;    // ||A_M E||^2
    double energy;   // energy of the current iterate (CG recurrence)
    double dprev;    // energy decrease of the previous step
    double btol;     // bound tolerance (0: residual test only)
    // best-iterate guard of the FP32-iteration form: exact energies of the
    // iterate at checkpoints, the lowest one kept in a copy of the field
    double eAE;      // (A_M E, E): the energy of e = 0
    double ebest;    // lowest checkpoint energy (the initial iterate's at start)
    double rrmin;    // smallest (r_k, r_k) so far
    int32_t rrmin_it;  // iteration of rrmin
    int32_t best_it;   // iteration of the kept copy
    int32_t stagnated; // stopped because FP32 rounding stalled the iteration
    int32_t ck_copy;   // set by a checkpoint: copy the iterate into the best copy
    int32_t ck_restore;  // set by a checkpoint: restore the iterate from the best copy
    int32_t iter;
    int32_t maxit;
    int32_t done;
    int32_t converged;
    int32_t breakdown;
    int32_t pad;
};

enum Prologue { PRO_PLAIN = 0, PRO_EXPAND = 1 };
enum Epilogue { EPI_PLAIN = 0, EPI_PROJECT = 1, EPI_WINDOW = 2 };
enum RowMode { ROW_OPER = 0, ROW_RHS = 1, ROW_GRAM = 2, ROW_C2R = 3, ROW_R2C = 4 };
enum SolveKind { KIND_E = 0, KIND_J = 1 };

// A batched 1D DFT along one strided axis ("pencils"), with optional
// prologue/epilogue.  Element (component c, outer o, position l, batch b) of
// an operand lives at base + c*cs + o*os + l*ls + b (complex units).  Stored
// position l of a length-L operand holds frequency wrap_L(l) (or grid point l
// when L equals the transform length n), placed in the transform at
// wrap_L(l) mod n.
struct PencilArgs {
    const void *in;
    void *out;
    long in_cs, out_cs, in_os, out_os, in_ls, out_ls;
    int L_in, L_out;
    int nb;       // batch extent (contiguous)
    int B;        // pencils per work-group
    int ncomp;    // transformed components (per solution)
    int cb;       // generic kernel: components transformed together (1 .. ncomp)
    int twl;      // generic kernel: table entries staged in LDS (0: read from the table)
    int sgn;      // +1: inverse DFT (omega^{+mk}); -1: forward
    double scale; // applied to every output value
    FftDesc f;
    const void *tw;
    int pro, epi;
    int fast;     // set by configure_pencil: specialised kernel for this length
    // frequency decoding for EXPAND / PROJECT / WINDOW
    int d, kind, nc, Nmid, Nh;
    // EXPAND: state vectors (component stride st_cs, solution stride st_ss)
    const void *st_r;
    void *st_p;
    const void *st_x;
    long st_cs, st_ss;
    int nsol;
    int update_p;
    const CgStatus *status;
    // PROJECT
    void *st_q;
    const void *st_dot;
    double *partial;
    // WINDOW: sinc window of a P-voxel image, times 1/|P|
    int Pw[3];
    double winscale;
    // reduced Ga (Lemma reduce_grid): EXPAND multiplies frequency k by
    // exp(-i pi sum_a shift_a k_a / Nfull_a) (S(s)), PROJECT by its conjugate
    // (S*(s)) and, with accumulate, adds to the vector already in out
    int shift[3];
    int Nfull[3];
    int accumulate;
    // 3D gradient fields between axis 1 and axis 2 (see pencil_fast): EXPAND and
    // PROJECT passes of two components (ncomp = 2), and the axis-2 passes that
    // make three of them and two of three (grad = 1)
    int grad;
};

// Batched real transforms along the last (contiguous, half-spectrum) axis,
// two rows packed per complex transform, with the material multiply fused.
struct RowArgs {
    void *data;       // complex rows: comp stride cs, row stride Nh_row
    long cs;
    int nrows;
    int Nh_row;
    int n;
    FftDesc f;
    const void *tw;
    int ncomp;
    int d;
    int mode;
    int RP;           // row pairs per work-group
    int fast;         // set by configure_row (1 specialised, 2 specialised isotropic, 3 isotropic
                      // with all loads of a work-group staged in LDS)
    int iso;          // A0 and D are multiples of the identity
    const void *g;    // material field g (M^d, precision of the kernel)
    double A0[9];     // A(x) = A0 + g(x) D
    double D[9];
    // nfield > 1: A(x) is the symmetric matrix whose entries 11, 12, [13,] 22,
    // [23,] 33 are the fields g + f * gstride (f = 0 .. nfield - 1); A0 and D
    // are unused
    int nfield;
    long gstride;
    // ROW_GRAM, generic kernel: 1 packs two components of one row per complex
    // transform (RP rows per work-group) instead of two rows of one component
    // (RP row pairs), halving the transform buffers for long rows
    int gpack;
    // generic kernel: the components' rows form one batch of transforms (LDS
    // for two buffers of every component) instead of one batch per component
    int zbatch;
    int L2;           // > 0: nrows planes x1 of L2 axis-2 frequencies (plane_iso); nrows rows otherwise
    double E[3];      // load for ROW_RHS
    void *real_out;   // ROW_C2R output rows (length n)
    const void *real_in;  // ROW_R2C input rows (length n)
    long real_stride;
    int imgmap;       // ROW_R2C: voxel value mapping (see map_voxel)
    double vmax;
    double scale;
    double *partial;  // RHS: |A_M E|^2 sums; GRAM: d*d sums per work-group
    double *partial2; // RHS: sums of (A_M E).E per work-group (may be null)
    const CgStatus *status;
};

// Per-problem arguments of the multi-problem CG kernels.
struct UpdArgs {
    void *x;
    void *r;
    const void *p;
    const void *q;
    long n_per_comp;
    long cs;
    int nc;
    int Nh;
    int nblocks;  // work-groups of this problem (fixes the reduction order)
    CgStatus *st;
    double *partial;
    const double *pq_part;  // partials of (p, K p) from the projection pass, or nullptr
    int npq;
    // K p as the sum of nq vectors q, q + q_ss, ... (the shifts of the reduced
    // Ga, added in that order); nq = 1 otherwise
    int nq;
    long q_ss;
};

// One 2D CG solve run entirely by one work-group (launch_solo): the CG
// vectors x, r, p (nc = 1 component of N0 x Nh coefficients, half spectrum),
// the status, the material A(x) = A0 + g(x) D (nfield = 1) or the fields g +
// f gstride holding the entries 11, 12, 22 of A(x) (nfield = 3) on the M0 x M1
// grid, the stage twiddles of both axes (entries tw0, tw1 of tw), the basis
// kind and the scale 1 / (M0 M1) of the forward transforms.
constexpr int kSoloStages = 4;
struct SoloStage {  // of a length n known at run time: radix R, P, butterflies n / R, first twiddle
    int R, P, TQ, tw;
    unsigned mTQ, mP;  // multipliers of the divisions by TQ and P (solo_div)
};
struct SoloArgs {
    void *x, *r, *p;
    CgStatus *st;
    CgStatus *mirror;  // copy of the status at the end of a launch, or nullptr
    double *hist;      // (rr, alpha) per iteration, or nullptr
    int hist_cap;
    const void *g;
    long gstride;
    int nfield;
    double A0[4], D[4];
    const void *tw;
    int tw0, tw1;
    int M0, M1, N0, Nh;
    int kind;
    double scale;
    // the kernel of run-time lengths: the stages of both axes and the
    // multipliers of the divisions by Nh, by the 2 Nh - 1 non-zero columns
    int nst[2];
    SoloStage stg[2][kSoloStages];
    unsigned mNh, mNA;
};

struct CgItem {
    CgStatus *st;
    const double *rr_part;
    int nrr;
    double *hist;      // (rr, alpha) per iteration, or nullptr
    int hist_cap;      // entries available in hist
    CgStatus *mirror;  // copy of the status after each check, or nullptr
};

struct InclDev {
    int shape;
    double c[3];
    double h[3];
    double w;  // weight of this inclusion's indicator
};

// ---- launchers (fftgal_kernels.hip) ----
// GaNi material at the grid points x = k / M (centred): w0 + sum_i w_i chi_i(x)
// for inclusions (periodic minimum image; boundary points outside), and the
// mapped value of the voxel containing x for images (voxel p covers
// [p/P - 1/(2P), p/P + 1/(2P))).  Output layout [x1][x2][x3], FP64.
hipError_t launch_sample_incl(double *g, int d, const int *M, const InclDev *inc, int n, double w0, hipStream_t s);
hipError_t launch_sample_voxel(double *g, const double *img, int d, const int *P, const int *M, int map, double vmax,
                               hipStream_t s);
// Upper / lower voxel images of an inclusion composite (Remark adjusting_A):
// per voxel (centre p/P, sides 1/P) the largest / smallest eigenvalue of the
// phases meeting it with positive measure; ext = (hi, lo) of the matrix, then
// of each inclusion phase.
hipError_t launch_envelope(double *upper, double *lower, int d, const int *P, const InclDev *inc, int n,
                           const double *ext, hipStream_t s);
size_t pencil_lds_bytes(const PencilArgs &a, bool fp64);
size_t row_lds_bytes(const RowArgs &a, bool fp64);
// Choose pencils per work-group / row pairs per work-group (and whether the
// specialised kernel runs) for a launch; sets a.B / r.RP.
void configure_pencil(PencilArgs &a, bool fp64);
void configure_row(RowArgs &r, bool fp64);
// LDS of a generic-kernel work-group (its transform buffers): at most 80 KB,
// two work-groups per CU
constexpr size_t kGenericLds = 80 * 1024;
// Generic pencil kernel: the most components per transform batch (a.cb) whose
// buffers fit kGenericLds at the batch a.B, then a.twl > 0 when the
// transform's table fits beside them too.
void fit_pencil_components(PencilArgs &a, bool fp64);
// Generic row kernel: a.zbatch = 1 when the batched buffers fit kGenericLds at a.RP.
void fit_row_batch(RowArgs &r, bool fp64);
hipError_t launch_pencil(const PencilArgs &a, int nouter, bool fp64, hipStream_t s);
hipError_t launch_row(const RowArgs &a, bool fp64, hipStream_t s);
// Whether the 3D transforms of f have specialised passes (also for two components).
bool fast_pencils(const FftDesc &f, bool fp64);
int row_grid(const RowArgs &a);
int pencil_grid_x(const PencilArgs &a);

// Best-iterate checkpoint of an FP32 solve (between iterations, after the
// operator was applied to the iterate x with partials of (x, K x) in
// part_xkx): partials of (b, x) per update work-group, then the exact energy
// (A_M E, E) - 2 (b, x) + (x, K x) compared with the best one: a lower energy
// is copied into xbest; a clear rise, or no gain while the residual has not
// reached a new minimum for `window` iterations, stops the solve and restores
// x from xbest.  final = 1 (after the last iteration of a solve that did not
// converge) only restores x when the kept copy is better.  Every kernel does
// nothing when the solve is done, except in the final checkpoint.
hipError_t launch_cg_checkpoint(const UpdArgs &u, const void *b, void *xbest, const double *part_xkx, int n_xkx,
                                double *part_bx, int window, int final, bool fp64, hipStream_t s);
hipError_t launch_copy_vec(void *dst, const void *src, size_t bytes, hipStream_t s);
// Matrix voxel images (n voxels of d x d, row-major per voxel): per work-group
// counts of voxels that are not finite, symmetric and positive definite into
// part (one entry per work-group of the launch, nparts returned in *nparts).
hipError_t launch_tensor_check(const double *img, long n, int d, double *part, int *nparts, hipStream_t s);
// out[i] = entry (a, b) of voxel i's matrix, or of its inverse (invert = 1).
hipError_t launch_tensor_component(const double *img, long n, int d, int a, int b, int invert, double *out,
                                   hipStream_t s);
// Start of a solve from e_0 = 0: sums of the right-hand side's partials into the status.
struct InitArgs {
    CgStatus *st;
    const double *rr_part, *load_part, *work_part;
    int n_rr, n_load;
    double inv_mtot, tol, floor_rel, btol;
    int maxit;
    double *hist;
};
hipError_t launch_cg_init(const InitArgs &a, hipStream_t s);
hipError_t launch_cg_init_multi(const InitArgs *args, int np, hipStream_t s);
// Up to kVecOps copies (src set) or clears (src null) of word-aligned vectors in one launch.
constexpr int kVecOps = 24;
struct VecOps {
    struct Op {
        void *dst;
        const void *src;
        unsigned long long words;
    } op[kVecOps];
    int n = 0;
};
hipError_t launch_vec_ops(const VecOps &ops, hipStream_t s);
// Multi-problem launches: `args` and `woff` are device arrays; problem i
// owns work-groups [woff[i], woff[i + 1]) of a grid of `total` work-groups.
// Optional pair of events that a dispatch records itself at its start and at
// its end (hipExtLaunchKernel): the kernel's own duration, with no marker
// packets between launches.  Both null: an ordinary launch.
struct LaunchEv {
    hipEvent_t start = nullptr;
    hipEvent_t stop = nullptr;
};
// The specialised kernels of one length: launchers, pencils (row pairs,
// transforms) per work-group and LDS bytes, by precision (1: FP64) and
// dimension (d - 2); a null launcher means there is none.
struct FastKernels {
    struct Pencil {
        void (*fn)(const PencilArgs *, const int *, int np, int total, hipStream_t, LaunchEv) = nullptr;
        int B = 0;
        size_t lds = 0;
    };
    struct Row {
        void (*fn)(const RowArgs *, const int *, int np, int total, hipStream_t, LaunchEv) = nullptr;
        int RP = 0;
        int nh_max = 0;  // longest half-spectrum row it takes
        size_t lds = 0;
    };
    Pencil pencil[2][2];
    Pencil pencil2[2];  // 3D gradient fields: EXPAND and PROJECT of two components
    Row row[2][2];    // any material: RP row pairs
    Row iso[2][2];    // isotropic: RP transforms (row pair, component)
    Row pairs[2][2];  // isotropic: RP transforms of whole row pairs
    Row plane[2];     // isotropic, 3D: whole planes, axis 2 and rows
    Row gram[2];      // FP64 energy Gram: RP row pairs
    // Bluestein transforms through this convolution length
    Pencil blue_pencil[2][2];
    Pencil blue_pencil2[2];
    Row blue_row[2][2];  // isotropic: RP transforms, of whole row pairs or one
};
constexpr int kFastParts = 8;
template <int PART> void fill_fast(FastKernels *table);  // entries fi with fi % kFastParts == PART
const FastKernels &fast_kernels(int fi);
hipError_t launch_pencil_multi(const PencilArgs &proto, const PencilArgs *args, const int *woff, int np,
                               int total, bool fp64, hipStream_t s, LaunchEv ev = LaunchEv{});
// Whether plane_iso takes planes of L2 x nh frequencies on an f.n x f.n grid.
bool plane_fits(const FftDesc &f, int L2, int nh, bool fp64);
hipError_t launch_row_multi(const RowArgs &proto, const RowArgs *args, const int *woff, int np, int total,
                            bool fp64, hipStream_t s, LaunchEv ev = LaunchEv{});
hipError_t launch_cg_check_multi(const CgItem *items, int np, hipStream_t s, LaunchEv ev = LaunchEv{});
// Whether the 2D Ga grid of `a` (M0, M1, N0, Nh; axes transformed as f[0], f[1])
// has the single-work-group solver (3,5,7-smooth lengths, the complex grid
// within the LDS of one work-group); fills the stages of `a` when it does.
bool solo_fits(SoloArgs &a, const FftDesc *f, bool fp64);
// `niter` CG iterations (fewer once a solve is done) of each of the np solves
// in `args` (device array; all of one grid and precision), one work-group each.
hipError_t launch_solo(const SoloArgs &proto, const SoloArgs *args, int np, int niter, bool fp64, hipStream_t s,
                       LaunchEv ev = LaunchEv{});
hipError_t launch_cg_update_multi(const UpdArgs *ua, const int *woff, int np, int total, bool fp64,
                                  hipStream_t s, LaunchEv ev = LaunchEv{});
int pencil_grid(const PencilArgs &a, int nouter);  // work-groups of one problem
int update_blocks(long n);                         // work-groups of one CG update
hipError_t launch_fill_zero(void *p, size_t bytes, hipStream_t s);
// Warm start: r <- r - q (r holds b on entry), partials of (r, r), (b, x0),
// (r, x0) into part_rr / part_bx / part_rx (one per work-group, update grid).
hipError_t launch_warm_residual(const UpdArgs &u, double *part_rr, double *part_bx, double *part_rx, bool fp64,
                                hipStream_t s);
// Status of a warm-started solve: rr = sum part_rr, reference rr0 = scal[0]
// ((b, b)), load2 = scal[1], energy at the initial iterate
// scal[2] / mtot - sum part_bx - sum part_rx (history slot 1).
hipError_t launch_cg_init_warm(CgStatus *st, const double *part_rr, const double *part_bx, const double *part_rx,
                               int nparts, const double *scal, double mtot, double tol, double floor_rel, int maxit,
                               double btol, double *hist, hipStream_t s);
// Copy the coefficient arrays of a coarse solve into a fine one: entries of
// frequencies inside the coarse grid are copied, all others set to zero.
hipError_t launch_prolong(const void *src, bool src64, void *dst, bool dst64, int d, int nc, const int *Nf,
                          const int *Nc, hipStream_t s);
hipError_t launch_convert_f2d(double *dst, const float *src, size_t n, hipStream_t s);
hipError_t launch_convert_d2f(float *dst, const double *src, size_t n, hipStream_t s);
hipError_t launch_sum_partials(double *out, const double *part, int nparts, int nvals,
                               hipStream_t s);
hipError_t launch_image_stats(const double *img, long n, double *part, double *out, hipStream_t s);
// Reduced Ga material (Lemma reduce_grid): fold a Fourier half-grid on
// Z_{2N-1} (layout [L0][L1][Lh], wrapped) onto Z_N (layout [N0][N1][Nh]) with
// the phase of the shift s: b(j) = sum_{k = j mod N} c(k) exp(-i pi s.k / N).
hipError_t launch_fold_series(void *out, const void *coef, int d, const int *N, const int *L, int Lh,
                              const int *shift, hipStream_t s);
hipError_t launch_incl_coeff(void *out, int d, int L1, int L2, int Lh, const InclDev *incl, int n_incl,
                             double w0, hipStream_t s);

}  // namespace fftgal
