// Internal declarations shared by the C-ABI host code and the gfx950 kernels.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace cvp {

constexpr int kWave = 64;             // CDNA wavefront
constexpr int kBlock = 256;           // threads per workgroup
constexpr int kWaves = kBlock / kWave;
constexpr int kRecFloats = 12;        // floats per cut-piece record

// Backprojection LDS per view of a record pass: GW x PMAX piece records, the
// GW piece counts and the 4 window bounds; a record pass covers
// back_views_per_pass views (64 lanes over GW columns x min(PMAX, 64 / GW)
// slots each).
constexpr int back_rec_floats(int gw, int pmax) { return gw * pmax * kRecFloats + gw + 4; }
constexpr int back_views_per_pass(int gw, int pmax) { return 64 / (gw * (pmax < 64 / gw ? pmax : 64 / gw)); }
constexpr float kYQuantumInv = 1024.0f;
constexpr int kBackPasses = 2;        // most 64-voxel passes per backprojection stack
// the launches from a transposed copy (no window limits them): columns and
// most passes per stack
constexpr int kDirectCols = 4, kDirectPasses = 4;
constexpr int kPmaxWide = 64;         // pieces per column of the wide-footprint backprojection

// Projector models of launch_project / launch_backproject: the cutting voxel
// projector with r at the voxel centre or at each cut piece's centroid, and
// the TT separable-footprint projector on the same work split.
constexpr int kModelRelaxed = 0;
constexpr int kModelExact = 1;
constexpr int kModelTT = 2;

// Per-view source-centred frame (Sec. II-C) and intrinsics, FP64.  e1 and d
// have no x3 component (that is what makes chi1 independent of x3, the column
// identity of Sec. III-A); chi2 runs along -x3.  A projection matrix of the
// view is K [R | -R s] with rows of R e1, (0,0,-1), d and
// K = [[fb1, 0, c1], [0, fb2, c2], [0, 0, 1]] (Sec. III-C).
struct ViewGeom {
    double s1, s2, s3;   // source position
    double e1x, e1y;     // detector chi1 axis
    double dx, dy;       // principal ray direction
    double c1, c2;       // principal point (pixel-index units)
    double fb1, fb2;     // f / b1, f / b2
    double ifb2;         // b2 / f
};

// Everything a kernel needs about one problem.  Passed by value.
struct DevGeom {
    int n1, n2, n3;
    int M, N;            // detector columns (chi1), rows (chi2)
    int nviews;
    double a1, a2, a3;
    double x1lo, x2lo, x3lo;   // lower corner of the volume box
    double b1, b2, c1, c2, f;
    double fb1, fb2, b2f;      // f / b1, f / b2, b2 / f
    const ViewGeom *views;     // device; view q of a launch is views[q * vstride]
    int vstride;               // view stride: a launch may cover views v0, v0 + vstride, ... (views and
                               // the projection pointer start at v0; 1 for all views)
    const float *sigma;        // device pixel factors (nullptr: 1): [N][M], or [views][N][M] if sigma_views
    int sigma_views;           // 1: one factor table per view (views with their own intrinsics)
    int raw_volume;            // weight = cut volume (no 1/r^2)
    // Bounds on any pixel's weight sum per unit |mu| (with and without the
    // 1/r^2 factor), used to scale the projection's fixed-point sums.
    double wsum_bound, wsum_bound_raw;   // a pixel's summed weight per unit |mu|
    double wone_bound, wone_bound_raw;   // one (voxel, pixel) weight per unit |mu|
    // The geometry's cached piece records (nullptr: the kernels compute
    // their own): rtab[((t n2 + j) n1 + i) pmax + s][kRecFloats] and the
    // piece counts rtab_n[(t n2 + j) n1 + i] of column (i, j) in view q of
    // the launch, t = q * rtab_vs (from the launch's first view; rtab_vs is
    // the view stride for a geometry's whole table, 1 for a table made for
    // the launch), pieces clipped to the detector columns; rtab_pmax slots
    // per column.
    const float *rtab;
    const int *rtab_n;
    int rtab_pmax;
    int rtab_vs;
    int rpad;            // most rows of a straight-line (fixed row count) piece, and the spare rows its
                         // kernels keep beyond each detector edge (<= kFixedRowsMax)
};

// Fixed row counts: a piece whose chi2 extent with its elevation-correction
// margin is at most R - 1 rows touches at most R rows, and the kernels then
// evaluate R rows for every lane without a loop.  piece_record stores the
// count (0: none) above the detector column in the record's word 0, bits
// 16..19 with the elevation correction, 20..22 without.
constexpr int kFixedRowsMax = 6;

struct ProjLaunch {
    int U;           // detector columns per band
    int nbands;
    int items;       // nbands * nviews
    int chunk;       // work-item slots per XCD (grid = 8 * chunk)
    int linear;      // 1: work items in order over the whole GPU instead of bands by XCD
    int pmax;        // 4 or 8 (8 with U <= 8 for wider footprints)
    int pad;         // spare rows at each end of a band column (the geometry's rpad, or 0 if they do not fit)
    size_t lds;      // dynamic LDS bytes
};

struct BackLaunch {
    int gw;          // columns per group (16, 8 or 4)
    int ngroups;     // groups per row (ceil(n1 / gw))
    int kp;          // 64-voxel passes per stack (1 or 2)
    int nkchunks;    // ceil(n3 / (64 * kp))
    int items;
    int chunk;
    int pmax;        // 4, 8 or kPmaxWide (then gw = 4)
    int win_cap;     // floats per wave window
    size_t lds;
    int wpc;         // workgroups per CU the LDS budget was sized for
    int shared;      // 1: one detector window per workgroup (cached records only)
};

// A backprojection from a transposed copy of the projections: stacks of
// kDirectCols columns x 64 kp slices.
struct DirectLaunch {
    int kp;
    int ngroups, nkchunks;
    int items;
    int pmax;        // 4 or 8
};

// The transposed, scaled projections of a launch's views (with `pad` zero
// rows on both sides) and the flags of their non-finite blocks.
struct BackCopy {
    float *pt = nullptr;
    int *bad = nullptr;
    int pad = 0;
};

// Batched, persistent launches over up to kMaxBatch problems.
constexpr int kMaxBatch = 32;

struct BatchProblem {        // device table entry (one per problem)
    DevGeom G;
    int U;                   // projection band width
    int pitems;              // projection work items
    int pad;                 // spare rows of a band column
    int pmax;                // the problem's projection piece stride (its own plan),
    int gw;                  // the batch's backprojection stack width,
    int kp;                  // passes per stack
    int win_cap;             // and per-wave window (floats)
    int ngroups;             // backprojection column groups per row
    int nkchunks;
    int bitems;              // backprojection work items
    const float *in;         // set per call by batch_setup
    float *out;
    unsigned *gmax;          // the problem's per-group maxima (owned by the batch)
    float *vt;               // its transposed volume (owned by the batch), or nullptr
    DirectLaunch direct;     // backprojection from its transposed copy (owned by the batch),
    BackCopy copy;           // where the batch has copies
    const double *stop;      // set per call: the problem's work items are skipped while *stop != 0
};

struct BatchTable {          // device: work segments, largest items first
    int n;
    int start[kMaxBatch + 1];
    int order[kMaxBatch];
};

struct BatchIO {             // per call, by value
    int n;
    int raw;
    const float *in[kMaxBatch];
    float *out[kMaxBatch];
    const float *sigma[kMaxBatch];
    const double *stop[kMaxBatch];   // per problem, or nullptr
};

// gw, pmax: the backprojection launch's stack width (16, 8 or 4; 0: from the
// transposed copies, with cached only) and piece stride (4 or 8); cached: the
// kernels read tables of records; vt: the projection reads the members'
// transposed volumes
hipError_t launch_batched(bool backward, BatchProblem *probs, const BatchTable *tab, int *counter,
                          const BatchIO &io, bool exact, bool ec, int grid, size_t lds, int gw, int pmax, bool cached,
                          bool vt, hipStream_t s);
int batched_blocks_per_cu(bool backward, size_t lds, int gw, int pmax, bool cached, bool vt);
size_t project_lds_bytes(int U, int N, int n2, int pmax);
size_t backproject_lds_bytes(int gw, int pmax, int winCap);

// CGLS workspace (FP64): scalars, then the |s|^2 and |r|^2 histories, then the
// reduction partials.
// Scalars: [0] gamma [1] |q|^2 [2] alpha [3] beta [4] gamma0 [5] |r|^2 [6] k
// [7] breakdown [8] stop flag [9] gamma threshold of the stop (0: none)
// [10] tol^2 and [11] reference gamma (0: gamma0) set by cvp_cgls_set_tolerance
constexpr int kCglsScalars = 16;
constexpr int kCglsStop = 8, kCglsThr = 9, kCglsTol2 = 10, kCglsRef = 11;
constexpr int kCglsHistory = 4096;
constexpr int kCglsPartials = 1024;
constexpr int64_t kCglsWorkDoubles = kCglsScalars + 2 * kCglsHistory + kCglsPartials;

// LSQR workspace (FP64): scalars, then the |r| and |A^T r| estimate
// histories, then the reduction partials.
enum : int {
    kLsqrAlpha = 0, kLsqrBeta = 1, kLsqrRhobar = 2, kLsqrPhibar = 3, kLsqrXStep = 4, kLsqrWStep = 5,
    kLsqrK = 6, kLsqrBreak = 7, kLsqrArnorm0 = 8, kLsqrScalars = 16
};
enum : int { kLsqrFinBeta0 = 0, kLsqrFinAlpha0 = 1, kLsqrFinBeta = 2, kLsqrFinAlpha = 3 };
constexpr int64_t kLsqrWorkDoubles = kLsqrScalars + 2 * kCglsHistory + kCglsPartials;

hipError_t blas_fill(float *p, int64_t n, float val, hipStream_t s);
hipError_t sart_residual_views(float *q, const float *b, const float *R, int64_t nm, int count, int64_t view_step,
                               hipStream_t s);
hipError_t sart_update_x(float *x, const float *z, const float *C, int64_t n, float lam, int nonneg, hipStream_t s);
hipError_t lsqr_axpby_norm(float *y, const float *x, int64_t n, double *sc, int ci, int mode, hipStream_t s);
hipError_t lsqr_norm(const float *a, int64_t n, double *sc, int mode, hipStream_t s);
hipError_t lsqr_scale(float *y, int64_t n, const double *sc, int ci, hipStream_t s);
hipError_t lsqr_update_vxw(float *v, float *x, float *w, int64_t n, const double *sc, int init, hipStream_t s);
// stop: optional device flag; a kernel returns at once while *stop != 0 (a
// converged CGLS keeps its state through the rest of a captured graph).
hipError_t blas_dot(const float *a, const float *b, int64_t n, double *partials, double *sc,
                    int mode, double *out, hipStream_t s, const double *stop = nullptr);
hipError_t blas_update_xr(float *x, const float *p, int64_t nv, float *r, const float *q, int64_t np,
                          double *sc, double *partials, hipStream_t s, const double *stop = nullptr);
hipError_t blas_update_p(float *p, const float *sv, int64_t n, const double *sc, int init,
                         hipStream_t s, const double *stop = nullptr);
hipError_t blas_set_tolerance(double *sc, double tol2, double ref, hipStream_t s);
hipError_t blas_residual(float *r, const float *b, const float *q, int64_t n, hipStream_t s);

// gmax: the per-group maxima of |vol| (launch_group_max or
// launch_transpose_max), or nullptr (the kernel scans the wedges).  vt: with
// gmax, the transposed volume (launch_transpose_max) that the kernel then
// reads, or nullptr (it reads vol).  The same bits in every case.
hipError_t launch_project(const DevGeom &g, const ProjLaunch &L, int model, bool ec,
                          const float *vol, float *proj, const unsigned *gmax, const float *vt, hipStream_t stream,
                          const double *stop = nullptr);
hipError_t launch_transpose_max(const DevGeom &g, const float *vol, float *vt, unsigned *gmax, hipStream_t stream,
                                const double *stop = nullptr);
int64_t group_max_cells(const DevGeom &g);
hipError_t launch_group_max(const DevGeom &g, const float *vol, unsigned *gmax, hipStream_t stream,
                            const double *stop = nullptr);
// Allocation-free projection: device address (on the current device) of the
// library's fixed scratch array for the per-group maxima, looked up once per
// device; kStaticScratchWords words (1 MiB).
constexpr int64_t kStaticScratchWords = int64_t(1) << 18;
hipError_t static_scratch(unsigned **out);
// SiddonK reference projector: K x K rays per pixel, exact chord lengths.
hipError_t launch_siddon(const DevGeom &g, int K, const float *vol, float *proj, hipStream_t s);
// Fills the record table of g's views (every column; pmax 4 or 8; tt: TT
// footprints).
hipError_t launch_record_table(const DevGeom &g, int pmax, bool tt, float *rec, int *cnt, hipStream_t stream,
                               const double *stop = nullptr);
// part: the sums of a backprojection taken over several launches, each over
// the next views of it (a multiple of kWaves views in all but the last):
// back_part_floats(L) floats, read unless this is the first launch, written
// (and vol left alone) unless it is the last.  The sums are then the bits of
// one launch over all views.
struct BackPart {
    float *sums = nullptr;
    bool first = true, last = true;
};
constexpr int64_t copy_floats(const DevGeom &g, int64_t views) { return views * g.M * (g.N + 2 * (int64_t)g.rpad); }
constexpr int64_t copy_flags(const DevGeom &g, int64_t views) { return views * ((g.M + kWave - 1) / kWave); }
// LDS of backproject_direct_kernel: the waves' records, or their sums at the end
constexpr size_t back_direct_lds(int pmax)
{
    const size_t rec = (size_t)kWaves * back_views_per_pass(kDirectCols, pmax) * back_rec_floats(kDirectCols, pmax);
    const size_t red = (size_t)kWaves * kDirectCols * kWave;
    return 4 * (rec > red ? rec : red);
}
hipError_t launch_transpose_projections(const DevGeom &g, const float *proj, const BackCopy &copy, hipStream_t stream,
                                        const double *stop = nullptr);
// From the copy and a table of records.
hipError_t launch_backproject_direct(const DevGeom &g, const DirectLaunch &L, int model, bool ec, const BackCopy &copy,
                                     float *vol, hipStream_t stream, const double *stop, const BackPart &part);
constexpr int64_t back_part_floats(const DirectLaunch &L)
{
    return (int64_t)L.items * kWaves * kDirectPasses * kDirectCols * kWave;
}
hipError_t launch_backproject(const DevGeom &g, const BackLaunch &L, int model, bool ec,
                              const float *proj, float *vol, hipStream_t stream, const double *stop = nullptr);

}  // namespace cvp
