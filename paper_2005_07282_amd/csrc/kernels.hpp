// Host-visible declarations shared by the kernel translation unit and the
// C-ABI implementation: device-side state records, workspace descriptors and
// the launch functions (each kernel is launched only from its own .hip file).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace rpcg {

enum Mode { MODE_PLAIN = 0, MODE_FPE = 1, MODE_EXBLAS = 2 };

// Flag bits collected on the device.
enum {
    FLAG_NONFINITE = 1, // inf/NaN input, overflowing product or overflowing expansion
    FLAG_INEXACT = 2,   // a nonzero product below 2^-969 (TwoProd error not representable)
    FLAG_NOT_SPD = 4,   // missing or non-positive diagonal entry
};

constexpr int MAX_BLOCK = 1024;
constexpr int MAX_WAVES = MAX_BLOCK / 64;
constexpr int MAX_FPE = 8;
constexpr int NUM_XCDS = 8; // accelerator dies, each with its own L2; workgroups are dealt to them round-robin
constexpr int ACC_WORDS = 68; // same as ACC_DIGITS in numerics.hpp

// Workspace of one of the solvers' dots.
struct DotWs {
    double *part;   // [workgroups] partial sums (plain)
    long long *acc; // [DOT_COPIES][DOT_PITCH] accumulators the workgroups add to (exact modes)
};

// Slots of the exact partials of up to `gmax` workgroups.
struct SlotWs {
    long long *digits; // [ACC_WORDS][gmax] workgroup accumulator words, word-major
    int *range;        // [gmax][2] nonzero word range of each workgroup accumulator
};

// The solvers' exact dots: workgroups add the words of their
// accumulators into one of DOT_COPIES copies (integers, any order), the next
// kernel sums the copies. Eight copies keep the adds to one address few
// enough to drain with the kernel; the escape count sits behind the words of copy 0.
constexpr int DOT_COPIES = 8, DOT_PITCH = 72, DOT_ESC = 70;

// Scalars of a matrix copy's construction (device memory).
struct DotInfo {
    int varying;         // slices whose first entries show that their values vary (see launch_row_widths)
    int flags;
    int max_len;         // longest row (SELL construction scratch)
    int pad1;
    long long max_delta; // column-code range (SELL construction scratch)
    // construction scratch of the diagonal-aligned copy
    int diag_fail;                // nonzero: the rows do not line up, or too many slices need stored values
    int diag_stored;              // slices that need stored values, counted where there may be too many
    unsigned long long diag_total;  // entry records of all slices
    unsigned long long diag_values; // those whose values must be stored
};

// PCG state on the device. Written only by the last workgroup of a kernel
// (or by a single thread of the setup), read by every workgroup of later
// kernels.
struct PcgState {
    double beta;   // beta of the current iteration (Fig. 2)
    double rho;    // rho = beta / <d, w>
    double gamma;  // beta_new / beta_old
    double tau;    // <r, r>
    double thr;    // RN(RN(tol*tol) * <b,b>)
    double delta;  // <d, w>
    double bb;     // <b, b>
    double tau0;
    int iter;      // iterations completed (L)
    int done;      // nonzero: every later kernel is a no-op
    int status;    // rpcg status code
    int maxit;
    int flags;
    int ended;     // the first iteration whose x update (S3) is not owed once the solve has
                   // ended (0 at setup, l at a breakdown in iteration l, l + 1 when the
                   // stopping test of iteration l stops); INT_MAX while running
    int it_cur;    // batched solves: iterations completed, as the kernels of the current
                   // iteration see it (committed by the SpMV kernel from iter)
    int pad2;
    double beta_par[2]; // batched solves: beta of iteration j in beta_par[j & 1]
    long long escapes;
    long long fallbacks;
};

// Sliced-ELL copy of the matrix with slice height 64 (one wavefront) and
// V-entry interleave: entry k of row 64*s + j sits at
//     off[s] + 64*V*(k/V) + V*j + (k%V),
// so lane j reads V consecutive entries of its row with one vector load while
// each load of the wavefront is one contiguous segment. The slice width is
// its longest row; when it is not a multiple of V (V = 2, odd width w) the
// last entry k = w-1 sits alone at off[s] + 64*(w-1) + j, so an odd row
// length costs no padding entry. Rows keep their CSR order and length;
// padding entries hold the value 0 and a valid column. T is the type the solver computes in and V
// = sell_vec<T>() (two for binary64: 16-byte loads; one for binary32).
//
// Columns: with col16 (16-bit column codes), the column of rank 0 of row
// i = 64 s + j is min(i, n-1) + cfirst[s] + (signed) code, and the column of
// rank k >= 1 is the column of rank k-1 plus the (unsigned) code: rows keep
// ascending columns in 16-bit steps and cfirst[s] is the first-column offset
// of the slice's longest row. Padding codes are 0 (the column repeats), and
// rows without entries get a rank-0 code that lands on a valid column.
// Otherwise col holds the columns as 32-bit indices. val64 optionally holds
// the caller's binary64 values in the same layout (used by the refinement's
// residual next to binary32 val).
#ifndef RPCG_SELL_VEC64
#define RPCG_SELL_VEC64 2
#endif
template <typename T>
__host__ __device__ constexpr int sell_vec()
{
    return sizeof(T) == 8 ? RPCG_SELL_VEC64 : 1;
}

// Diagonal-aligned slices of 128 rows: the layout of operators whose rows share
// their column offsets (stencils, bands), used instead of the columns above
// when the rows of the slices line up. The entries of a slice's rows are
// merged by offset = column - row into records; a record holds the offset and
// the masks of the rows that have an entry there (lane j owns the rows 2 j and
// 2 j + 1: mask[0] and mask[1]), in an order that keeps every row's storage order. So a
// row's columns cost no memory traffic, its gathers are contiguous runs, and a slice
// whose entries agree along every record (a constant-coefficient operator) stores one
// value per record and none per row; other slices store the values of record k
// of row 2 j + r at vpos + 128 k + 2 j + r. The records are followed by at least
// 16 empty ones (empty masks, offset 0), so a loop may read whole batches.
constexpr int DIAG_ROWS = 128;
struct DiagEnt {
    double v;                   // constant slices: the value,
    unsigned long long mask[2]; // rows with an entry
    int off;                    // column - row
    float vf;                   // and the value rounded to binary32
};
struct DiagSlice {
    long long mpos; // first record
    long long vpos; // first value (slices that are not constant)
    int width;      // records
    int flags;
};
enum {
    DIAG_CONST = 1, // one value per record
    DIAG_CLAMP = 2, // masked-out rows may point outside the vector
    DIAG_TRI = 4,   // records 3 q, 3 q + 1, 3 q + 2 sit at neighbouring offsets
};
// Records per batch of loads: a 7-point row is one batch, a 27-point row three
// (in runs of three neighbours).
constexpr int DIAG_BATCH = 7, DIAG_TRI_BATCH = 9;
constexpr int DIAG_PAD = 24; // empty records after a slice's own
// Records of slice s start here (w64: 64 times the widths, that is the longest
// rows, of the 64-row slices before it): room for the widths of its two
// 64-row slices and a few more, and the empty records.
__host__ __device__ constexpr long long diag_mpos(long long w64, long long s) { return (w64 >> 6) + (DIAG_PAD + 8) * s; }
// Kept while the values that must be stored stay within 1.25 times the
// entries (8 bytes against 10 an entry in the general copy) and the records
// within twice.
__host__ constexpr bool diag_worth_it(unsigned long long records, unsigned long long values, long long nnz)
{
    return 4 * DIAG_ROWS * values <= 5 * (unsigned long long)nnz && DIAG_ROWS * records <= 2 * (unsigned long long)nnz;
}
// The rows that an aligned copy is tried for: those of a matrix wider than twice its
// longest row (nearly every slice of others is at an end, where the gathers are clamped one by
// one: binary32 solver, 1000 rows, constant band of 1001 67 us an iteration
// in general slices, 77 us aligned), none longer than DIAG_MAX_ROW (the merge
// walks a row entry by entry).
constexpr int DIAG_MAX_ROW = 1024;
__host__ constexpr bool diag_to_try(int n, int max_len) { return max_len > 0 && max_len <= DIAG_MAX_ROW && 2ll * max_len <= n; }
// Slices (of all nslices) whose values may have to be stored, or DIAG_ANY. Two rows a lane
// give stored values half the wavefronts of the general copy, each with one
// batch of loads in flight: less HBM traffic, but more latency, and up to five slices
// a CU it is latency that counts (prepared product, general and aligned, us: 20 k rows of 31
// 4.5 and 7.3, of 201 16.6 and 33.6; 100 k rows of 21 6.1 and 7.3, of 101 20.8 and
// 27.9; 150 k rows 9.3 and 9.2, 32.6 and 36.0; 200 k rows 10.6 and 8.1, 39.4 and 28.9; 512 k rows of 27
// 28.2 and 19.3). Rows of one batch only cross at half of that (solves of 7-point operators: 64 k
// rows 2.38 and 2.55 ms; factored, 85 k rows 2.94 and 2.90 ms, 157 k rows 4.57 and 4.43 ms). A few
// stored slices among constant ones, which are faster aligned at any size, do no harm.
constexpr int DIAG_ANY = 2147483647;
__host__ constexpr bool diag_few(long long nslices, int num_cus) { return nslices < 5ll * num_cus; }
__host__ constexpr int diag_max_stored(long long nslices, int max_len, int num_cus)
{
    const bool enough = !diag_few(max_len <= DIAG_BATCH ? 2 * nslices : nslices, num_cus);
    return enough ? DIAG_ANY : (int)(nslices / 16);
}
constexpr int DIAG_TABLE = 8192; // hash slots of record lists, a power of two (see k_diag_share)

// A CSR matrix whose slices of 64 rows start at slice0.
template <typename TIN>
struct DiagCsr {
    const int *rp, *col;
    const TIN *val;
    int n, nnz;
    long long slice0;
};

// Column layouts of the solvers' matrix copies.
enum { LAY_COL32 = 0, LAY_COL16 = 1, LAY_DIAG = 2 };

template <typename T>
struct SellMat {
    int n;
    int nslices;          // of the layout: 64 rows, diagonal-aligned 128
    const long long *off; // [nslices + 1]
    const T *val;
    const int *col;
    const int *row_ptr;   // the caller's CSR row pointers (row lengths)
    const unsigned char *len8; // row lengths as bytes when every row has < 256 entries, else null
    const unsigned short *col16; // when non-null: column codes (col unused)
    const int *cfirst;    // with col16: [nslices] first-column offset of each slice
    const double *val64;  // optional binary64 values (same layout), else null
    const DiagSlice *ds;  // when non-null: diagonal-aligned slices (off, col, col16, cfirst, len8 unused)
    const DiagEnt *de;

    int layout() const { return ds ? LAY_DIAG : (col16 ? LAY_COL16 : LAY_COL32); }
};

struct LaunchCfg {
    int grid;
    int block;
    bool early_exit;
    int fpe_size;
    bool fallback;
    int xcd_parts; // SpMV: number of contiguous slice ranges (one per XCD), 0 = by the layout
    hipStream_t stream;
};

// ---- launch functions (return hipError_t of the launch) ----
// `stride` is the slot capacity of a SlotWs.

// Workspace of one standalone dot call.
struct ExdotWs {
    long long *blk;          // DOT_COPIES x DOT_PITCH words, all zero; left so
    double *part;            // [grid] (plain)
    unsigned long long *rec; // optional: the call's record (escapes; seq << 32 | flags), host-visible or device memory
    unsigned seq;
};
hipError_t launch_exdot(int mode, long long n, const double *x, const double *y, double *out, const ExdotWs &w,
                        const LaunchCfg &cfg);
hipError_t launch_exdot_partial(long long n, const double *x, const double *y, long long *digits, const ExdotWs &w,
                                const LaunchCfg &cfg);
hipError_t launch_acc_round(const long long *digits, double *out, hipStream_t s);
// Exponent range (floor(log2 |v|)) of the nonzero finite entries of v, merged into *emin, *emax.
hipError_t launch_exp_range(long long n, const double *v, int *emin, int *emax, hipStream_t s);
// CSR SpMV (nnz = row_ptr[n]): workgroups of 64 to 512 rows by the number that
// n leaves for num_cus CUs; the staging chunk is chosen by the average row length.
hipError_t launch_spmv_csr(int n, long long nnz, const int *row_ptr, const int *col, const double *val,
                           const double *x, double *y, int num_cus, hipStream_t s);

// Slice widths (longest row of each 64 rows) into w, longest row, and the
// check of row_ptr (info->flags set if malformed), of one matrix (slice0 = 0) or, with
// nmats > 1, of all in mats (device memory, in order, each from an even slice0 on); rows past a matrix's
// last are empty. table (DIAG_TABLE ints) is set to -1. sample (for diag_few): info->varying, a lower bound for twice the 128-row slices whose values vary.
template <typename TIN>
hipError_t launch_row_widths(const DiagCsr<TIN> &one, const DiagCsr<TIN> *mats, int nmats, int nslices, bool sample, int *w,
                             int *table, DotInfo *info, hipStream_t s);
// out[j stride] = 64 sum(len[0..j)), j < m (and j = m with `total`).
hipError_t launch_scan_len(const int *len, int m, long long *out, int stride, bool total, hipStream_t s);
// CSR structural check (*bad set if malformed), longest row, and the range of
// the 16-bit column codes (*max_delta <= 32767 iff every code fits), one
// wavefront per 64-row slice.
hipError_t launch_csr_scan(int n, int nnz, const int *row_ptr, const int *col, int *bad, int *max_len,
                           long long *max_delta, hipStream_t s);
// Diagonal-aligned slices (nslices of 128 rows in all) from CSRs whose row_ptr have been
// checked, matrices as above: the merge (records, DiagSlice without vpos, ulen, column check,
// totals or diag_fail in info; max_stored: slices whose values may vary, else
// diag_fail; off: 64 times the widths of the 64-row slices before; table: as
// launch_row_widths leaves it), the sharing of equal record lists (over all matrices),
// and the stored values of the slices that need them.
template <typename TIN>
hipError_t launch_diag_align(const DiagCsr<TIN> &one, const DiagCsr<TIN> *mats, int nmats, int nslices, const long long *off,
                             DiagEnt *de, DiagSlice *ds, int *ulen, int *table, DotInfo *info, int max_stored, int num_cus,
                             hipStream_t s);
hipError_t launch_diag_share(int nslices, const DiagEnt *de, DiagSlice *ds, const int *table, hipStream_t s);
template <typename TIN>
hipError_t launch_diag_fill(const DiagCsr<TIN> &one, const DiagCsr<TIN> *mats, int nmats, int nslices, const DiagEnt *de,
                            const DiagSlice *ds, double *sval64, float *sval32, hipStream_t s);

// Fill the sliced-ELL arrays from the CSR. The source values are binary64
// (val64_in) or binary32 (val32_in, exactly one of the two non-null); sval64
// receives them as binary64, sval32 rounded to nearest binary32; either
// output may be null.
hipError_t launch_sell_fill(int n, const int *row_ptr, const int *col, const double *val64_in,
                            const float *val32_in, int vec, const long long *off, double *sval64, float *sval32,
                            int *scol, unsigned short *scol16, int *cfirst, unsigned char *len8, hipStream_t s);
// y = A x on a binary64 copy (grid workgroups of `waves` wavefronts, at most four).
hipError_t launch_sell_spmv(const SellMat<double> &A, const double *x, double *y, int grid, int waves, hipStream_t s);

template <typename T>
struct PcgVecs {
    const T *b;
    T *x, *r, *z, *d, *w, *dinv;
    double *hist;      // optional [maxit + 1]: tau history (widened to binary64)
    double *beta_hist; // [maxit + 1]: beta of every iteration (widened to binary64)
};

// The PCG launchers exist for T = double (the paper's solver) and T = float
// (the binary32 inner solver of the mixed-precision refinement). Scalars in
// PcgState are held as binary64; binary32 values widen to it exactly.

// Setup (state init, partials, one-workgroup finalize) into ws3[0..2], which it leaves empty.
template <typename T>
hipError_t launch_pcg_setup(int mode, const SellMat<T> &A, const PcgVecs<T> &v, PcgState *st, const DotWs *ws3,
                            double tol, int maxit, const LaunchCfg &cfg);
// Iteration l: K1 adds <d,w> to ws3[0]; K2 merges it (from Gd workgroups) and
// adds <z,r> to ws3[1] and <r,r> to ws3[2]; K3 merges those (from G
// workgroups). Each dot is emptied by the kernel after the one that reads it
// (K3 empties ws3[0], K1 the others).
template <typename T>
hipError_t launch_pcg_spmv_dot(int mode, const SellMat<T> &A, const PcgVecs<T> &v, PcgState *st, const DotWs *ws3,
                               const LaunchCfg &cfg);
template <typename T>
hipError_t launch_pcg_update(int mode, int l, int n, const PcgVecs<T> &v, PcgState *st, const DotWs *ws3, int Gd,
                             const LaunchCfg &cfg);
// s3: also apply the iterate update of iteration l (the Jacobi solver; the
// factored solver's update kernel applies it itself).
template <typename T>
hipError_t launch_pcg_direction(int mode, int l, int n, const PcgVecs<T> &v, PcgState *st, const DotWs *ws3, int G,
                                const LaunchCfg &cfg, bool s3);

// ---- mixed-precision refinement (binary64 outer loop) ----

// Outer-loop state on the device.
struct IrState {
    double rr;      // <r, r> of the current outer step (exact, rounded once)
    double bb;      // <b, b>
    double thr;     // RN(RN(tol*tol) * <b,b>)
    int k;          // outer step whose residual was last formed
    int stop;       // nonzero: converged, out of outer steps or failed
    int status;     // outer status (rpcg codes)
    int scale;      // s of the current correction: inner rhs = RN32(r 2^-s)
    int flags;
    int pad;
    long long escapes;
};

// r = RN(b - A x) with every row summed exactly (binary64 values A.val64 of
// the sliced-ELL copy), and the workgroup partials of <r, r> into ws (exact
// dot, expansion length 3).
hipError_t launch_ir_residual(const SellMat<float> &A, const double *b, const double *x, double *r, IrState *ist,
                              const SlotWs &ws, int stride, const LaunchCfg &cfg);
// Merge <r, r> (G slots), record rr_hist[k], decide whether to stop, and for
// a further correction the inner right-hand side rf = RN32(r 2^-s) and c = 0.
hipError_t launch_ir_prepare(int k, int maxit, double tol, int n, const double *r, float *rf, float *c,
                             double *rr_hist, IrState *ist, const SlotWs &ws, int G, int stride, const LaunchCfg &cfg);
// x = RN(x + c 2^s).
hipError_t launch_ir_update(int n, double *x, const float *c, const IrState *ist, const LaunchCfg &cfg);


// ---- PCG with a factored preconditioner M^-1 = G G^T + eps I ----

// G and G^T as CSR (device arrays), both n x n.
struct FacPre {
    const int *g_rp, *g_col;
    const double *g_val;
    const int *gt_rp, *gt_col;
    const double *gt_val;
    double eps;
};

// Setup: r = b - A x0, <r,r> (ws3[1]) and <b,b> (ws3[2]); t = G^T r;
// z = G t + eps r, d = z, <z,r> (ws3[0]); merge of the three, left empty.
// Every step that adds to a dot runs on cfg.grid workgroups.
hipError_t launch_fac_setup(int mode, const SellMat<double> &A, const FacPre &P, const PcgVecs<double> &v, double *t,
                            PcgState *st, const DotWs *ws3, double tol, int maxit, const LaunchCfg &cfg);
// Iteration l after the SpMV kernel (<d,w> in ws3[0], from Gd workgroups), two
// launches: merge delta, rho; x update; r update read from v.r and written to
// r_new (the caller alternates the two buffers), <r,r> added to ws3[2],
// t = G^T r; then z = G t + eps r with <z,r> added to ws3[1]. The direction
// kernel then merges those as in the Jacobi solver.
hipError_t launch_fac_update(int mode, int l, int n, const FacPre &P, const PcgVecs<double> &v, double *r_new,
                             double *t, PcgState *st, const DotWs *ws3, int Gd, const LaunchCfg &cfg);

// ---- batched solves (many independent systems per launch) ----

// Per-system constants of a batch. Rows of system s sit at [row0, row0 + n)
// of the concatenated vectors, its slices at [slice0, slice0 + nslices) of
// the concatenated sliced-ELL copy (slices never span systems), and its runs
// are numbered slot0, ..., slot1 - 1.
struct BatchSys {
    long long row0;   // multiple of 128
    long long slice0; // row0 / 64
    int n;
    int nslices;      // 64-row slices
    int slot0;
    int slot1;
    const int *row_ptr; // the caller's CSR row pointers of the system
    long long acc0;     // first word of its dots' accumulators
    long long copies;   // copies of each (see batch_copies)
};

// Accumulator copies of a system's dots: one per run that its size allows at a time
// (runs have 16 slices on average, or more, but for hand-set tiles). Eight for every system made
// batches of thousands of small ones clear and read more accumulators than
// vectors (4096 systems of 64 rows 200 us an iteration and 13.8 KB a system, now
// 179 us with the same schedule and 1.7 KB; 20 000 of 27 rows 658 and 553 us).
__host__ constexpr int batch_copies(int nslices)
{
    const int c = (nslices + 15) / 16;
    return c < 1 ? 1 : (c < DOT_COPIES ? c : DOT_COPIES);
}

// One run of work: slices [s0, s1) of system `sys`, processed by one
// workgroup, number `slot` of all runs (those of a system are consecutive).
struct BatchRun {
    int sys;
    int s0;
    int s1;
    int slot;
};

struct BatchArgs {
    int nsys;
    const BatchSys *sys;
    const BatchRun *runs;  // runs of workgroup g: [wg_run[g], wg_run[g + 1])
    const int *wg_run;
    // concatenated sliced-ELL copy (binary64 values, two-entry interleave)
    const long long *off;
    const double *val;
    const int *col;
    const unsigned short *col16;
    const int *cfirst;
    const unsigned char *len8; // indexed by concatenated row
    const DiagSlice *ds;       // when non-null: diagonal-aligned slices (all systems)
    const DiagEnt *de;
    // concatenated vectors
    const double *b;
    double *x, *r, *z, *d, *w, *dinv;
    PcgState *st;          // [nsys]
    long long *acc;        // accumulators of the systems' dots: [3][copies][DOT_PITCH] from acc0 on
    double *part;          // [3][part_cap] workgroup sums (plain), by slot
    int part_cap;
    double *const *hist;   // [nsys] tau histories (maxit + 1 each, entries may be null), or null
    int *active;           // number of systems not done
};

// Setup of every system (state, <z,r>, <r,r>, <b,b>, one workgroup per system
// to merge them; the dots are left empty).
hipError_t launch_batch_setup(int mode, int layout, const BatchArgs &a, int grid, int block, double tol, int maxit,
                              const LaunchCfg &cfg);
// One iteration of every system not done: SpMV + <d,w> (dot 0), per-system
// rho, updates + <z,r>, <r,r> (dots 1, 2), per-system stopping test and gamma,
// iterate and direction update. Emptied as in the single solver.
hipError_t launch_batch_iteration(int mode, int layout, const BatchArgs &a, int grid, int block, const LaunchCfg &cfg);

} // namespace rpcg
