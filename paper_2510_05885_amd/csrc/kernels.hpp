// kernels.hpp — device-side plan and launchers of the KKT factor/solve kernels.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

#include "plan.hpp"


namespace ncl {

constexpr int kNrhsMax = 16;   // columns per solve sweep (wider solves are chunked)
// Columns from which sweeps and residuals take kNrhsMax at a time.  That costs the same
// for any number of them (a solve at order 100k 1240 us, at 500k 3140, with one column 552
// and 1392), so two go one by one: 1062 and 2733 us; three would take 1600 and 4100.
constexpr int kManyColumns = 3;
constexpr int kPanel = 64;       // pivot block width of the large-front path
constexpr int kSmallMax = 128;   // largest front order of the LDS-resident path
constexpr int kTile = 64;        // tile order of the large-front MFMA update
constexpr int kInertiaSlots = 64;  // partial inertia counters per system (spreads the atomics)
constexpr int kNonfiniteInput = 1;   // status bit: NaN/Inf in the assembled K (its norms)
constexpr int kNonfiniteFactor = 4;  // status bit: NaN/Inf pivot met by the factorization
constexpr int kResWidth = 6;         // residual figures per (row chunk, column), see launch_residual
constexpr size_t kAsmLdsMax = 96 * 1024;  // large-front column assembly staged in LDS (4 columns per
                                           // workgroup) up to this size

// A large-front task (diagonal block, 32 panel rows or update tile) with its
// front's fields, so that one load brings all of it: pivots first .. first + p,
// order f, panel k0, a = first panel row or tile row, b = tile column.
struct LargeTask {
    int first, p, f, k0, a, b, sys, s;
    int64_t L_off, M_off;
};

// A small front: pivots first .. first + p, order f, its children's maps
// (kids kid0 .. kid0 + nkid) and its K entries (k0 .. k0 + kn of kent_csr / kent_rc).
struct FrontTask {
    int first, p, f, sys, s, kid0, nkid, kn;
    int64_t L_off, CB_off, k0;
    int CB_ld, pad;
};
// A child of a small front: its contribution block and its map, one byte per
// row of the parent: the contribution row that lands there, 255 for none.
struct KidMap {
    int64_t CB_off;
    int ld, map_off;
};
// What the small-front kernels read of the plan.
struct FrontPlan {
    const KidMap* kids;
    const uint8_t* kid_map;
    const int64_t* kent_csr;
    const int* kent_rc;        // front row + 256 * front column of each K entry (small fronts)
    const int8_t* piv_sign;
    const double* sys_thr;
    unsigned long long* inertia_part;
    int* nonfinite;
};

// A block's rows of K (one system) in assembly, norms and residuals: rows row0 ..
// row0 + rows, entries ent0 .. ent1, products prod0 .. prod0 + nprod.
struct RowChunk {
    int row0, rows, sys;
    unsigned int nprod;
    int64_t ent0, ent1, prod0;
};

// Device copies of the plan (all device pointers), passed by value.
struct DevPlan {
    int64_t N;
    int64_t n_primal;          // rows [0, n_primal) form the primal block (N for the condensed form)
    int S;
    // full CSR of K with value sources
    const int64_t* Kp;
    const int* Kj;
    const int* src;            // an entry's value: W's index, -2 - J's index, or -1
    const uint8_t* src_flag;
    const unsigned int* prod_ptr;   // its first product, from the row chunk's first
    const int* prod_a;
    const int* prod_b;
    const int* row_sys;
    const int* perm;
    const int8_t* piv_sign;    // per pivot: +1 primal, -1 dual
    // supernodes
    const int* sn_rows;
    const int* jrow_of;        // row of J of each stored J entry (condensed form)
    const int64_t* kent_csr;
    const int* kent_pos;
    const int* rel;
    // large-front column assembly tasks (see Plan::asm_*)
    const int64_t* asm_col;
    const int* asm_fj;
    const int64_t* asm_kr;
    const int64_t* asm_seg_ptr;
    const int64_t* asm_seg_cb;
    const int64_t* asm_seg_rel;
    const int* asm_seg_bc;
    // per system
    const double* sys_thr;     // static-pivot thresholds, 2 per system: primal, dual pivots
    unsigned long long* inertia_part;  // kInertiaSlots x 4 per system: npos, nneg, nzero, nperturbed
    int* nonfinite;            // status bits kNonfiniteInput | kNonfiniteFactor
};

// ---- assembly (FP64) ------------------------------------------------------
// Optional per-launch timing.  While a LaunchTimer is installed on the
// calling thread, every kernel launch asks it for a start/stop event pair and,
// when given one, is launched with hipExtLaunchKernel, whose events carry the
// kernel's own begin and end timestamps (no launch gaps in the figure).
struct LaunchTimer {
    virtual bool take(hipEvent_t* start, hipEvent_t* stop) = 0;
    virtual ~LaunchTimer() = default;
};
LaunchTimer* set_launch_timer(LaunchTimer* t);   // returns the previous one

// omega: per row of J, the weight of its products (K1s), or nullptr (K1, K2r).
// partial[3c..3c+2], per chunk: max |K_ij|, max row sum of |K|, max |K_ij| over the
// primal block.
void launch_assemble(const DevPlan& d, const RowChunk* chunks, int nchunks, const double* W, const double* Sigma,
                     const double* J, const double* sys_rho, const double* omega, double* K, double* partial,
                     hipStream_t st);
// ---- slack elimination (K1s) and step recovery (vectors in the caller's
// order; rows of J of all systems concatenated; rho per system) -------------
void launch_k1s_omega(int64_t nrows, const double* Sigma_s, const int* Jrow_sys, const double* sys_rho, double* omega,
                      int* nonfinite, hipStream_t st);
void launch_k1s_rhs(int64_t n, const int64_t* Jt_ptr, const int* Jt_row, const int* Jt_k, const double* J,
                    const double* r_t, const double* r_s, const double* Sigma_s, const int* Jrow_sys,
                    const double* sys_rho, const int* row_sys, double* b, hipStream_t st);
void launch_k1s_ds(int64_t nrows, const int64_t* Jp, const int* Jj, const double* J, const double* dt,
                   const double* r_s, const double* Sigma_s, const int* Jrow_sys, const double* sys_rho, double* ds,
                   hipStream_t st);
void launch_recover_dy(int64_t nrows, const int64_t* Jp, const int* Jj, const double* J, const double* dx,
                       const double* c, const double* y_k, const double* y, const int* Jrow_sys, const double* sys_rho,
                       double* dy, hipStream_t st);
void launch_recover_dr(int64_t nrows, const double* dy, const double* y_k, const double* y, const double* r,
                       const int* Jrow_sys, const double* sys_rho, double* dr, hipStream_t st);
void launch_recover_dz(int64_t n, const double* x, const double* l, const double* u, const double* z_l,
                       const double* z_u, const double* dx, double mu, double* dz_l, double* dz_u, hipStream_t st);
void launch_add_scalar(int64_t n, const double* in, double delta, double* out, hipStream_t st);
void launch_barrier_sigma(int64_t n, const double* x, const double* l, const double* u, const double* z_l,
                          const double* z_u, double* sigma, hipStream_t st);
// out[s*width + k] = reduction over the chunks of system s of partial[c*width + k]:
// a sum where bit (k mod period) of sum_mask is set, else a max.  Fixed order
// (deterministic).  1 <= period <= 32.
void launch_reduce(const int* sys_chunk_ptr, int S, int width, int period, unsigned int sum_mask,
                   const double* partial, double* out, hipStream_t st);
// kinf and the two static-pivot thresholds per system (thr[2s] primal,
// thr[2s+1] dual) from the chunks' norms.  mode 0: eps * max |K_ij| for both;
// 1, block rule: primal eps * max |K_xx|, dual eps / rho; 2: eps for both.
// Flags non-finite norms.
void launch_thresholds(const int* sys_chunk_ptr, int S, const double* partial, double eps, int mode,
                       const double* sys_rho, double* kinf, double* thr, int* nonfinite, hipStream_t st);

// ---- numeric factorization (T = double or float) --------------------------
// One launch of small fronts of order up to fmax; strip: elements of LDS for
// the pivot columns of the largest (front_strip).
template <typename T>
void launch_fronts(const FrontPlan& d, const FrontTask* tasks, int count, int fmax, int strip, const double* K, T* F,
                   T* D, hipStream_t st);
template <typename T>
void launch_large_asm(const DevPlan& d, int64_t first, int count, int fmax, const double* K, T* F, hipStream_t st);
template <typename T>
void launch_large_diag(const DevPlan& d, const LargeTask* tasks, int count, T* F, T* D, T* M, hipStream_t st);
template <typename T>
void launch_large_panel(const LargeTask* tasks, int count, T* F, const T* D, const T* M, hipStream_t st);
// Panel k's trailing update (utasks) and panel k+1's diagonal blocks (dtasks)
// in one launch.
template <typename T>
void launch_large_dstep(const DevPlan& d, const LargeTask* dtasks, int nd, const LargeTask* utasks, int nu, T* F,
                        T* D, T* M, hipStream_t st);

// ---- solves -----------------------------------------------------------------
// Vectors in pivot order with one value a row (nrhs = 1), or with kNrhsMax ("many";
// unused columns zero).
// B: column q of row i (caller's order) at B[i si + q sq].
template <typename T>
void launch_permute_in(const DevPlan& d, const double* B, int64_t si, int64_t sq, int nrhs, T* Y, hipStream_t st);
template <typename T>
void launch_permute_out(const DevPlan& d, const T* X, int nrhs, double* Xo, int64_t ldx, hipStream_t st);
// One step of a sweep: np panel tasks and ns small fronts.  Y: right-hand side
// (updated in place for rows not yet solved), Y2: the pivots' y, X: their x, U: update
// vectors; the backward tasks' sums go to pw, the previous step's are read from
// pr (slots x 128 values or rows of kNrhsMax, two halves used in turn).
template <typename T>
void launch_fwd(bool many, const PanelTask* pt, int np, const SmallTask* sm, int ns, const int* gat, const T* F,
                const T* Z, T* Y, T* Y2, T* U, hipStream_t st);
template <typename T>
void launch_bwd(bool many, const PanelTask* pt, int np, const SmallTask* sm, int ns, const int* rows, const T* F,
                const T* Z, const T* D, const T* Y2, T* X, T* pw, const T* pr, hipStream_t st);

// ---- refinement -------------------------------------------------------------
// R = B - K X; per chunk of rows (all of one system) and column, kResWidth figures:
// max |r|, max |x|, max |b|, sum r^2, sum b^2, max |r_i| / (|K||x| + |b|)_i.
// From kManyColumns columns R is row-major, kNrhsMax a row, and Xr (N x kNrhsMax) is
// scratch; with fewer R is N x nrhs by columns.
void launch_residual(const DevPlan& d, const double* K, const double* B, int64_t ldb, const double* X, int64_t ldx,
                     double* Xr, double* R, int nrhs, const RowChunk* chunks, int nchunks, double* partial,
                     hipStream_t st);
void launch_axpy_cols(double* X, int64_t ldx, const double* DX, int64_t N, int nrhs, hipStream_t st);
void launch_copy_cols(double* dst, int64_t ldd, const double* src, int64_t lds, int64_t N, int nrhs,
                      hipStream_t st);
// Before and after a factorization (host: pinned memory, see the kernels).
void launch_begin(int S, const double* rho_host, double* rho, int* nonfinite, unsigned long long* part,
                  hipStream_t st);
void launch_end(const DevPlan& d, const double* kinf, unsigned long long* host, hipStream_t st);

// Raises the dynamic-LDS limit of the LDS-resident kernels to the device maximum.
hipError_t configure_kernels(int max_dynamic_lds);

// ---- adjoint (condensed) ----------------------------------------------------
void launch_adjoint(const DevPlan& d, int64_t nnzW, const int* W_row, const int* W_col, int64_t nJrows,
                    const int64_t* Jp, const int* Jj, const int* Jrow_sys, const double* Jval, const double* sys_rho,
                    const double* X, const double* Lam, int64_t ld, int nrhs, double* gW, double* gSigma,
                    double* gJ, double* gRho, double* JX, double* JL, const int64_t* sys_jrow, hipStream_t st);

}  // namespace ncl
