// plan.hpp — host-side symbolic plan of the supernodal multifrontal LDL^T.
//
// Everything here is computed once per sparsity pattern (the paper reuses the
// symbolic factorization across iterations, Sec. 4.1) and uploaded once.
#pragma once

#include <cstdint>
#include <string>
#include <vector>

namespace ncl {

struct PlanConfig {
    int small_front_max = 90;   // fronts with f <= this run in one workgroup (at most kSmallMax)
    int panel = 64;             // pivot block width of the large-front path
    int tile = 64;              // tile order of the large-front update
    int nd_leaf = 64;           // nested-dissection leaf size (compressed vertices)
    int relax_big_front = 128;  // fronts above this order (the global-memory path, swept in
    double relax_big_zeros = 0.2;  // panels anyway) may carry up to this fraction of zeros
};

// LDS elements that the pivot columns of a small front of order f with p pivots
// take: whole 16-column sub-panels, leading dimension an odd multiple of 16
// that covers f.
inline int front_strip(int f, int p) { return 16 * (((f + 15) / 16) | 1) * 16 * ((p + 15) / 16); }

struct LevelBatch {            // one launch of the small-front kernel
    int level = 0;
    int fmax = 0;              // largest front in the batch
    int strip = 0;             // LDS elements of the pivot columns, see front_strip()
    int64_t first = 0, count = 0;  // range in Plan::small_list
};

struct LargeStep {             // launches of the large-front path for one level
    int level = 0;
    int64_t asm_first = 0, asm_count = 0;     // (front, column) tasks in Plan::asm_*
    int asm_fmax = 0;                         // largest front of the level (column buffer size)
    // per panel step k: diagonal-block, panel (TRSM) and update tasks
    std::vector<int64_t> diag_first, diag_count;
    std::vector<int64_t> panel_first, panel_count;
    std::vector<int64_t> upd_first, upd_count;
    std::vector<double> upd_flops;            // algorithmic flops of each update launch
};

// A task of a sweep: 64 rows r0 .. r1 below a pair of panels (columns c0 .. c0 +
// w1 + w2, w2 = 0 for a lone one) of a large front (pivots first .. first + p,
// order f); task `index` of ntask (index -1: a record that only finishes).
// Backward: sums go to partial slot slot0 + index; a task with fntask > 0
// first finishes panel `which` of the pair at fc0 from its fntask sums at
// fslot0.  gat, gk, deep: the front's gather table (gk = 0 unless c0 = 0).
struct PanelTask {
    int first, p, f, c0, w1, w2, r0, r1, index, ntask, slot0, gk, deep;
    int fc0, fw1, fw2, fslot0, fntask, which;
    int64_t L_off, U_off, M_off, rows_off, gat;
};
struct SmallTask {             // a small front's sweep
    int first, p, f, gk, deep, pad;
    int64_t L_off, U_off, rows_off, gat;
};
// One launch of a sweep, in execution order.  k: pair step of the level (backward
// partial half), -1 for the records that finish the first pairs of a level.
struct SolveStep {
    int level = 0, k = 0;
    int64_t p_first = 0, p_count = 0;   // tasks in Plan::fwd_tasks / bwd_tasks
    int64_t s_first = 0, s_count = 0;   // small fronts in Plan::solve_small
    double bytes = 0.0;                 // algorithmic bytes of L read by the step (FP64; padding
                                        // zeros of amalgamated fronts not counted)
};

struct Plan {
    // ---- problem --------------------------------------------------------
    int form = 0;               // 0 condensed, 1 stabilized
    int S = 1;                  // number of independent systems (batched)
    int64_t N = 0;              // order of the (block-diagonal) matrix
    std::vector<int> sys_n, sys_m;
    std::vector<int64_t> sys_voff;   // S+1: first unpermuted index of each system
    std::vector<int64_t> sys_woff, sys_joff;  // offsets of each system's W / J values
    int64_t nnzW = 0, nnzJ = 0, nJrows = 0;
    std::vector<int> row_sys;        // N: system of each unpermuted index
    std::vector<int8_t> row_sign;    // N: +1 primal, -1 dual (unpermuted)

    // ---- full symmetric CSR of K (unpermuted), with value sources -------
    std::vector<int64_t> Kp;         // N+1
    std::vector<int> Kj;             // nnzF column indices
    std::vector<int> src;            // nnzF: W value index, -2 - J value index (stabilized J / J^T blocks) or -1
    std::vector<uint8_t> src_flag;   // bit0: add Sigma[row]; bit1: add -1/rho
    std::vector<int64_t> prod_ptr;   // nnzF+1: pairs of J value indices (condensed)
    std::vector<int> prod_a, prod_b;
    int64_t nnz_lower = 0;

    // ---- J structure (for the adjoint) -----------------------------------
    std::vector<int64_t> Jp;          // rows of the concatenated J
    std::vector<int> Jj;              // unpermuted column indices (global)
    std::vector<int> Jrow_sys;
    std::vector<int64_t> Wcol_of;     // per stored W entry: global column; row in Wrow_of
    std::vector<int> Wrow_of, Wcol_of32;

    // ---- ordering --------------------------------------------------------
    std::vector<int> perm, iperm;    // perm[k] = unpermuted index of pivot k

    // ---- supernodes ------------------------------------------------------
    int nsn = 0;
    std::vector<int> sn_first;       // nsn+1
    std::vector<int> sn_parent;      // nsn
    std::vector<int64_t> sn_rowptr;  // nsn+1
    std::vector<int> sn_rows;        // pivot numbering; pivots first then CB rows
    std::vector<int> sn_level;
    std::vector<int> sn_sys;
    std::vector<int> child_ptr, child_list;
    std::vector<uint8_t> sn_large;

    // front assembly of K entries: per supernode (csr position, local position)
    std::vector<int64_t> kent_ptr;   // nsn+1
    std::vector<int64_t> kent_csr;
    std::vector<int> kent_pos;       // local row + local col * f
    std::vector<int> kent_col;       // local column (large fronts, sorted by it)
    std::vector<int64_t> kcol_ptr;   // large fronts: per (front, local col) segment, indexed by
    std::vector<int64_t> kcol_base;  //   kcol_base[s] + j, length p+1

    // extend-add maps: child CB row a -> local row in the parent front
    std::vector<int64_t> rel_ptr;    // nsn+1 (length c_s)
    std::vector<int> rel;

    // ---- storage ---------------------------------------------------------
    std::vector<int64_t> L_off;      // offset of front s's L (ld = f) in the factor buffer
    std::vector<int64_t> CB_off;     // offset of the contribution block
    std::vector<int> CB_ld;
    int64_t factor_elems = 0;        // factor buffer length (elements of T)
    std::vector<int64_t> U_off;      // solve: update vector of each front (c_s * nrhs_max)
    std::vector<int64_t> M_off;      // large fronts: per-panel inverses L_kk^-1 (panel^2 each)
    int64_t M_elems = 0;
    int64_t U_elems = 0;

    // ---- schedule --------------------------------------------------------
    int nlevels = 0;
    std::vector<int> small_list;     // supernodes, grouped by level then size batch
    std::vector<LevelBatch> small_batches;
    std::vector<int> level_ptr;      // nlevels+1 into level_list (all fronts by level)
    std::vector<int> level_list;
    std::vector<LargeStep> large_steps;
    // large-front tasks
    // assembly tasks (front, column j): column base in the factor buffer, (f, j),
    // K-entry range, and its contribution segments (children whose CB has a column
    // mapping to j): CB column offset, relative-index offset, (first row, rows)
    std::vector<int64_t> asm_col, asm_kr, asm_seg_ptr, asm_seg_cb, asm_seg_rel;
    std::vector<int> asm_fj, asm_seg_bc;
    std::vector<int> large_diag;     // pairs (front, k0): diagonal block update, factorization, inverse
    std::vector<int> large_panel;    // triples (front, k0, 32-row block start >= min(k0 + panel, pivots))
    std::vector<int> large_upd;      // quads (front, k0, tile row start, tile col start); the next
                                     // panel's diagonal tile is left to large_diag
    // solve schedule
    std::vector<SolveStep> fwd_steps, bwd_steps;
    std::vector<PanelTask> fwd_tasks, bwd_tasks;
    std::vector<SmallTask> solve_small;
    // Gather tables of the update vectors: row i of a front takes entries gather[gat +
    // k f + i], k = 0 .. gk - 1 (-1: none), in the children's order; where a row takes
    // more (`deep`), f + 1 starts and the further entries by rows follow the table.
    std::vector<int> gather;
    int64_t solve_max_slots = 0;     // backward tasks in the largest step (partial-sum slots)

    // ---- stats ------------------------------------------------------------
    int64_t nnzL = 0;
    double flops = 0.0, small_flops = 0.0, large_flops = 0.0;   // as executed (padding included)
    int64_t nnzL_exact = 0;          // column counts of the elimination tree (no padding)
    double flops_exact = 0.0;        // sum over columns of c (c + 2), c = below-diagonal count
    std::vector<double> sn_flop_ratio;  // per supernode: exact / executed flops of its pivots
    std::vector<double> sn_nnz_ratio;   // per supernode: exact / stored entries of its L columns
    int max_front = 0;
    int n_large = 0;
    double analyze_seconds = 0.0;
    PlanConfig cfg;
};


}  // namespace ncl
