// Descriptors of the levels whose cycle k_tail.hip assembles as an operator.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace amgp2 {

struct TailLevel {
    int n = 0;          // nodes
    int ncolors = 0;    // Gauss-Seidel colours (0 for Jacobi / coarsest)
    int lds_off = 0;    // offset (doubles) of x, b, r (3n each) in LDS
    int nc = 0;         // nodes of the next coarser level
    const int *cptr = nullptr;  // colour ranges of the grouped rows
    const int *g_rowptr = nullptr, *g_col = nullptr;
    const double *g_val = nullptr;
    int64_t g_nnz = 0;
    const int *g_rowid = nullptr;
    const int *a_rowptr = nullptr, *a_col = nullptr;
    const double *a_val = nullptr;
    int64_t a_nnz = 0;
    const double *dinv = nullptr;
    const int *r_rowptr = nullptr, *r_col = nullptr;  // restriction (nc rows)
    const double *r_val = nullptr;
    const int *p_rowptr = nullptr, *p_col = nullptr;  // prolongation (n rows)
    const double *p_val = nullptr;
    double omega = 0.5;
};

struct TailArgs {
    int nlev = 0;        // tail levels, the last one the coarsest
    int smoother = 1;    // AMG_SMOOTH_JA or AMG_SMOOTH_GS
    int pre = 1, post = 1;
    int nu = 1;          // visits of a level per visit of its parent
    int top_visits = 1;  // visits of the first tail level, from zero
    const TailLevel *lv = nullptr;  // device array of nlev descriptors
    const double *cinv = nullptr;   // coarsest explicit inverse (cm x cm)
    int cm = 0, cnc = 1;
    // workgroup j solves for the j-th unit right-hand side (mode 3: e_j over
    // the 3n unknowns; mode 1: component 0 of node j) and writes its result as
    // column j of the row-major m x m matrix x_out
    double *x_out = nullptr;
    int m = 0;
    int unit_base = 0;   // workgroup j handles unit right-hand side unit_base + j
    // if set, workgroup j keeps its level vectors at gscratch + j * gstride
    // (doubles) instead of LDS
    double *gscratch = nullptr;
    int64_t gstride = 0;
};

constexpr int TAIL_LEVELS_MAX = 32;       // levels of a tail at most
constexpr int TAIL_LDS_MAX = 64 * 1024;   // bytes of LDS a workgroup's level vectors may take
// The finest level is part of the operator where its assembly costs little: the
// level vectors in LDS and this many stored entries (about 2 ms; a cycle's
// launches take 90 us against 5-10 us for the product)
constexpr int64_t TAIL_NNZ_MAX = 40000;
constexpr int TAIL_DENSE_MAX = 9000;      // largest tail operator kept as an explicit matrix
// The same for several visits of a level (nu > 1). Each of m columns is a whole
// W-cycle then, so the assembly grows with m^2 and more, while the visits that
// it saves are cheap on larger levels: setup and one solve together must not
// take longer than without. ms of setup + solve without any map / with it
// (W-cycles, 2-2 steps):
//   GS  m  980 (x3) elasticity  9^3  70 + 25 / 42 + 5     JA  m  737 Laplacian  8^3  35 +  2 /  25 + 1
//      1272 (x3)   elasticity 24^3  187 + 117 / 98 + 24      1272  Laplacian 24^3   89 + 11 /  69 + 4
//      5217        Laplacian 16^3    97 + 32 / 213 + 4       2846  Laplacian 32^3  124 + 14 / 143 + 7
//      2293 (x3)   elasticity 12^3   99 + 44 / 171 + 6       5217  Laplacian 16^3   57 +  5 / 180 + 3
// (JA also assembles again when a caller sets its weights: 3, 9, 47 and 146 ms.)
constexpr int TAIL_W_GS_MAX = 4000;
constexpr int TAIL_W_JA_MAX = 1500;

// `grid` columns from unit_base on
void launch_tail(int mode, const TailArgs &a, int lds_bytes, int grid, hipStream_t s);

}  // namespace amgp2
