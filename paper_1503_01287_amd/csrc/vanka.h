// Multiplicative Vanka smoother (Section 3.3): one patch per pressure DOF
// holding that DOF and the velocity nodes coupled to it through B; each
// patch's local saddle matrix is inverted once at setup (batched
// Gauss-Jordan, FP64) and a sweep applies x_P += omega K_P^{-1} (b - K x)_P
// patch by patch, colour by colour (patches of one colour share no node and
// are not coupled, so they update at the same time).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace amgp2 {

struct VankaView {
    int npatch = 0;
    const int *pptr = nullptr, *pnode = nullptr;  // patch i: velocity nodes pnode[pptr[i] .. pptr[i+1])
    const int64_t *moff = nullptr;                // inverse of patch i at inv + moff[i], m_i x m_i, column-major
    double *inv = nullptr;
    // the level's operators (planes)
    int n = 0;                                    // velocity nodes
    const int *arow = nullptr, *acol = nullptr;
    const double *aval = nullptr;
    int64_t annz = 0;
    const int *brow = nullptr, *bcol = nullptr;   // B (1x3)
    const double *bval = nullptr;
    int64_t bnnz = 0;
    const int *btrow = nullptr, *btcol = nullptr; // B^T (3x1)
    const double *btval = nullptr;
    int64_t btnnz = 0;
    const int *crow = nullptr, *ccol = nullptr;   // C (may be null)
    const double *cval = nullptr;
};

// local matrices [[A_P, B_P^T], [B_P, -C_ii]] of every patch, then their
// inverses in place; flag |= 1 on an exactly zero pivot
void launch_vanka_assemble(const VankaView &v, int max_nodes, hipStream_t s);
void launch_vanka_invert(const VankaView &v, int max_m, int *flag, hipStream_t s);
// 64 rows of a patch's correction
struct VankaTile {
    int64_t inv = 0;   // the patch's inverse in VankaView::inv
    int m = 0;         // its unknowns
    int row0 = 0;      // first row of the tile
    int res = 0;       // the patch's residual in rbuf
    int node0 = 0;     // its first node in pnode
    int patch = 0;
    int pad = 0;
};

// What one colour's patches read: their residual rows (a patch's velocity
// nodes, then its pressure; rown: node, or ~pressure, and place in rbuf;
// rowa: entries of A and B^T, or of B and C) and their correction tiles
struct VankaColour {
    int count = 0, nrows = 0, ntiles = 0;
    const int2 *rown = nullptr;
    const int4 *rowa = nullptr;
    const VankaTile *tile = nullptr;
};

// rowa from rown and the level's operators
void launch_vanka_rows(const VankaView &v, int nrows, const int2 *rown, int4 *rowa, hipStream_t s);
// One colour, x = [u (3n); p], in two kernels: the patches' residuals into
// rbuf, rg lanes per row (16, 32 or 64), then the corrections over 64-row
// tiles of every inverse, aw (4, 8 or 16) wavefronts per tile splitting its
// columns.
void launch_vanka_colour_rows(const VankaView &v, const VankaColour &c, int rg, int aw, double *rbuf,
                              const double *b, double *x, double omega, hipStream_t s);
// The same colour in three kernels, for few, large patches: the residuals,
// then partial corrections over 64-row x cc-column tiles of every inverse
// into pbuf (patch i's ceil(m_i / cc) chunks of m_i values at pbuf +
// poff[i]; its residual at rbuf + roff[i]; upre: prefix of the tiles
// ceil(m_i / 64) ceil(m_i / cc) over the colour's patches order[0 .. count),
// nunits their total), then the chunks summed in order into x over the
// 64-row tiles (tpre: prefix of their counts over the colour's patches)
void launch_vanka_colour_tiled(const VankaView &v, const VankaColour &c, const int *order, const int *tpre,
                               const int *upre, int nunits, int cc, int rg, const int64_t *roff, double *rbuf,
                               const int64_t *poff, double *pbuf, const double *b, double *x, double omega,
                               hipStream_t s);

}  // namespace amgp2
