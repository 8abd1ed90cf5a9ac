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
// Some rows of a patch's correction (64, or in k_vanka_sweep `rows` in
// `groups` groups)
struct VankaTile {
    int64_t inv = 0;   // the patch's inverse in VankaView::inv
    int m = 0;         // its unknowns
    int row0 = 0;      // first row of the tile
    int res = 0;       // the patch's residual in rbuf
    int node0 = 0;     // its first node in pnode
    int patch = 0;
    int row = 0;       // its first residual row
    int rows = 0, groups = 0;
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

// A residual row of k_vanka_sweep
struct VankaRow {
    int node = 0, res = 0;     // as VankaColour::rown
    int first = 0, pad = 0;    // its entries in VankaSweep::entry
    int4 entries = {};         // as VankaColour::rowa
};
constexpr int VANKA_ITEM_ROWS = 32;  // rows of 32 lanes in an item (of 64: half)
constexpr int VANKA_SHORT = 64;      // most entries of a row that has 32 lanes

// What a sweep over all colours in one launch reads and writes
// (k_vanka_sweep). Patches' unknowns are known by their residual rows, in
// colour order: a row stands for a patch's node, or its pressure.
struct VankaSweep {
    int nitems = 0;
    const int2 *item = nullptr;     // colour by colour: residual rows (first in row; count: 32 lanes each, -count: 64),
                                    // then tiles (~tile, 0)
    const VankaRow *row = nullptr;
    const int2 *rown = nullptr;     // the rows in colour order
    const int2 *entry = nullptr;    // by their last writers' colours: the row that wrote the column's value last, or
                                    // ~column; the entry's number among those of A and B^T (B and C)
    const int2 *own = nullptr;      // of a row: the row that wrote its unknowns before, or ~0; 1 if none does after
    const VankaTile *tile = nullptr;
    double *xs = nullptr, *rs = nullptr;  // written unknowns (4 a row) and residuals: two buffers each,
    int64_t xs_half = 0, rs_half = 0;     // filled with "absent" before the first sweep
    int *ctl = nullptr;             // VANKA_CTL_INTS words, zero before the first sweep
    const double *b = nullptr, *x_old = nullptr;  // x_old: another buffer than x, which holds the same on entry
    double *x = nullptr;
    double omega = 1.0;
};
constexpr int VANKA_CTL_INTS = 128;
void launch_vanka_sweep(const VankaView &v, const VankaSweep &a, int grid, hipStream_t s);
// entry and own from the rows' entries; node n's writers, by colour, are
// writer[nptr[n] .. nptr[n + 1]) (residual row, colour), those of pressure i
// writer[nptr[v.n + i] ..]
void launch_vanka_entries(const VankaView &v, int nrows, const int2 *rown, const int4 *rowa, const int *pptr,
                          const int *colour, const int *nptr, const int2 *writer, int2 *entry, int2 *own,
                          hipStream_t s);
void launch_vanka_absent(double *p, int64_t n, hipStream_t s);

}  // namespace amgp2
