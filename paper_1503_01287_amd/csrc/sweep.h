// Gauss-Seidel sweeps over all colours of a level in one launch (k_sweep.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace amgp2 {

// What an entry is: a 3x3 block, a scalar applied to 3-component vectors, or
// a scalar applied to a scalar vector (Schur complements).
enum SweepMode : int { SWEEP_BLOCK = 3, SWEEP_SCALAR3 = 1, SWEEP_SCALAR1 = 0 };
enum SweepKind : int { SWEEP_F64 = 0, SWEEP_F32 = 1, SWEEP_BF16 = 2 };

constexpr int SWEEP_THREADS_MIN = 512;  // threads of a workgroup: these, or twice as many
constexpr int SWEEP_MAX_COLOURS = 1023;
constexpr int SWEEP_PAD = 32;         // a colour's range of the swept vector starts at a multiple of this many nodes
// control words of a level's sweeps: ticket, exits, sweeps so far (odd and even
// ones take the two buffers in turn), the last sweep that gave up
constexpr int SWEEP_CTL_INTS = 128;

// Grouped rows: a row's entries with earlier colours come first, then the
// diagonal, then those with later colours.
struct SweepArgs {
    int ncolors = 0, ntiles = 0;
    const int *cptr = nullptr;      // grouped rows of colour c
    const int *tpre = nullptr;      // first tile of colour c (ncolors + 1)
    const int *base = nullptr;      // first node of colour c in xg
    const int4 *rows = nullptr;     // of grouped row g: first entry, diagonal, end, node
    const int *col = nullptr;       // node of an entry's column
    const int *gcol = nullptr;      // its place in xg
    const void *val = nullptr;      // planes nnz apart
    int64_t nnz = 0;
    const void *dinv = nullptr;     // inverted diagonal blocks, planes dinv_n apart
    int64_t dinv_n = 0;
    const float *rscale = nullptr;  // BF16: scale of a scalar row
    const void *b = nullptr;
    const void *x_old = nullptr;    // the iterate on entry, another buffer than x (not read if x_zero)
    void *x = nullptr;              // the iterate on return
    void *xg = nullptr;             // swept values by colour, 4 (scalar vectors: 1) per node: two buffers,
    int64_t xg_half = 0;            // xg_half values apart, the first one filled with "absent" before the first sweep
    void *part = nullptr;           // if set: b - (entries of earlier colours and the diagonal) x
    int forward = 1;
    int x_zero = 0;                 // x is zero on entry (its buffer need not hold the zeros; forward only)
    int *ctl = nullptr;             // SWEEP_CTL_INTS words of this level, zero before the first launch
};

// G lanes per row (8, 16, 32, 64), at most `grid` workgroups of `threads`
struct SweepShape {
    int G = 16, grid = 256, threads = 2 * SWEEP_THREADS_MIN;
    int tile_rows() const { return threads / G; }
};
// Swept values are read at 32-bit byte offsets through a buffer descriptor of
// one half of xg: whether `places` of `stride` FP64 values stay below 2 GiB.
// (Past it an offset wraps, and a load past the descriptor's size returns 0,
// which is not "absent".)
constexpr bool sweep_half_fits(int64_t places, int stride) { return places * stride * 8 < (int64_t(1) << 31); }

constexpr int SWEEP_TILE_SIZES = 5;  // tiles of (SWEEP_THREADS_MIN / 64) << t rows

// Whether a level's sweeps run a launch per colour although one launch could
// take them all: with many entries a colour the launches cost little (5 us
// each), and their rows need no waits and no second copy of x (k_sweep's tiles
// stream 15 to 30% slower). What one launch saves besides, half of a residual,
// it saves once a cycle, after the last of `pre` sweeps, so the line lies lower
// for more than two sweeps or none before the residual. us per cycle, one
// launch / a launch for each of the finest level's 14 colours, at thousands of
// entries a colour:
//   3x3 blocks FP64   GS-1-1  361  712 / 726    538 1012 / 983   1817 2854 / 2477
//                     GS-2-2  289 1088 / 1078   361 1264 / 1234  1817 5372 / 4391
//          FP32       GS-1-1 1218 1129 / 1137  1400 1273 / 1266  1817 1600 / 1558
//                     GS-2-2  361  788 / 839    538 1091 / 1045  1817 2905 / 2721
//   scalar FP64       GS-1-1  766  628 / 645   1051  835 / 822   4306 2982 / 2587
//                     GS-2-2  901 1260 / 1252  1051 1461 / 1413
//          FP32       GS-1-1 1817 1043 / 1060  2310 1272 / 1202  4306 2193 / 2080
//                     GS-2-2 1399 1347 / 1343  1817 1904 / 1798
// and of level 1, 30 colours of rows of 70 entries (both levels by colour):
//   scalar FP64       GS-1-1  476 1846 / 1872   711 2587 / 2534
//          BF16       GS-1-1  476 1495 / 1537   711 2080 / 2050
//   blocks FP64       GS-2-2  309 4391 / 4662
inline bool sweep_by_colour(int mode, bool fp64, int64_t nnz, int nrows, int ncolors, int pre, int post) {
    const bool few = pre > 0 && pre + post <= 2;
    int64_t most = 600000;
    if (mode == SWEEP_BLOCK) most = fp64 ? (few ? 450000 : 350000) : (few ? 1300000 : 450000);
    else if (nnz <= 40 * static_cast<int64_t>(nrows)) most = fp64 ? 950000 : (few ? 2200000 : 1400000);
    return ncolors > 0 && nnz > most * ncolors;
}

// "absent" into both buffers of xg (n values in all, of the sweep's precision)
void launch_sweep_absent(int kind, void *xg, int64_t n, hipStream_t s);
void launch_sweep(int mode, int kind, const SweepShape &q, const SweepArgs &a, hipStream_t s);
// part -= (entries of later colours) x on the nrows grouped rows: the residual
// after a forward sweep with the same arguments
void launch_later(int mode, int kind, int nrows, const SweepShape &q, const SweepArgs &a, hipStream_t s);

// place[i]: node i's place in xg; base[c]: first place of colour c. Rows
// order[g] gathered into the grouped copy with their entries split as
// SweepArgs wants them (a stable partition by the columns' places); rows, gcol
// written with it. coupled |= 1 where a row has an entry of its own colour
// beside one diagonal, or of a node that is not swept.
void launch_split_rows(int np, int nrows, const int *order, const int *place, const int *base, int ncolors,
                       const int *rowptr, const int *col, const double *val, int64_t nnz, const int *g_rowptr,
                       int *g_col, double *g_val, int64_t g_nnz, int4 *rows, int *gcol, int *coupled, hipStream_t s);

}  // namespace amgp2
