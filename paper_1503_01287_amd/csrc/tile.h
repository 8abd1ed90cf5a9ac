// The natural-order operator of a large scalar finest level in tiles
// (k_tile.hip): the residual, damped Jacobi step, product, and product with <x, A x> of
// k_row.hip / k_mixed.hip on rows regrouped so that a tile's rows lie close
// together in the mesh and x is gathered from LDS.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace amgp2 {

constexpr int TILE_ROWS = 256;
constexpr int TILE_LANES = 2;     // lanes per row
constexpr int TILE_TRIP = 4;      // entries per lane and trip
constexpr int TILE_SLICE = 64 / TILE_LANES;  // rows whose entries are stored step by step
constexpr int TILE_AHEAD = TILE_TRIP * 64;  // places that are read past the last entry's (never used)
constexpr int TILE_LIST = 2048;   // most nodes of x that a tile may read

enum TileKind : int { TILE_F64 = 0, TILE_F32 = 1 };
enum TileOp : int { TILE_SPMV = 0, TILE_RESID, TILE_JACOBI, TILE_SPMV_DOT };

// Row q (of the tiles' order): node rows[q].x with rows[q].y entries; entry
// k of a slice's row r at base[slice] + (k / TILE_LANES) 64 + TILE_LANES r +
// k % TILE_LANES. A tile reads x at the nodes list[TILE_LIST t ..] (count[t]
// of them); lcol is an entry's place among these.
struct TileArgs {
    int nrows = 0;
    const int2 *rows = nullptr;
    const int *base = nullptr;
    const int *list = nullptr, *count = nullptr;
    int lds_nodes = 0;              // the largest count
    const uint16_t *lcol = nullptr;
    const void *val = nullptr;
    bool stream = false;            // values and places are not to stay in the caches
    const void *x = nullptr, *b = nullptr;
    void *y = nullptr;              // not x
    const void *dinv = nullptr;     // TILE_JACOBI: inverted diagonal, by node
    double omega = 1.0;
    double *partial = nullptr;      // TILE_SPMV_DOT: a partial of <x, y> per tile
};

void launch_tile(TileOp op, TileKind kind, const TileArgs &a, hipStream_t s);

// count, list and lcol from a CSR pattern; a tile that would read more than
// TILE_LIST nodes gets count TILE_LIST + 1 and nothing else
void launch_tile_lists(int nrows, const int2 *rows, const int *base, const int *rowptr, const int *col, int *count,
                       int *list, uint16_t *lcol, hipStream_t s);
// dst = the rows' values in the tiles' order
void launch_tile_values(TileKind kind, int nrows, const int2 *rows, const int *base, const int *rowptr,
                        const void *src, void *dst, hipStream_t s);

}  // namespace amgp2
