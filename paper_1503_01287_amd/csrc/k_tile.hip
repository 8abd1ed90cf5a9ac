// Kernels of a scalar operator in tiles (see tile.h).
//
// In row order such a pass is bound by its gathers of x, not by memory: an
// entry is 8 or 12 bytes, but its column's 3 components are 12 or 24 bytes in
// a line of their own, and the L1 serves about one line a cycle (48^3
// Laplacian, 25.4 M entries: FP64 operator 123 us, FP32 residual 85 us, where
// their 345 and 230 MB take 66 and 44 us at the rate of a large copy). 256
// rows that are close in the mesh read each node of x about 6 times, so a
// tile loads its nodes (4.5 a row) once, into LDS, and an entry holds its
// 2-byte place among these instead of a 4-byte column. Entries are stored step
// by step over the lanes of a slice of rows, so that a wavefront's loads of
// values and places are contiguous; a tile's rows are ordered by length, and
// the padding is 9%. Now 87 and 54 us (4.2 TB/s of 367 and 225 MB). Tiles of
// 128 rows (6.6 nodes a row with the padding at 26%: 99 and 65 us) and of 512
// (lists past 2048 nodes, one or two workgroups in a CU's LDS) are slower;
// four lanes a row, 12 steps of loads instead of 4 ahead, no better. The
// coarse levels' rows are too dense (47 entries, 6.8 nodes a row: FP32/BF16
// passes no faster in tiles).
#include "common.h"
#include "tile.h"

namespace amgp2 {

constexpr int NT = TILE_ROWS * TILE_LANES;

template <int KIND>
struct TileType { using T = float; };
template <>
struct TileType<TILE_F64> { using T = double; };

template <bool STREAM, typename T>
__device__ __forceinline__ T once(const T *p) {
    if constexpr (STREAM) return __builtin_nontemporal_load(p);
    else return *p;
}

// Lane h of a row takes its entries h, h + 2, ..., four sums each (entry k in
// the sums k mod 8 of the row), U entries a trip with the next trip's
// loads in flight.
template <int KIND, int OP, bool STREAM>
__global__ void __launch_bounds__(NT) k_tile(const TileArgs a) {
    using X = typename TileType<KIND>::T;
    constexpr int U = TILE_TRIP;
    extern __shared__ __align__(16) unsigned char smem[];
    X *xs = reinterpret_cast<X *>(smem);
    // XCD k (every eighth workgroup) takes the k-th eighth of the tiles, so
    // that the nodes which neighbouring tiles share meet in one L2
    const int per = gridDim.x / 8, more = gridDim.x % 8, xcd = blockIdx.x % 8;
    const int t = xcd * per + min(xcd, more) + blockIdx.x / 8;
    const int h = threadIdx.x % TILE_LANES;
    const int q = t * TILE_ROWS + threadIdx.x / TILE_LANES;
    const bool on = q < a.nrows;
    // three chains of loads side by side: row; base, first entries (read
    // before the row's length is known); list, x
    const int at = __builtin_amdgcn_readfirstlane(on ? a.base[q / TILE_SLICE] : 0) + static_cast<int>(threadIdx.x & 63);
    const int m = a.count[t];
    const int *list = a.list + static_cast<int64_t>(t) * TILE_LIST;
    int node[TILE_LIST / NT];
#pragma unroll
    for (int u = 0; u < TILE_LIST / NT; ++u) {
        const int k = threadIdx.x + u * NT;
        node[u] = k < a.lds_nodes ? list[k] : 0;
    }
    const int2 row = on ? a.rows[q] : make_int2(0, 0);
    const int n = (row.y - h + TILE_LANES - 1) / TILE_LANES;  // entries of this lane
    const X *val = static_cast<const X *>(a.val) + at;
    const uint16_t *lc = a.lcol + at;
    X v[U];
    int c[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        v[u] = once<STREAM>(val + u * 64);
        c[u] = once<STREAM>(lc + u * 64);
    }
    const X *x = static_cast<const X *>(a.x);
#pragma unroll
    for (int u = 0; u < TILE_LIST / NT; ++u) {
        const int k = threadIdx.x + u * NT;
        if (k < m) {
            const X *xj = x + 3 * static_cast<int64_t>(node[u]);
            xs[k] = xj[0];
            xs[m + k] = xj[1];
            xs[2 * m + k] = xj[2];
        }
    }
    const int64_t o = 3 * static_cast<int64_t>(row.x);
    const bool ep = on && h == 0;
    X b0 = 0, b1 = 0, b2 = 0, w0 = 0, w1 = 0, w2 = 0, d = 0;
    if (ep) {
        if constexpr (OP == TILE_RESID || OP == TILE_JACOBI) {
            const X *b = static_cast<const X *>(a.b) + o;
            b0 = b[0];
            b1 = b[1];
            b2 = b[2];
        }
        if constexpr (OP == TILE_JACOBI || OP == TILE_SPMV_DOT) {
            w0 = x[o];
            w1 = x[o + 1];
            w2 = x[o + 2];
        }
        if constexpr (OP == TILE_JACOBI) d = static_cast<const X *>(a.dinv)[row.x];
    }
    __syncthreads();
    X s[3][U] = {};
    for (int k = 0; k < n; k += U) {
        X vn[U];
        int cn[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool more = k + U + u < n;
            vn[u] = more ? once<STREAM>(val + (k + U + u) * 64) : X(0);
            cn[u] = more ? once<STREAM>(lc + (k + U + u) * 64) : 0;
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (k + u < n) {  // (a value past the row's end must not meet an infinite x)
                s[0][u] += v[u] * xs[c[u]];
                s[1][u] += v[u] * xs[m + c[u]];
                s[2][u] += v[u] * xs[2 * m + c[u]];
            }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            v[u] = vn[u];
            c[u] = cn[u];
        }
    }
    X r[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        r[i] = (s[i][0] + s[i][2]) + (s[i][1] + s[i][3]);
        r[i] += __shfl_xor(r[i], 1, TILE_LANES);
    }
    X *y = static_cast<X *>(a.y) + o;
    if (ep) {
        if constexpr (OP == TILE_SPMV || OP == TILE_SPMV_DOT) {
            y[0] = r[0];
            y[1] = r[1];
            y[2] = r[2];
        } else if constexpr (OP == TILE_RESID) {
            y[0] = b0 - r[0];
            y[1] = b1 - r[1];
            y[2] = b2 - r[2];
        } else {
            const X om = static_cast<X>(a.omega);
            y[0] = w0 + om * (d * (b0 - r[0]));
            y[1] = w1 + om * (d * (b1 - r[1]));
            y[2] = w2 + om * (d * (b2 - r[2]));
        }
    }
    if constexpr (OP == TILE_SPMV_DOT) {
        __shared__ double red[NT / 64];
        double p = ep ? static_cast<double>(w0 * r[0] + w1 * r[1] + w2 * r[2]) : 0.0;
#pragma unroll
        for (int i = 32; i > 0; i >>= 1) p += __shfl_xor(p, i, 64);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = p;
        __syncthreads();
        if (threadIdx.x == 0) {
            double sum = 0.0;
#pragma unroll
            for (int i = 0; i < NT / 64; ++i) sum += red[i];
            a.partial[t] = sum;
        }
    }
}

template <int KIND, bool STREAM>
static void tile_op(TileOp op, const TileArgs &a, hipStream_t s) {
    const int nb = ceil_div(a.nrows, TILE_ROWS);
    const size_t lds = 3 * static_cast<size_t>(a.lds_nodes) * sizeof(typename TileType<KIND>::T);
    switch (op) {
        case TILE_SPMV: k_tile<KIND, TILE_SPMV, STREAM><<<nb, NT, lds, s>>>(a); break;
        case TILE_RESID: k_tile<KIND, TILE_RESID, STREAM><<<nb, NT, lds, s>>>(a); break;
        case TILE_JACOBI: k_tile<KIND, TILE_JACOBI, STREAM><<<nb, NT, lds, s>>>(a); break;
        case TILE_SPMV_DOT:
            AMG_REQUIRE(KIND == TILE_F64, AMG_EINVAL, "tiled operator: the product with <x, y> runs in FP64");
            if constexpr (KIND == TILE_F64) k_tile<KIND, TILE_SPMV_DOT, STREAM><<<nb, NT, lds, s>>>(a);
            break;
    }
    AMG_CHECK_LAUNCH();
}

void launch_tile(TileOp op, TileKind kind, const TileArgs &a, hipStream_t s) {
    if (a.nrows <= 0) return;
    AMG_REQUIRE(a.lds_nodes <= TILE_LIST, AMG_EINVAL, "tiled operator: a list is too long");
    AMG_REQUIRE(a.x != a.y, AMG_EINVAL, "tiled operator: in place");
    if (kind == TILE_F64) a.stream ? tile_op<TILE_F64, true>(op, a, s) : tile_op<TILE_F64, false>(op, a, s);
    else a.stream ? tile_op<TILE_F32, true>(op, a, s) : tile_op<TILE_F32, false>(op, a, s);
}

// One workgroup per tile: its columns into a hash table in LDS (setup only;
// bound by the probes), the distinct ones sorted, the entries' places found
// by bisection. The list is sorted, so it does not depend on the order in
// which the table was filled.
constexpr int HASH = 4 * TILE_LIST;
__global__ void __launch_bounds__(NT) k_tile_lists(int nrows, const int2 *rows, const int *base, const int *rowptr,
                                                   const int *col, int *count, int *list, uint16_t *lcol) {
    __shared__ int table[HASH];
    __shared__ int sorted[TILE_LIST];
    __shared__ int found, placed;
    const int t = blockIdx.x, h = threadIdx.x % TILE_LANES;
    const int q = t * TILE_ROWS + threadIdx.x / TILE_LANES;
    const bool on = q < nrows;
    const int2 row = on ? rows[q] : make_int2(0, 0);
    const int beg = on ? rowptr[row.x] : 0;
    for (int k = threadIdx.x; k < HASH; k += NT) table[k] = -1;
    for (int k = threadIdx.x; k < TILE_LIST; k += NT) sorted[k] = 0x7fffffff;
    if (threadIdx.x == 0) found = placed = 0;
    __syncthreads();
    for (int k = h; k < row.y; k += TILE_LANES) {
        // past the limit nothing more is entered: each thread adds one node at
        // most after it, so the table (4 TILE_LIST) always has free places
        if (__hip_atomic_load(&found, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) > TILE_LIST) break;
        const int j = col[beg + k];
        unsigned p = (static_cast<unsigned>(j) * 2654435761u) >> 19;
        static_assert(HASH == 1 << 13, "the hash keeps 13 bits");
        while (true) {
            const int was = atomicCAS(&table[p], -1, j);
            if (was == j) break;
            if (was == -1) {
                atomicAdd(&found, 1);
                break;
            }
            p = (p + 1) % HASH;
        }
    }
    __syncthreads();
    const int m = found;
    if (threadIdx.x == 0) count[t] = m <= TILE_LIST ? m : TILE_LIST + 1;
    if (m > TILE_LIST) return;
    for (int k = threadIdx.x; k < HASH; k += NT)
        if (table[k] >= 0) sorted[atomicAdd(&placed, 1)] = table[k];
    __syncthreads();
    for (int w = 2; w <= TILE_LIST; w *= 2)
        for (int d = w / 2; d > 0; d /= 2) {
            for (int k = threadIdx.x; k < TILE_LIST; k += NT) {
                const int other = k ^ d;
                if (other > k) {
                    const int lo = sorted[k], hi = sorted[other];
                    if ((lo > hi) == ((k & w) == 0)) {
                        sorted[k] = hi;
                        sorted[other] = lo;
                    }
                }
            }
            __syncthreads();
        }
    for (int k = threadIdx.x; k < m; k += NT) list[static_cast<int64_t>(t) * TILE_LIST + k] = sorted[k];
    if (!on) return;
    uint16_t *lc = lcol + base[q / TILE_SLICE] + static_cast<int64_t>(threadIdx.x & 63);
    for (int k = h; k < row.y; k += TILE_LANES) {
        const int j = col[beg + k];
        int lo = 0, hi = m - 1;
        while (lo < hi) {
            const int mid = (lo + hi) / 2;
            if (sorted[mid] < j) lo = mid + 1;
            else hi = mid;
        }
        lc[(k / TILE_LANES) * 64] = static_cast<uint16_t>(lo);
    }
}

void launch_tile_lists(int nrows, const int2 *rows, const int *base, const int *rowptr, const int *col, int *count,
                       int *list, uint16_t *lcol, hipStream_t s) {
    if (nrows <= 0) return;
    k_tile_lists<<<ceil_div(nrows, TILE_ROWS), NT, 0, s>>>(nrows, rows, base, rowptr, col, count, list, lcol);
    AMG_CHECK_LAUNCH();
}

template <typename V>
__global__ void __launch_bounds__(NT) k_tile_values(int nrows, const int2 *rows, const int *base, const int *rowptr,
                                                    const V *src, V *dst) {
    const int h = threadIdx.x % TILE_LANES, q = blockIdx.x * TILE_ROWS + threadIdx.x / TILE_LANES;
    if (q >= nrows) return;
    const int2 row = rows[q];
    const V *from = src + rowptr[row.x];
    V *to = dst + base[q / TILE_SLICE] + static_cast<int64_t>(threadIdx.x & 63);
    for (int k = h; k < row.y; k += TILE_LANES) to[(k / TILE_LANES) * 64] = from[k];
}

void launch_tile_values(TileKind kind, int nrows, const int2 *rows, const int *base, const int *rowptr,
                        const void *src, void *dst, hipStream_t s) {
    if (nrows <= 0) return;
    const int nb = ceil_div(nrows, TILE_ROWS);
    if (kind == TILE_F64)
        k_tile_values<<<nb, NT, 0, s>>>(nrows, rows, base, rowptr, static_cast<const double *>(src), static_cast<double *>(dst));
    else
        k_tile_values<<<nb, NT, 0, s>>>(nrows, rows, base, rowptr, static_cast<const float *>(src), static_cast<float *>(dst));
    AMG_CHECK_LAUNCH();
}

}  // namespace amgp2
