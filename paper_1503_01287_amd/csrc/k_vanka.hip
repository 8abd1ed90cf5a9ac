// Multiplicative Vanka kernels (see vanka.h): local-matrix assembly, batched
// Gauss-Jordan inversion and the coloured patch update. One workgroup per
// patch; local DOF a < 3 n_P is component a % 3 of node a / 3 of the patch,
// a = 3 n_P is the patch's pressure.
#include "common.h"
#include "vanka.h"

namespace amgp2 {

constexpr int VB = 256;

// position of column c in the sorted row [b, e) of idx, or -1
__device__ __forceinline__ int find_col(const int *idx, int b, int e, int c) {
    int lo = b, hi = e - 1;
    while (lo <= hi) {
        const int mid = (lo + hi) >> 1;
        const int v = idx[mid];
        if (v == c) return mid;
        if (v < c) lo = mid + 1;
        else hi = mid - 1;
    }
    return -1;
}

__global__ void __launch_bounds__(VB) k_vanka_assemble(const VankaView v) {
    extern __shared__ int nodes[];
    const int i = blockIdx.x;
    const int p0 = v.pptr[i], nn = v.pptr[i + 1] - p0;
    for (int k = threadIdx.x; k < nn; k += VB) nodes[k] = v.pnode[p0 + k];
    __syncthreads();
    const int m = 3 * nn + 1;
    double *M = v.inv + v.moff[i];
    for (int64_t e = threadIdx.x; e < static_cast<int64_t>(m) * m; e += VB) {
        const int a = static_cast<int>(e % m), bcol = static_cast<int>(e / m);  // column-major
        double val = 0.0;
        const bool ap = a == 3 * nn, bp = bcol == 3 * nn;
        if (!ap && !bp) {
            const int ua = nodes[a / 3], ub = nodes[bcol / 3];
            const int q = find_col(v.acol, v.arow[ua], v.arow[ua + 1], ub);
            if (q >= 0) val = v.aval[static_cast<int64_t>((a % 3) * 3 + bcol % 3) * v.annz + q];
        } else if (!ap && bp) {  // B^T(u_a, i)[c_a]
            const int ua = nodes[a / 3];
            const int q = find_col(v.btcol, v.btrow[ua], v.btrow[ua + 1], i);
            if (q >= 0) val = v.btval[static_cast<int64_t>(a % 3) * v.btnnz + q];
        } else if (ap && !bp) {  // B(i, u_b)[c_b] = B^T(u_b, i)[c_b]
            const int ub = nodes[bcol / 3];
            const int q = find_col(v.btcol, v.btrow[ub], v.btrow[ub + 1], i);
            if (q >= 0) val = v.btval[static_cast<int64_t>(bcol % 3) * v.btnnz + q];
        } else if (v.crow) {     // -C(i, i)
            const int q = find_col(v.ccol, v.crow[i], v.crow[i + 1], i);
            if (q >= 0) val = -v.cval[q];
        }
        M[e] = val;
    }
}

void launch_vanka_assemble(const VankaView &v, int max_nodes, hipStream_t s) {
    if (v.npatch <= 0) return;
    k_vanka_assemble<<<v.npatch, VB, max_nodes * sizeof(int), s>>>(v);
    AMG_CHECK_LAUNCH();
}

// In-place Gauss-Jordan inversion with partial (row) pivoting of one
// column-major m x m matrix per workgroup; row swaps are undone as column
// swaps at the end.
__global__ void __launch_bounds__(VB) k_vanka_invert(const VankaView v, int *flag) {
    extern __shared__ unsigned char smem[];
    __shared__ double rv[VB];
    __shared__ int ri[VB];
    const int i = blockIdx.x;
    const int m = 3 * (v.pptr[i + 1] - v.pptr[i]) + 1;
    double *f = reinterpret_cast<double *>(smem);
    int *perm = reinterpret_cast<int *>(f + m);
    double *M = v.inv + v.moff[i];
    auto E = [&](int r, int c) -> double & { return M[static_cast<int64_t>(c) * m + r]; };
    for (int k = 0; k < m; ++k) {
        double best = -1.0;
        int bi = k;
        for (int r = k + threadIdx.x; r < m; r += VB) {
            const double a = fabs(E(r, k));
            if (a > best) {
                best = a;
                bi = r;
            }
        }
        rv[threadIdx.x] = best;
        ri[threadIdx.x] = bi;
        __syncthreads();
        for (int o = VB / 2; o > 0; o >>= 1) {
            if (threadIdx.x < o) {
                const double b2 = rv[threadIdx.x + o];
                const int i2 = ri[threadIdx.x + o];
                if (b2 > rv[threadIdx.x] || (b2 == rv[threadIdx.x] && i2 < ri[threadIdx.x])) {
                    rv[threadIdx.x] = b2;
                    ri[threadIdx.x] = i2;
                }
            }
            __syncthreads();
        }
        const int piv = ri[0];
        const bool zero = rv[0] == 0.0;
        __syncthreads();
        if (zero) {
            if (threadIdx.x == 0) atomicOr(flag, 1);
            return;  // uniform across the workgroup
        }
        if (threadIdx.x == 0) perm[k] = piv;
        if (piv != k)
            for (int c = threadIdx.x; c < m; c += VB) {
                const double t = E(k, c);
                E(k, c) = E(piv, c);
                E(piv, c) = t;
            }
        __syncthreads();
        const double p = E(k, k);
        for (int r = threadIdx.x; r < m; r += VB) f[r] = E(r, k);
        __syncthreads();
        for (int r = threadIdx.x; r < m; r += VB) E(r, k) = r == k ? 1.0 : 0.0;
        __syncthreads();
        for (int c = threadIdx.x; c < m; c += VB) E(k, c) /= p;
        __syncthreads();
        for (int64_t e = threadIdx.x; e < static_cast<int64_t>(m) * m; e += VB) {
            const int r = static_cast<int>(e % m), c = static_cast<int>(e / m);
            if (r != k) E(r, c) -= f[r] * E(k, c);
        }
        __syncthreads();
    }
    for (int k = m - 1; k >= 0; --k) {
        const int q = perm[k];
        if (q != k)
            for (int r = threadIdx.x; r < m; r += VB) {
                const double t = E(r, k);
                E(r, k) = E(r, q);
                E(r, q) = t;
            }
        __syncthreads();
    }
}

void launch_vanka_invert(const VankaView &v, int max_m, int *flag, hipStream_t s) {
    if (v.npatch <= 0) return;
    k_vanka_invert<<<v.npatch, VB, static_cast<size_t>(max_m) * (sizeof(double) + sizeof(int)), s>>>(v, flag);
    AMG_CHECK_LAUNCH();
}

// Descriptors of the residual rows: from where a row's entries are read, so
// that a row's chain of loads is descriptor, column, x.
__global__ void __launch_bounds__(VB) k_vanka_rows(const VankaView v, int nrows, const int2 *rown, int4 *rowa) {
    const int t = blockIdx.x * VB + threadIdx.x;
    if (t >= nrows) return;
    const int u = rown[t].x;
    if (u >= 0)
        rowa[t] = make_int4(v.arow[u], v.arow[u + 1], v.btrow[u], v.btrow[u + 1]);
    else
        rowa[t] = make_int4(v.brow[~u], v.brow[~u + 1], v.crow ? v.crow[~u] : 0, v.crow ? v.crow[~u + 1] : 0);
}

void launch_vanka_rows(const VankaView &v, int nrows, const int2 *rown, int4 *rowa, hipStream_t s) {
    if (nrows <= 0) return;
    k_vanka_rows<<<ceil_div(nrows, VB), VB, 0, s>>>(v, nrows, rown, rowa);
    AMG_CHECK_LAUNCH();
}

// 64 rows of one patch's correction per workgroup: lane = row, the NW
// wavefronts take 1 / NW of the columns each, partial sums added in LDS in
// wavefront order. Bound by the read of the inverses on fine levels and by
// the chain tile, residual and columns, LDS, x on coarse ones: the tile's
// descriptor, the residual's values (64 a load, broadcast from the lanes)
// and the entries of x are loaded ahead of the columns that they meet.
template <int NW>
__global__ void __launch_bounds__(64 * NW) k_vanka_apply(const VankaView v, const VankaTile *tile, const double *rbuf,
                                                         double *x, double omega) {
    __shared__ double part[NW][64];
    const VankaTile t = tile[blockIdx.x];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int a = t.row0 + lane, m = t.m;
    int64_t at = 0;
    double old = 0.0;
    if (wave == 0 && a < m) {
        // (no other patch of the colour touches these entries)
        at = a < m - 1 ? 3 * static_cast<int64_t>(v.pnode[t.node0 + a / 3]) + a % 3 : 3 * static_cast<int64_t>(v.n) + t.patch;
        old = x[at];
    }
    const double *r = rbuf + t.res;
    const double *M = v.inv + t.inv;
    const int c0 = wave * m / NW, c1 = (wave + 1) * m / NW;
    const int ar = a < m ? a : m - 1;
    double acc = 0.0;
    for (int cb = c0; cb < c1; cb += 64) {
        const int nc = c1 - cb < 64 ? c1 - cb : 64;
        const double rl = lane < nc ? r[cb + lane] : 0.0;
        int u = 0;
        for (; u + 16 <= nc; u += 16) {
            double mv[16];
#pragma unroll
            for (int k = 0; k < 16; ++k) mv[k] = M[static_cast<int64_t>(cb + u + k) * m + ar];
#pragma unroll
            for (int k = 0; k < 16; ++k) acc += mv[k] * __shfl(rl, u + k, 64);
        }
        if (u < nc) {
            double mv[16];
#pragma unroll
            for (int k = 0; k < 16; ++k) mv[k] = u + k < nc ? M[static_cast<int64_t>(cb + u + k) * m + ar] : 0.0;
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                const double rk = __shfl(rl, u + k < 64 ? u + k : 63, 64);
                if (u + k < nc) acc += mv[k] * rk;
            }
        }
    }
    part[wave][lane] = acc;
    __syncthreads();
    if (wave != 0 || a >= m) return;
    double sum = part[0][lane];
#pragma unroll
    for (int w = 1; w < NW; ++w) sum += part[w][lane];
    x[at] = old + omega * sum;
}

// Partial corrections of one colour's large patches, tiled in two dimensions
// so that a colour of few, large patches still fills the GPU: workgroup u
// takes 64 rows (row tile rt) and a chunk of cc columns (chunk q) of one
// patch's inverse (upre: prefix of the units ceil(m_i / 64) ceil(m_i / cc)
// over the colour's patches, rt fastest); its 4 wavefronts take a quarter of
// the chunk each, eight column loads in flight per lane, and their sums are
// added in a fixed order into pbuf (chunk q of patch i at pbuf + poff[i] +
// q m_i).
__global__ void __launch_bounds__(VB) k_vanka_apply_part(const VankaView v, const int *order, const int *upre,
                                                         int count, int cc, const int64_t *roff, const double *rbuf,
                                                         const int64_t *poff, double *pbuf) {
    __shared__ double part[4][64];
    int lo = 0, hi = count - 1;
    const int u = blockIdx.x;
    while (lo < hi) {  // last patch whose first unit is <= u
        const int mid = (lo + hi + 1) >> 1;
        if (upre[mid] <= u) lo = mid;
        else hi = mid - 1;
    }
    const int i = order[lo];
    const int m = 3 * (v.pptr[i + 1] - v.pptr[i]) + 1;
    const int RT = (m + 63) / 64;
    const int local = u - upre[lo];
    const int rt = local % RT, q = local / RT;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int a = rt * 64 + lane;
    const int c0 = q * cc, c1 = min(m, c0 + cc);
    const int w0 = c0 + wave * (c1 - c0) / 4, w1 = c0 + (wave + 1) * (c1 - c0) / 4;
    const double *r = rbuf + roff[i];
    const double *M = v.inv + v.moff[i];
    double acc = 0.0;
    if (a < m) {
        int c = w0;
        for (; c + 8 <= w1; c += 8) {
            double mv[8], rv[8];
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                mv[t] = M[static_cast<int64_t>(c + t) * m + a];
                rv[t] = r[c + t];
            }
#pragma unroll
            for (int t = 0; t < 8; ++t) acc += mv[t] * rv[t];
        }
        for (; c < w1; ++c) acc += M[static_cast<int64_t>(c) * m + a] * r[c];
    }
    part[wave][lane] = acc;
    __syncthreads();
    if (wave == 0 && a < m) pbuf[poff[i] + static_cast<int64_t>(q) * m + a] = ((part[0][lane] + part[1][lane]) +
                                                                               part[2][lane]) + part[3][lane];
}

// x_P += omega (sum of the chunks' partials, in chunk order) over 64-row tiles
// (tpre: prefix of ceil(m_i / 64) over the colour's patches)
__global__ void __launch_bounds__(64) k_vanka_reduce(const VankaView v, const int *order, const int *tpre,
                                                     int count, int cc, const int64_t *poff, const double *pbuf,
                                                     double *x, double omega) {
    int lo = 0, hi = count - 1;
    const int t = blockIdx.x;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (tpre[mid] <= t) lo = mid;
        else hi = mid - 1;
    }
    const int i = order[lo];
    const int p0 = v.pptr[i], nn = v.pptr[i + 1] - p0;
    const int m = 3 * nn + 1;
    const int a = (t - tpre[lo]) * 64 + threadIdx.x;
    if (a >= m) return;
    const int kc = (m + cc - 1) / cc;
    double sum = 0.0;
    for (int q = 0; q < kc; ++q) sum += pbuf[poff[i] + static_cast<int64_t>(q) * m + a];
    const double d = omega * sum;
    if (a < 3 * nn) x[3 * static_cast<int64_t>(v.pnode[p0 + a / 3]) + a % 3] += d;
    else x[3 * static_cast<int64_t>(v.n) + i] += d;
}

// Residuals of one colour's patches: G lanes per row, a patch's rows its
// velocity nodes and last its pressure. Row-to-row chains bound it (a colour
// holds a few thousand rows at most), so nothing is searched: descriptor,
// columns of A and B^T together, x, two entries of A per lane in flight.
template <int G>
__global__ void __launch_bounds__(VB) k_vanka_resid_rows(const VankaView v, int nrows, const int2 *rown,
                                                         const int4 *rowa, double *rbuf, const double *b,
                                                         const double *x) {
    const int t = (blockIdx.x * VB + threadIdx.x) / G, lane = threadIdx.x % G;
    if (t >= nrows) return;  // whole G-lane groups leave together
    const int2 rn = rown[t];
    const int4 ra = rowa[t];
    const int64_t nu = 3 * static_cast<int64_t>(v.n);
    const double *p = x + nu;
    const int u = rn.x;
    double s0 = 0.0, s1 = 0.0, s2 = 0.0;
    if (u >= 0) {
        const double bi = lane < 3 ? b[3 * static_cast<int64_t>(u) + lane] : 0.0;
        int q = ra.x + lane, w = ra.z + lane;
        int j0 = q < ra.y ? v.acol[q] : -1, j1 = q + G < ra.y ? v.acol[q + G] : -1;
        const int jb = w < ra.w ? v.btcol[w] : -1;
        for (; q < ra.y; q += 2 * G) {
            const double *x0 = x + 3 * static_cast<int64_t>(j0 < 0 ? 0 : j0), *x1 = x + 3 * static_cast<int64_t>(j1 < 0 ? 0 : j1);
            double e0[9], e1[9], y0[3], y1[3];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                y0[k] = x0[k];
                y1[k] = j1 < 0 ? 0.0 : x1[k];
            }
#pragma unroll
            for (int k = 0; k < 9; ++k) {
                e0[k] = v.aval[k * v.annz + q];
                e1[k] = j1 < 0 ? 0.0 : v.aval[k * v.annz + q + G];
            }
            s0 += e0[0] * y0[0] + e0[1] * y0[1] + e0[2] * y0[2];
            s1 += e0[3] * y0[0] + e0[4] * y0[1] + e0[5] * y0[2];
            s2 += e0[6] * y0[0] + e0[7] * y0[1] + e0[8] * y0[2];
            if (j1 >= 0) {
                s0 += e1[0] * y1[0] + e1[1] * y1[1] + e1[2] * y1[2];
                s1 += e1[3] * y1[0] + e1[4] * y1[1] + e1[5] * y1[2];
                s2 += e1[6] * y1[0] + e1[7] * y1[1] + e1[8] * y1[2];
            }
            j0 = q + 2 * G < ra.y ? v.acol[q + 2 * G] : -1;
            j1 = q + 3 * G < ra.y ? v.acol[q + 3 * G] : -1;
        }
        for (; w < ra.w; w += G) {
            const double pq = p[w == ra.z + lane ? jb : v.btcol[w]];
            s0 += v.btval[w] * pq;
            s1 += v.btval[v.btnnz + w] * pq;
            s2 += v.btval[2 * v.btnnz + w] * pq;
        }
#pragma unroll
        for (int o = G / 2; o > 0; o >>= 1) {
            s0 += __shfl_xor(s0, o, G);
            s1 += __shfl_xor(s1, o, G);
            s2 += __shfl_xor(s2, o, G);
        }
        if (lane < 3) rbuf[rn.y + lane] = bi - (lane == 0 ? s0 : (lane == 1 ? s1 : s2));
    } else {
        // pressure row: g_i - B_i u + C_i p
        const double bi = lane == 0 ? b[nu + ~u] : 0.0;
        for (int q = ra.x + lane; q < ra.y; q += G) {
            const int64_t j = v.bcol[q];
            s0 += v.bval[q] * x[3 * j] + v.bval[v.bnnz + q] * x[3 * j + 1] + v.bval[2 * v.bnnz + q] * x[3 * j + 2];
        }
        for (int q = ra.z + lane; q < ra.w; q += G) s0 -= v.cval[q] * p[v.ccol[q]];
#pragma unroll
        for (int o = G / 2; o > 0; o >>= 1) s0 += __shfl_xor(s0, o, G);
        if (lane == 0) rbuf[rn.y] = bi - s0;
    }
}

static void resid_rows(const VankaView &v, const VankaColour &c, int rg, double *rbuf, const double *b,
                       const double *x, hipStream_t s) {
    const int nb = ceil_div(static_cast<int64_t>(c.nrows) * rg, VB);
    switch (rg) {
        case 16: k_vanka_resid_rows<16><<<nb, VB, 0, s>>>(v, c.nrows, c.rown, c.rowa, rbuf, b, x); break;
        case 32: k_vanka_resid_rows<32><<<nb, VB, 0, s>>>(v, c.nrows, c.rown, c.rowa, rbuf, b, x); break;
        case 64: k_vanka_resid_rows<64><<<nb, VB, 0, s>>>(v, c.nrows, c.rown, c.rowa, rbuf, b, x); break;
        default: throw Error(AMG_EINVAL, "Vanka residual: 16, 32 or 64 lanes per row");
    }
    AMG_CHECK_LAUNCH();
}

void launch_vanka_colour_rows(const VankaView &v, const VankaColour &c, int rg, int aw, double *rbuf,
                              const double *b, double *x, double omega, hipStream_t s) {
    if (c.count <= 0) return;
    resid_rows(v, c, rg, rbuf, b, x, s);
    switch (aw) {
        case 4: k_vanka_apply<4><<<c.ntiles, 256, 0, s>>>(v, c.tile, rbuf, x, omega); break;
        case 8: k_vanka_apply<8><<<c.ntiles, 512, 0, s>>>(v, c.tile, rbuf, x, omega); break;
        case 16: k_vanka_apply<16><<<c.ntiles, 1024, 0, s>>>(v, c.tile, rbuf, x, omega); break;
        default: throw Error(AMG_EINVAL, "Vanka corrections: 4, 8 or 16 wavefronts per tile");
    }
    AMG_CHECK_LAUNCH();
}

void launch_vanka_colour_tiled(const VankaView &v, const VankaColour &c, const int *order, const int *tpre,
                               const int *upre, int nunits, int cc, int rg, const int64_t *roff, double *rbuf,
                               const int64_t *poff, double *pbuf, const double *b, double *x, double omega,
                               hipStream_t s) {
    if (c.count <= 0) return;
    resid_rows(v, c, rg, rbuf, b, x, s);
    k_vanka_apply_part<<<nunits, VB, 0, s>>>(v, order, upre, c.count, cc, roff, rbuf, poff, pbuf);
    AMG_CHECK_LAUNCH();
    k_vanka_reduce<<<c.ntiles, 64, 0, s>>>(v, order, tpre, c.count, cc, poff, pbuf, x, omega);
    AMG_CHECK_LAUNCH();
}

// ------------------------------------------------- all colours in one launch
// Two launches per colour cost 5 to 7 us each, most of it the launch and a
// chain of dependent loads; a colour has 5 to 40 patches, well under 2 us of
// bandwidth. Here the workgroups stay for the whole sweep and take items
// from a ticket counter: a colour's residual rows, then its patches'
// corrections. An item loads what does not depend on the others (operator
// entries, columns of the inverse, 100 of its 128 registers a lane), waits
// for the values that do, and stores its own at device scope (sc1, which the
// 8 XCDs see alike). A value that is not there yet holds a NaN of a fixed
// payload, as in the Gauss-Seidel sweeps: an unknown has a place for every
// patch that it is in, so each place is written once in a sweep, and a reader
// knows (VankaSweep::entry) whose place holds the value of its colour. Two
// buffers of places: a sweep uses one and fills the other with the payload;
// the last workgroup out turns them over.
//
// Progress: an item waits only for items of smaller tickets, and a ticket is
// taken by a running workgroup, so the smallest unfinished one never waits,
// whatever part of the grid is resident. The waits are bounded all the same;
// past the bound the values become NaN, which the Krylov loops report as
// divergence.
//
// What bounds it: two trips to memory a colour (residual to corrections,
// corrections to the next colour's residual), 4.2 us in all on small levels;
// with many patches a colour also how many items are in flight ahead of it,
// so items are large (1024 threads; 49 rows of an inverse a wavefront, four
// or two groups of rows where 26 columns a lane cover it) and a residual row
// has 32 lanes, 64 only past 64 entries. Where it has more than two entries
// a lane, the last written are its last. us per sweep, launches per colour ->
// this kernel, mixed elasticity:
//    4^3 level 0 (  125 patches, 44 colours)   358 -> 182
//    8^3 level 0 (  729 patches, 59 colours)   530 -> 251
//   12^3 level 0 (2,197 patches, 62 colours)   738 -> 353
//   12^3 level 1 (  343 patches, 72 colours)   865 -> 398
//   16^3 level 0 (4,913 patches)             1,051 -> 631
// (64 lanes for every row: 12^3 425 and 415; two workgroups of 512 threads to
// a CU: 535 and 437; 64-row tiles of every inverse: 461 and 408; 50 columns a
// lane spill: 1,134.)
namespace {

constexpr int SWEEP_WAVES = 16;
constexpr unsigned SPIN_MAX = 1u << 21;  // a second or two of polls
constexpr uint64_t ABSENT = 0x7ffdead0beef0001ull;  // payload of "not there yet" (a quiet NaN)

template <typename T>
__device__ __forceinline__ T agent_load(const T *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ void agent_store(T *p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double absent() { return __longlong_as_double(static_cast<long long>(ABSENT)); }
__device__ __forceinline__ bool is_absent(double v) { return static_cast<uint64_t>(__double_as_longlong(v)) == ABSENT; }
__device__ __forceinline__ double present(double v, bool bad) { return bad || is_absent(v) ? __builtin_nan("") : v; }

__device__ __forceinline__ double lane_value(double v, int k) {
    const uint64_t w = static_cast<uint64_t>(__double_as_longlong(v));
    const uint32_t lo = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(w), k));
    const uint32_t hi = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(w >> 32), k));
    return __longlong_as_double(static_cast<long long>(static_cast<uint64_t>(hi) << 32 | lo));
}

// sum over each 32 lanes, in the order of a butterfly: 4 of its 5 steps
// without a trip through LDS
template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
    const uint64_t w = static_cast<uint64_t>(__double_as_longlong(v));
    const uint32_t lo = static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(w), CTRL, 0xf, 0xf, true));
    const uint32_t hi = static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(w >> 32), CTRL, 0xf, 0xf, true));
    return __longlong_as_double(static_cast<long long>(static_cast<uint64_t>(hi) << 32 | lo));
}
__device__ __forceinline__ double sum32(double v) {
    v += dpp<0xb1>(v);   // lane ^ 1 (quad_perm 1, 0, 3, 2)
    v += dpp<0x4e>(v);   // lane ^ 2 (quad_perm 2, 3, 0, 1)
    v += dpp<0x141>(v);  // the other quad of 8 (row_half_mirror)
    v += dpp<0x140>(v);  // the other 8 of 16 (row_mirror)
    return v + __shfl_xor(v, 16, 64);
}

// device-scope loads of a row's unknowns (the buffer's descriptor covers one
// half of xs)
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
constexpr int AUX_SC1 = 16;  // the scope bit of device-scope accesses
__device__ __forceinline__ double from_words(uint32_t lo, uint32_t hi) {
    return __longlong_as_double(static_cast<long long>(static_cast<uint64_t>(hi) << 32 | lo));
}
__device__ __forceinline__ void gather(__amdgpu_buffer_rsrc_t xs, int row, double *v) {
    const u32x4 q = __builtin_amdgcn_raw_buffer_load_b128(xs, 32 * row, 0, AUX_SC1);
    const u32x2 w = __builtin_amdgcn_raw_buffer_load_b64(xs, 32 * row + 16, 0, AUX_SC1);
    v[0] = from_words(q.x, q.y);
    v[1] = from_words(q.z, q.w);
    v[2] = from_words(w.x, w.y);
}

// load() until it is true in every lane, or the bound is reached (bad)
template <typename Load>
__device__ __forceinline__ void wait_for(Load &&load, int *gave_up, int sweep, bool &bad) {
    bool there = false;
    unsigned n = 0;
    for (;;) {
        if (!there) {
            asm volatile("" ::: "memory");  // a new load every time
            there = load();
        }
        if (__all(there) || bad) break;
        if ((++n & 0xfff) == 0) {
            if (n > SPIN_MAX) agent_store(gave_up, sweep);
            bad = agent_load(gave_up) == sweep;
        }
        if (n > 2) __builtin_amdgcn_s_sleep(1);
    }
}

}  // namespace

__global__ void __launch_bounds__(64 * SWEEP_WAVES, 4) k_vanka_sweep(const VankaView v, const VankaSweep a) {
    constexpr int NW = SWEEP_WAVES;
    constexpr int U = 2;    // entries per lane loaded before the wait
    constexpr int KC = 26;  // columns of an inverse per lane loaded before the wait
    __shared__ int sh_ticket[2];
    __shared__ double part[NW][64];
    const int tid = threadIdx.x;
    int *const ticket = a.ctl, *const exits = a.ctl + 32, *const turn = a.ctl + 64, *const gave_up = a.ctl + 96;
    int next = 0;
    if (tid == 0) {
        next = atomicAdd(ticket, 1);
        sh_ticket[0] = next;
        next = atomicAdd(ticket, 1);
    }
    const unsigned sweep = static_cast<unsigned>(*turn) + 1u;  // this sweep's number, from 1 on
    const int which = (sweep & 1u) == 0u;
    double *const xs = a.xs + (which ? a.xs_half : 0), *const xfill = a.xs + (which ? 0 : a.xs_half);
    double *const rs = a.rs + (which ? a.rs_half : 0), *const rfill = a.rs + (which ? 0 : a.rs_half);
    const __amdgpu_buffer_rsrc_t xsr =
        __builtin_amdgcn_make_buffer_rsrc(xs, 0, static_cast<int>(a.xs_half * sizeof(double)), 0x00027000);
    const int64_t nu = 3 * static_cast<int64_t>(v.n);
    __syncthreads();
    bool bad = false;
    int t = sh_ticket[0], phase = 1;
    // an item and what it is described by, loaded while the one before it
    // waits
    int2 it = make_int2(0, 0);
    VankaRow row_next;
    VankaTile tl_next;
    auto fetch = [&](int k) {
        if (k >= a.nitems) return;
        it = a.item[k];
        it.x = __builtin_amdgcn_readfirstlane(it.x);
        it.y = __builtin_amdgcn_readfirstlane(it.y);
        if (it.x >= 0) {
            const int grp = tid / (it.y > 0 ? 32 : 64), count = it.y > 0 ? it.y : -it.y;
            row_next = a.row[it.x + (grp < count ? grp : 0)];
        } else {
            tl_next = a.tile[~it.x];
        }
    };
    fetch(t);
    while (t < a.nitems) {
        if (tid == 0) sh_ticket[phase] = next;
        __syncthreads();
        const int t_next = sh_ticket[phase];
        phase ^= 1;
        if (tid == 0 && t_next < a.nitems) next = atomicAdd(ticket, 1);
        const int2 item = it;
        const VankaRow rd = row_next;
        const VankaTile tl = tl_next;
        fetch(t_next);
        t = t_next;
        if (item.x >= 0) {
            // residual rows, 32 or 64 lanes each
            const int G = item.y > 0 ? 32 : 64, lane = tid & (G - 1), grp = tid / G;
            const bool on = grp < (item.y > 0 ? item.y : -item.y);
            const int2 rn = make_int2(rd.node, rd.res);
            const int4 ra = rd.entries;
            const int p0 = rd.first;
            const bool vel = rn.x >= 0;
            const int n0 = ra.y - ra.x, n1 = on ? n0 + ra.w - ra.z : 0;  // entries of A (B), and with those of B^T (C)
            const int comps = vel ? 3 : 1;
            double bc = 0.0;
            if (on && lane < comps) {
                bc = a.b[vel ? 3 * static_cast<int64_t>(rn.x) + lane : nu + ~rn.x];
                rfill[rn.y + lane] = absent();
            }
            double s0 = 0.0, s1 = 0.0, s2 = 0.0;
            for (int k = lane; __any(k < n1); k += U * G) {
                int j[U];
                bool first[U];  // an entry of A or B (its column is a node), else of B^T or C
                double e[U][9], y[U][3];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int ku = k + u * G;
                    const bool in = ku < n1;
                    const int2 en = in ? a.entry[p0 + ku] : make_int2(0, 0);
                    first[u] = en.y < n0;
                    j[u] = en.x;
#pragma unroll
                    for (int q = 0; q < 9; ++q) e[u][q] = 0.0;
                    y[u][0] = y[u][1] = y[u][2] = 0.0;
                    if (in) {
                        if (vel) {
                            if (first[u]) {
#pragma unroll
                                for (int q = 0; q < 9; ++q) e[u][q] = v.aval[q * v.annz + ra.x + en.y];
                            } else {
#pragma unroll
                                for (int q = 0; q < 3; ++q) e[u][3 * q] = v.btval[q * v.btnnz + ra.z + en.y - n0];
                            }
                        } else if (first[u]) {
#pragma unroll
                            for (int q = 0; q < 3; ++q) e[u][q] = v.bval[q * v.bnnz + ra.x + en.y];
                        } else {
                            e[u][0] = -v.cval[ra.z + en.y - n0];
                        }
                        if (j[u] < 0) {  // no patch of an earlier colour has it
                            const int64_t at = first[u] ? 3 * static_cast<int64_t>(~j[u]) : nu + ~j[u];
                            y[u][0] = a.x_old[at];
                            if (first[u]) {
                                y[u][1] = a.x_old[at + 1];
                                y[u][2] = a.x_old[at + 2];
                            }
                        }
                    }
                }
                // most of them were written a while ago: an ordinary load finds
                // these, in the L2 for its XCD's other rows. (It never finds an
                // earlier sweep's: the launch before this one wrote "absent"
                // over them.) The others are waited for at device scope.
                bool got[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    got[u] = k + u * G >= n1 || j[u] < 0;
                    if (!got[u]) {
                        const double *q = xs + 4 * static_cast<int64_t>(j[u]);
                        y[u][0] = q[0];
                        if (first[u]) {
                            y[u][1] = q[1];
                            y[u][2] = q[2];
                        }
                        got[u] = !is_absent(y[u][0]) && !is_absent(y[u][1]) && !is_absent(y[u][2]);
                    }
                }
                wait_for(
                    [&] {
#pragma unroll
                        for (int u = 0; u < U; ++u)
                            if (!got[u]) {
                                gather(xsr, j[u], y[u]);
                                got[u] = !is_absent(y[u][0]) && (!first[u] || (!is_absent(y[u][1]) && !is_absent(y[u][2])));
                            }
                        bool there = true;
#pragma unroll
                        for (int u = 0; u < U; ++u) there = there && got[u];
                        return there;
                    },
                    gave_up, static_cast<int>(sweep), bad);
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (k + u * G < n1) {
                        if (vel && first[u]) {
                            s0 += e[u][0] * y[u][0] + e[u][1] * y[u][1] + e[u][2] * y[u][2];
                            s1 += e[u][3] * y[u][0] + e[u][4] * y[u][1] + e[u][5] * y[u][2];
                            s2 += e[u][6] * y[u][0] + e[u][7] * y[u][1] + e[u][8] * y[u][2];
                        } else if (vel) {
                            s0 += e[u][0] * y[u][0];
                            s1 += e[u][3] * y[u][0];
                            s2 += e[u][6] * y[u][0];
                        } else if (first[u]) {
                            s0 += e[u][0] * y[u][0] + e[u][1] * y[u][1] + e[u][2] * y[u][2];
                        } else {
                            s0 += e[u][0] * y[u][0];
                        }
                    }
            }
            s0 = sum32(s0);
            s1 = sum32(s1);
            s2 = sum32(s2);
            if (G == 64) {
                s0 += __shfl_xor(s0, 32, 64);
                s1 += __shfl_xor(s1, 32, 64);
                s2 += __shfl_xor(s2, 32, 64);
            }
            if (on && lane < comps) agent_store(rs + rn.y + lane, present(bc - (lane == 0 ? s0 : (lane == 1 ? s1 : s2)), bad));
        } else {
            // rows row0 .. of a patch's correction: RG groups of up to 64, the
            // columns split over the wavefronts of each
            const int wave = tid >> 6, l64 = tid & 63, m = tl.m;
            const int RG = tl.groups, CG = NW / RG, rg = wave % RG, cg = wave / RG;
            const int width = (tl.rows + RG - 1) / RG, local = rg * width + l64;
            const bool in = l64 < width && local < tl.rows;
            const int r = tl.row0 + (in ? local : 0);
            const bool mine = in && cg == 0;
            double old = 0.0;
            int2 own = make_int2(0, 0);
            int64_t at = 0;
            int slot = 0;
            if (mine) {
                const int row = tl.row + r / 3;
                own = a.own[row];
                at = r < m - 1 ? 3 * static_cast<int64_t>(a.rown[row].x) + r % 3 : nu + tl.patch;
                slot = 4 * row + r % 3;
                xfill[slot] = absent();
                if (own.x < 0) old = a.x_old[at];
            }
            const double *M = v.inv + tl.inv + r;
            // (the first column group has columns whatever m is)
            const int per = (m + CG - 1) / CG, c0 = min(cg * per, m), c1 = min(c0 + per, m);
            double acc = 0.0;
            for (int c = c0; c < c1; c += KC) {
                const int nc = c1 - c < KC ? c1 - c : KC;
                double mv[KC];
#pragma unroll
                for (int k = 0; k < KC; ++k) mv[k] = k < nc ? M[static_cast<int64_t>(c + k) * m] : 0.0;
                double rl = 0.0;
                wait_for(
                    [&] {
                        if (l64 < nc) rl = agent_load(rs + tl.res + c + l64);
                        if (mine && own.x >= 0) old = agent_load(xs + 4 * static_cast<int64_t>(own.x) + r % 3);
                        return !is_absent(rl) && (own.x < 0 || !is_absent(old));
                    },
                    gave_up, static_cast<int>(sweep), bad);
#pragma unroll
                for (int k = 0; k < KC; ++k)
                    if (k < nc) acc += mv[k] * lane_value(rl, k);
            }
            part[wave][l64] = acc;
            __syncthreads();
            if (mine) {
                double sum = part[rg][l64];
                for (int w = 1; w < CG; ++w) sum += part[rg + w * RG][l64];
                const double xn = present(old + a.omega * sum, bad);
                agent_store(xs + slot, xn);
                if (own.y) a.x[at] = xn;
            }
            // (part is written again only past the loop's barrier)
        }
    }
    // The last workgroup out readies the control words for the next sweep. Other
    // wavefronts of a workgroup that has counted itself out may still wait, and
    // give up, so the flag is not cleared: it names the sweep that set it. (A
    // barrier before the count cost 0.2 to 0.4 us a sweep.)
    if (tid == 0 && atomicAdd(exits, 1) == static_cast<int>(gridDim.x) - 1) {
        agent_store(ticket, 0);
        agent_store(exits, 0);
        agent_store(turn, static_cast<int>(sweep));
    }
}

void launch_vanka_sweep(const VankaView &v, const VankaSweep &a, int grid, hipStream_t s) {
    if (a.nitems <= 0) return;
    AMG_REQUIRE(a.x != a.x_old, AMG_EINVAL, "Vanka sweep: in place");
    k_vanka_sweep<<<grid, 64 * SWEEP_WAVES, 0, s>>>(v, a);
    AMG_CHECK_LAUNCH();
}

// One wavefront per residual row. The last writer before the row's colour is
// the last of the column's list (by colour) below it; entries are ranked by
// it, so that a row's later trips are those that wait (a row of more entries
// than LDS holds here keeps its order).
constexpr int RANKED = 1024;
__global__ void __launch_bounds__(VB) k_vanka_entries(const VankaView v, int nrows, const int2 *rown, const int4 *rowa,
                                                      const int *pptr, const int *colour, const int *nptr,
                                                      const int2 *writer, int2 *entry, int2 *own) {
    __shared__ int keys[VB / 64][RANKED];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, row = blockIdx.x * (VB / 64) + wave;
    const bool on = row < nrows;
    const int u = on ? rown[row].x : 0, c = on ? colour[row] : 0;
    const int4 ra = on ? rowa[row] : make_int4(0, 0, 0, 0);
    const int n0 = ra.y - ra.x, n1 = n0 + ra.w - ra.z;
    int2 *const mine = entry + (on ? pptr[row] : 0);
    for (int k = lane; k < n1; k += 64) {
        int j, list;  // the column, the list of its writers
        if (k < n0) {
            j = u >= 0 ? v.acol[ra.x + k] : v.bcol[ra.x + k];
            list = j;
        } else {
            j = u >= 0 ? v.btcol[ra.z + k - n0] : v.ccol[ra.z + k - n0];
            list = v.n + j;
        }
        int at = ~j;
        for (int q = nptr[list]; q < nptr[list + 1] && writer[q].y < c; ++q) at = writer[q].x;
        mine[k] = make_int2(at, k);
        if (n1 <= RANKED) keys[wave][k] = at;
    }
    __syncthreads();
    if (n1 <= RANKED)
        for (int k = lane; k < n1; k += 64) {
            const int key = keys[wave][k];
            int rank = 0;
            for (int q = 0; q < n1; ++q) rank += keys[wave][q] < key || (keys[wave][q] == key && q < k);
            mine[rank] = make_int2(key, k);
        }
    if (on && lane == 0) {
        const int list = u >= 0 ? u : v.n + ~u;
        int2 o = make_int2(~0, 1);
        for (int q = nptr[list]; q < nptr[list + 1]; ++q) {
            if (writer[q].y < c) o.x = writer[q].x;
            if (writer[q].y > c) o.y = 0;
        }
        own[row] = o;
    }
}

void launch_vanka_entries(const VankaView &v, int nrows, const int2 *rown, const int4 *rowa, const int *pptr,
                          const int *colour, const int *nptr, const int2 *writer, int2 *entry, int2 *own,
                          hipStream_t s) {
    if (nrows <= 0) return;
    k_vanka_entries<<<ceil_div(nrows, VB / 64), VB, 0, s>>>(v, nrows, rown, rowa, pptr, colour, nptr, writer, entry, own);
    AMG_CHECK_LAUNCH();
}

__global__ void __launch_bounds__(VB) k_vanka_absent(double *p, int64_t n) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * VB + threadIdx.x;
    if (i < n) p[i] = absent();
}

void launch_vanka_absent(double *p, int64_t n, hipStream_t s) {
    if (n <= 0) return;
    k_vanka_absent<<<ceil_div(n, VB), VB, 0, s>>>(p, n);
    AMG_CHECK_LAUNCH();
}

}  // namespace amgp2
