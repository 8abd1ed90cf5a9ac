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

}  // namespace amgp2
