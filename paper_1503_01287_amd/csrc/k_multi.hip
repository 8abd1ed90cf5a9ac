// Kernels for blocks of K right-hand sides on one SPD hierarchy (multi.h):
// the row kernels of k_row.hip / k_mixed.hip with K interleaved vectors, so
// each stored entry (and its column index) is read once for all K, the
// dense coarse-end GEMV with K columns, and the Krylov vector work with one
// scalar per right-hand side.
#include <type_traits>

#include "common.h"
#include "multi.h"

namespace amgp2 {

constexpr int TB = 256;

template <int VK>
using vec_t = typename std::conditional<VK == MK_F64, double, float>::type;

template <int VK>
__device__ __forceinline__ vec_t<VK> ldv(const void *p, int64_t idx) {
    if constexpr (VK == MK_F64)
        return static_cast<const double *>(p)[idx];
    else if constexpr (VK == MK_F32)
        return static_cast<const float *>(p)[idx];
    else
        return __uint_as_float(static_cast<uint32_t>(static_cast<const uint16_t *>(p)[idx]) << 16);
}

template <int G, typename T>
__device__ __forceinline__ T gsum(T v) {
#pragma unroll
    for (int o = G / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, G);
    return v;
}

// One group of G = E K lanes per row. Lane (e, r) = (lane / K, lane % K)
// walks the row's entries e, e + E, ... for right-hand side r, U entries per
// trip (their column indices, then their values and gathers, in flight
// together; entries past the row's end are skipped): the K lanes of one
// entry slot read its column index and values at the same addresses and the
// 3 K contiguous values of x at that column together (x at column j,
// component c, right-hand side r sits at (3 j + c) K + r). The 3 sums of
// every lane are reduced over the E slots in a fixed butterfly order, and the
// slot-0 lanes write their right-hand side's 3 outputs of the row.
template <int MODE, int E, int U, int OP, int VK, int K>
__global__ void __launch_bounds__(TB) k_mrow(const MRowArgs a) {
    using T = vec_t<VK>;
    constexpr int G = E * K;
    static_assert(G <= 64 && (64 % G) == 0, "a row group stays inside one wavefront");
    const int64_t t = static_cast<int64_t>(blockIdx.x) * TB + threadIdx.x;
    const int g = static_cast<int>(t / G), lane = static_cast<int>(t % G);
    if (g >= a.nrows) return;  // whole groups leave together (G divides 64)
    const int e = lane / K, r = lane % K;
    const int i = a.rowid ? a.rowid[g] : g;
    const T *x = static_cast<const T *>(a.x);
    const T *b = static_cast<const T *>(a.b);
    T *y = static_cast<T *>(a.y);
    const T *D = static_cast<const T *>(a.dinv);
    const int64_t o0 = static_cast<int64_t>(3) * i * K + r;  // output (i, 0, r); (i, c, r) at o0 + c K
    constexpr bool NEEDS_B = OP == M_RESID || OP == M_JACOBI || OP == M_GS;
    constexpr bool NEEDS_D = OP == M_JACOBI || OP == M_GS;
    // the epilogue's row operands, loaded before the row's entries so that
    // their latency overlaps the row
    T b0 = T(0), b1 = T(0), b2 = T(0), w0 = T(0), w1 = T(0), w2 = T(0);
    T dm[MODE == 3 ? 9 : 1];
#pragma unroll
    for (int q = 0; q < (MODE == 3 ? 9 : 1); ++q) dm[q] = T(0);
    float q0 = 1.f, q1 = 1.f, q2 = 1.f;
    if (e == 0) {
        if constexpr (NEEDS_B) {
            b0 = b[o0];
            b1 = b[o0 + K];
            b2 = b[o0 + 2 * K];
        }
        if constexpr (NEEDS_D) {
            if constexpr (MODE == 3) {
#pragma unroll
                for (int q = 0; q < 9; ++q) dm[q] = D[q * a.dinv_n + i];
            } else {
                dm[0] = D[i];
            }
        }
        if constexpr (OP == M_SPMV_ADD || OP == M_GS || OP == M_JACOBI) {
            const T *own = OP == M_JACOBI ? x : y;
            w0 = own[o0];
            w1 = own[o0 + K];
            w2 = own[o0 + 2 * K];
        }
        if constexpr (VK == MK_BF16) {
            if constexpr (MODE == 3) {
                q0 = a.rscale[3 * i];
                q1 = a.rscale[3 * i + 1];
                q2 = a.rscale[3 * i + 2];
            } else {
                q0 = q1 = q2 = a.rscale[i];
            }
        }
    }
    T s0 = T(0), s1 = T(0), s2 = T(0);
    const int beg = a.rowptr[g], end = a.rowptr[g + 1];
    const int64_t nz = a.nnz;
    constexpr int NV = MODE == 3 ? 9 : 1;
    for (int k = beg + e; k < end; k += U * E) {
        int j[U];
#pragma unroll
        for (int u = 0; u < U; ++u) j[u] = k + u * E < end ? a.col[k + u * E] : -1;
        T v[U][NV], xv[U][3];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (j[u] >= 0) {
#pragma unroll
                for (int q = 0; q < NV; ++q) v[u][q] = ldv<VK>(a.val, q * nz + k + u * E);
                const T *xj = x + static_cast<int64_t>(3) * j[u] * K + r;
                xv[u][0] = xj[0];
                xv[u][1] = xj[K];
                xv[u][2] = xj[2 * K];
            } else {
#pragma unroll
                for (int q = 0; q < NV; ++q) v[u][q] = T(0);
                xv[u][0] = xv[u][1] = xv[u][2] = T(0);
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if constexpr (MODE == 3) {
                s0 += v[u][0] * xv[u][0] + v[u][1] * xv[u][1] + v[u][2] * xv[u][2];
                s1 += v[u][3] * xv[u][0] + v[u][4] * xv[u][1] + v[u][5] * xv[u][2];
                s2 += v[u][6] * xv[u][0] + v[u][7] * xv[u][1] + v[u][8] * xv[u][2];
            } else {
                s0 += v[u][0] * xv[u][0];
                s1 += v[u][0] * xv[u][1];
                s2 += v[u][0] * xv[u][2];
            }
        }
    }
    // over the entry slots: lanes of one right-hand side differ by multiples of K
#pragma unroll
    for (int o = G / 2; o >= K; o >>= 1) {
        s0 += __shfl_xor(s0, o, G);
        s1 += __shfl_xor(s1, o, G);
        s2 += __shfl_xor(s2, o, G);
    }
    if (e != 0) return;
    if constexpr (VK == MK_BF16) {
        s0 *= q0;
        s1 *= q1;
        s2 *= q2;
    }
    if (a.zero_out) {
        T *z = static_cast<T *>(a.zero_out);
        z[o0] = T(0);
        z[o0 + K] = T(0);
        z[o0 + 2 * K] = T(0);
    }
    T y0, y1, y2;
    if constexpr (OP == M_SPMV) {
        y0 = s0;
        y1 = s1;
        y2 = s2;
    } else if constexpr (OP == M_SPMV_ADD) {
        y0 = w0 + s0;
        y1 = w1 + s1;
        y2 = w2 + s2;
    } else if constexpr (OP == M_RESID) {
        y0 = b0 - s0;
        y1 = b1 - s1;
        y2 = b2 - s2;
    } else {
        const T r0 = b0 - s0, r1 = b1 - s1, r2 = b2 - s2;
        T d0, d1, d2;
        if constexpr (MODE == 3) {
            d0 = dm[0] * r0 + dm[1] * r1 + dm[2] * r2;
            d1 = dm[3] * r0 + dm[4] * r1 + dm[5] * r2;
            d2 = dm[6] * r0 + dm[7] * r1 + dm[8] * r2;
        } else {
            d0 = dm[0] * r0;
            d1 = dm[0] * r1;
            d2 = dm[0] * r2;
        }
        if constexpr (OP == M_JACOBI) {
            const T om = static_cast<T>(a.omega);
            y0 = w0 + om * d0;
            y1 = w1 + om * d1;
            y2 = w2 + om * d2;
        } else {  // M_GS, in place
            y0 = w0 + d0;
            y1 = w1 + d1;
            y2 = w2 + d2;
        }
    }
    y[o0] = y0;
    y[o0 + K] = y1;
    y[o0 + 2 * K] = y2;
}

// 16 lanes per row (E = 16 / K entry slots), 4 entries per slot and trip for
// scalar entries, 2 for 3x3 blocks: the fastest of the shapes measured on
// the 48^3 Laplacian's finest operator with 8 right-hand sides (E in 1..16,
// U in 1..8; 2- and 4-wide vector gathers per lane and per-XCD row chunks
// were slower)
template <int MODE, int OP, int VK, int K>
static void mrow_launch(const MRowArgs &a, hipStream_t s) {
    constexpr int G = 16, E = G / K, U = MODE == 3 ? 2 : 4;
    const int nb = ceil_div(static_cast<int64_t>(a.nrows) * G, TB);
    if (nb == 0) return;
    k_mrow<MODE, E, U, OP, VK, K><<<nb, TB, 0, s>>>(a);
}

template <int MODE, int VK, int K>
static void mrow_op(int op, const MRowArgs &a, hipStream_t s) {
    switch (op) {
        case M_SPMV: mrow_launch<MODE, M_SPMV, VK, K>(a, s); break;
        case M_SPMV_ADD: mrow_launch<MODE, M_SPMV_ADD, VK, K>(a, s); break;
        case M_RESID: mrow_launch<MODE, M_RESID, VK, K>(a, s); break;
        case M_JACOBI: mrow_launch<MODE, M_JACOBI, VK, K>(a, s); break;
        case M_GS: mrow_launch<MODE, M_GS, VK, K>(a, s); break;
        default: throw Error(AMG_EINVAL, "multi row kernel: unknown operation");
    }
}

template <int MODE, int VK>
static void mrow_k(int op, int K, const MRowArgs &a, hipStream_t s) {
    switch (K) {
        case 2: mrow_op<MODE, VK, 2>(op, a, s); break;
        case 4: mrow_op<MODE, VK, 4>(op, a, s); break;
        case 8: mrow_op<MODE, VK, 8>(op, a, s); break;
        case 16:
            // (one entry slot per row: the scalar FP64 operators of the
            // setup's blocked map assembly)
            if constexpr (MODE == 1 && VK == MK_F64) {
                mrow_op<MODE, VK, 16>(op, a, s);
                break;
            }
            [[fallthrough]];
        default: throw Error(AMG_EINVAL, "multi row kernel: K must be 2, 4 or 8 (16: scalar FP64 operators)");
    }
}

template <int MODE>
static void mrow_kind(int op, int kind, int K, const MRowArgs &a, hipStream_t s) {
    switch (kind) {
        case MK_F64: mrow_k<MODE, MK_F64>(op, K, a, s); break;
        case MK_F32: mrow_k<MODE, MK_F32>(op, K, a, s); break;
        case MK_BF16: mrow_k<MODE, MK_BF16>(op, K, a, s); break;
        default: throw Error(AMG_EINVAL, "multi row kernel: unknown value kind");
    }
}

void launch_mrow(int mode, int op, int kind, int K, const MRowArgs &a, hipStream_t s) {
    if (a.nrows <= 0) return;
    if (mode == 3)
        mrow_kind<3>(op, kind, K, a, s);
    else
        mrow_kind<1>(op, kind, K, a, s);
    AMG_CHECK_LAUNCH();
}

// ---------------------------------------------------------------- diagonal solves
// one thread per (node, component, rhs)
template <int MODE, typename T>
__global__ void k_mdiag(int nrows, const int *rowid, const T *dinv, int64_t n, const T *b, T omega, int K, T *x) {
    const int64_t t = static_cast<int64_t>(blockIdx.x) * TB + threadIdx.x;
    if (t >= static_cast<int64_t>(3) * K * nrows) return;
    const int64_t g = t / (3 * K);
    const int rem = static_cast<int>(t - g * 3 * K);
    const int c = rem / K, r = rem % K;
    const int64_t i = rowid ? rowid[g] : g;
    const int64_t base = 3 * i * K;
    T d;
    if constexpr (MODE == 3)
        d = dinv[(3 * c) * n + i] * b[base + r] + dinv[(3 * c + 1) * n + i] * b[base + K + r] +
            dinv[(3 * c + 2) * n + i] * b[base + 2 * K + r];
    else
        d = dinv[i] * b[base + c * K + r];
    x[base + c * K + r] = omega * d;
}

template <typename T>
static void mdiag(int mode, int K, int nrows, const int *rowid, const void *dinv, int64_t n, const void *b,
                  double omega, void *x, hipStream_t s) {
    if (nrows <= 0) return;
    const int nb = ceil_div(static_cast<int64_t>(3) * K * nrows, TB);
    if (mode == 3)
        k_mdiag<3, T><<<nb, TB, 0, s>>>(nrows, rowid, static_cast<const T *>(dinv), n, static_cast<const T *>(b),
                                         static_cast<T>(omega), K, static_cast<T *>(x));
    else
        k_mdiag<1, T><<<nb, TB, 0, s>>>(nrows, rowid, static_cast<const T *>(dinv), n, static_cast<const T *>(b),
                                         static_cast<T>(omega), K, static_cast<T *>(x));
    AMG_CHECK_LAUNCH();
}

void launch_mjacobi_zero(int mode, int kind, int K, int64_t nn, const void *dinv, const void *b, double omega,
                         void *x, hipStream_t s) {
    if (kind == MK_F64)
        mdiag<double>(mode, K, static_cast<int>(nn), nullptr, dinv, nn, b, omega, x, s);
    else
        mdiag<float>(mode, K, static_cast<int>(nn), nullptr, dinv, nn, b, omega, x, s);
}

void launch_mdiag_solve(int mode, int kind, int K, int nrows, const int *rowid, const void *dinv, int64_t n,
                        const void *b, void *x, hipStream_t s) {
    if (kind == MK_F64)
        mdiag<double>(mode, K, nrows, rowid, dinv, n, b, 1.0, x, s);
    else
        mdiag<float>(mode, K, nrows, rowid, dinv, n, b, 1.0, x, s);
}

// ---------------------------------------------------------------- dense coarse end
// Y = M X with NC columns (M's rows ld values apart), FP64: one wavefront per
// row of M, lane j walks columns j, j + 64, ... and keeps NC partial sums
template <int NC>
__global__ void __launch_bounds__(TB) k_mdense(const double *M, int m, int ld, const double *X, double *Y) {
    using T = double;
    const int row = blockIdx.x * (TB / 64) + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (row >= m) return;
    T acc[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) acc[c] = T(0);
    const int64_t base = static_cast<int64_t>(row) * ld;
    for (int j = lane; j < m; j += 64) {
        const T v = M[base + j];
#pragma unroll
        for (int c = 0; c < NC; ++c) acc[c] += v * X[static_cast<int64_t>(j) * NC + c];
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) acc[c] = gsum<64>(acc[c]);
#pragma unroll
    for (int c = 0; c < NC; ++c)
        if (lane == c) Y[static_cast<int64_t>(row) * NC + c] = acc[c];
}

// The same with an FP32 or BF16 M (16-byte aligned, ld a multiple of 8, zeros
// past m) and FP32 matrix instructions: a workgroup takes 16 rows and all
// columns, its 16 wavefronts chunks of 32 of the sum. With a wavefront per row
// every row reads all of X again (273 KB at m = 2846, 24 columns: 37 us for 16
// MB of M); here 16 rows share it. A lane's 8 values of M are neighbours in
// its row, so the k-th instruction of a chunk sums the columns 8 g + k of its
// four lane groups g. Each output is a sum of 64 partial sums, as with a
// wavefront per row (relative error against 64 bits, m = 100 to 6880, 2 to 24
// columns: 0.7e-7 to 2.0e-7 either way). Bound by the reads of X and of M from
// the L2: m = 2846, BF16, 24 columns 37 -> 17 us; 5217: 127 -> 50 us, 6
// columns 39 -> 28; 6880, 8 columns 76 -> 36.
constexpr int DW = 16;  // wavefronts
template <int MK, int NC>
__global__ void __launch_bounds__(64 * DW) k_mdense_mfma(const void *M, int m, int ld, const float *X, float *Y) {
    typedef float float4_t __attribute__((ext_vector_type(4)));
    typedef uint32_t uint4_t __attribute__((ext_vector_type(4)));
    constexpr int CT = (NC + 15) / 16;
    __shared__ float part[DW][CT][256];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
    const int row0 = blockIdx.x * 16, row = row0 + r < m ? row0 + r : m - 1;
    const int64_t base = static_cast<int64_t>(row) * ld;
    float4_t acc[CT][4];
#pragma unroll
    for (int t = 0; t < CT; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[t][q] = float4_t{0.f, 0.f, 0.f, 0.f};
    for (int k0 = 32 * w; k0 < m; k0 += 32 * DW) {
        const int k = k0 + 8 * g;
        float a[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) a[u] = 0.f;
        if (k < ld) {
            if constexpr (MK == MK_BF16) {
                const uint4_t v = *reinterpret_cast<const uint4_t *>(static_cast<const uint16_t *>(M) + base + k);
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    a[2 * u] = __uint_as_float(v[u] << 16);
                    a[2 * u + 1] = __uint_as_float(v[u] & 0xffff0000u);
                }
            } else {
                const float4_t *v = reinterpret_cast<const float4_t *>(static_cast<const float *>(M) + base + k);
                const float4_t lo = v[0], hi = v[1];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    a[u] = lo[u];
                    a[4 + u] = hi[u];
                }
            }
        }
        float b[CT][8];
#pragma unroll
        for (int t = 0; t < CT; ++t)
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int c = 16 * t + r;
                b[t][u] = k + u < m && c < NC ? X[static_cast<int64_t>(k + u) * NC + c] : 0.f;
            }
#pragma unroll
        for (int u = 0; u < 8; ++u)
#pragma unroll
            for (int t = 0; t < CT; ++t)
                acc[t][u % 4] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u], b[t][u], acc[t][u % 4], 0, 0, 0);
    }
#pragma unroll
    for (int t = 0; t < CT; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i)
            part[w][t][16 * (4 * g + i) + r] = (acc[t][0][i] + acc[t][1][i]) + (acc[t][2][i] + acc[t][3][i]);
    __syncthreads();
    for (int o = threadIdx.x; o < CT * 256; o += 64 * DW) {
        const int t = o >> 8, e = o & 255, i = row0 + (e >> 4), c = 16 * t + (e & 15);
        if (i >= m || c >= NC) continue;
        float v[DW];
#pragma unroll
        for (int u = 0; u < DW; ++u) v[u] = part[u][t][e];
#pragma unroll
        for (int h = DW / 2; h > 0; h /= 2)
#pragma unroll
            for (int u = 0; u < h; ++u) v[u] += v[u + h];
        Y[static_cast<int64_t>(i) * NC + c] = v[0];
    }
}

template <int MK>
static void mdense_mfma(const void *M, int m, int ld, int nc, const float *X, float *Y, hipStream_t s) {
    const int nb = ceil_div(m, 16);
    switch (nc) {
        case 2: k_mdense_mfma<MK, 2><<<nb, 64 * DW, 0, s>>>(M, m, ld, X, Y); break;
        case 4: k_mdense_mfma<MK, 4><<<nb, 64 * DW, 0, s>>>(M, m, ld, X, Y); break;
        case 6: k_mdense_mfma<MK, 6><<<nb, 64 * DW, 0, s>>>(M, m, ld, X, Y); break;
        case 8: k_mdense_mfma<MK, 8><<<nb, 64 * DW, 0, s>>>(M, m, ld, X, Y); break;
        case 12: k_mdense_mfma<MK, 12><<<nb, 64 * DW, 0, s>>>(M, m, ld, X, Y); break;
        case 24: k_mdense_mfma<MK, 24><<<nb, 64 * DW, 0, s>>>(M, m, ld, X, Y); break;
        default: throw Error(AMG_EINVAL, "multi dense kernel: unsupported column count");
    }
}

static void mdense_f64(const double *M, int m, int ld, int nc, const double *X, double *Y, hipStream_t s) {
    const int nb = ceil_div(m, TB / 64);
    switch (nc) {
        case 2: k_mdense<2><<<nb, TB, 0, s>>>(M, m, ld, X, Y); break;
        case 4: k_mdense<4><<<nb, TB, 0, s>>>(M, m, ld, X, Y); break;
        case 6: k_mdense<6><<<nb, TB, 0, s>>>(M, m, ld, X, Y); break;
        case 8: k_mdense<8><<<nb, TB, 0, s>>>(M, m, ld, X, Y); break;
        case 12: k_mdense<12><<<nb, TB, 0, s>>>(M, m, ld, X, Y); break;
        case 24: k_mdense<24><<<nb, TB, 0, s>>>(M, m, ld, X, Y); break;
        default: throw Error(AMG_EINVAL, "multi dense kernel: unsupported column count");
    }
}

void launch_mdense(int mkind, const void *M, int m, int ld, int nc, const void *X, void *Y, hipStream_t s) {
    if (m <= 0) return;
    AMG_REQUIRE(ld >= m && (mkind == MK_F64 || ld % 8 == 0), AMG_EINVAL, "multi dense kernel: row stride");
    switch (mkind) {
        case MK_F64: mdense_f64(static_cast<const double *>(M), m, ld, nc, static_cast<const double *>(X), static_cast<double *>(Y), s); break;
        case MK_F32: mdense_mfma<MK_F32>(M, m, ld, nc, static_cast<const float *>(X), static_cast<float *>(Y), s); break;
        default: mdense_mfma<MK_BF16>(M, m, ld, nc, static_cast<const float *>(X), static_cast<float *>(Y), s); break;
    }
    AMG_CHECK_LAUNCH();
}

// ---------------------------------------------------------------- Krylov vectors
constexpr int MDOT_MAX_BLOCKS = 1024;

int mdot_blocks(int64_t nd) {
    const int64_t nb = (nd + TB - 1) / TB;
    return static_cast<int>(nb < MDOT_MAX_BLOCKS ? (nb > 0 ? nb : 1) : MDOT_MAX_BLOCKS);
}

// partial[o] = the workgroup's sum of acc[o], a fixed-order tree
template <int N>
__device__ __forceinline__ void mpartials(const double *acc, double *partial) {
    __shared__ double red[N][TB / 64];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
#pragma unroll
    for (int o = 0; o < N; ++o) {
        const double v = gsum<64>(acc[o]);
        if (lane == 0) red[o][w] = v;
    }
    __syncthreads();
    if (threadIdx.x < N) {
        double v = 0.0;
#pragma unroll
        for (int u = 0; u < TB / 64; ++u) v += red[threadIdx.x][u];
        partial[static_cast<int64_t>(blockIdx.x) * N + threadIdx.x] = v;
    }
}

// per block: sums over the dofs d = t, t + stride, ... (a fixed assignment,
// the same in every kernel below that sums), then a fixed-order tree over the
// block; partial[blk * K + r]
template <int K, typename T>
__global__ void __launch_bounds__(TB) k_mdot(const T *a, const double *b, int64_t nd, double *partial) {
    double acc[K];
#pragma unroll
    for (int r = 0; r < K; ++r) acc[r] = 0.0;
    const int64_t stride = static_cast<int64_t>(gridDim.x) * TB;
    for (int64_t d = static_cast<int64_t>(blockIdx.x) * TB + threadIdx.x; d < nd; d += stride)
#pragma unroll
        for (int r = 0; r < K; ++r) acc[r] += static_cast<double>(a[d * K + r]) * b[d * K + r];
    mpartials<K>(acc, partial);
}

// out[o] = sum of partial[blk][o] over the nb blocks: one workgroup per
// output; thread u sums blocks u, u + TB, ... in order, then a fixed-order
// tree over the workgroup. (out is host memory: no copy after it.)
__global__ void __launch_bounds__(TB) k_mdot_reduce(const double *partial, int nb, int no, double *out) {
    __shared__ double red[TB / 64];
    const int o = blockIdx.x;
    double v = 0.0;
    for (int b = threadIdx.x; b < nb; b += TB) v += partial[static_cast<int64_t>(b) * no + o];
    v = gsum<64>(v);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        double w = 0.0;
#pragma unroll
        for (int u = 0; u < TB / 64; ++u) w += red[u];
        out[o] = w;
    }
}

static void mreduce(int nb, int no, const double *partial, double *out, hipStream_t s) {
    AMG_CHECK_LAUNCH();
    k_mdot_reduce<<<no, TB, 0, s>>>(partial, nb, no, out);
    AMG_CHECK_LAUNCH();
}

template <typename T>
void launch_mdot(int K, int64_t nd, const T *a, const double *b, double *partial, double *out, hipStream_t s) {
    const int nb = mdot_blocks(nd);
    switch (K) {
        case 2: k_mdot<2><<<nb, TB, 0, s>>>(a, b, nd, partial); break;
        case 4: k_mdot<4><<<nb, TB, 0, s>>>(a, b, nd, partial); break;
        case 8: k_mdot<8><<<nb, TB, 0, s>>>(a, b, nd, partial); break;
        default: throw Error(AMG_EINVAL, "multi dot: K must be 2, 4 or 8");
    }
    mreduce(nb, K, partial, out, s);
}
template void launch_mdot<double>(int, int64_t, const double *, const double *, double *, double *, hipStream_t);
template void launch_mdot<float>(int, int64_t, const float *, const double *, double *, double *, hipStream_t);

// The iteration's vector work is bound by memory (52 MB a vector of the 32^3
// Laplacian with 8 right-hand sides), so each vector is read once per
// synchronisation: both updates, <r, r> and the cycle's FP32 copy of r in one
// pass, the next direction with its <p, r>; z stays in the cycle's FP32.
// Thread t takes two neighbouring values (of columns c, c + 1), 16-byte loads
// and stores side by side over the lanes (a dof's K values per thread, 64 bytes
// apart, is stored at two thirds of the rate: 88 and 54 us). 52 and 31 us,
// before them five passes and two conversions, 137 us.
typedef double double2_t __attribute__((ext_vector_type(2)));
typedef float float2_t __attribute__((ext_vector_type(2)));

// partial[c] = the workgroup's sum over the threads of column c
template <int K>
__device__ __forceinline__ void mcolumns(double2_t acc, double *partial) {
    __shared__ double red[K][TB / 64];
    constexpr int H = K / 2;
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    double a0 = acc.x, a1 = acc.y;
#pragma unroll
    for (int o = 32; o >= H; o >>= 1) {
        a0 += __shfl_xor(a0, o, 64);
        a1 += __shfl_xor(a1, o, 64);
    }
    if (lane < H) {
        red[2 * lane][w] = a0;
        red[2 * lane + 1][w] = a1;
    }
    __syncthreads();
    if (threadIdx.x < K) {
        double v = 0.0;
#pragma unroll
        for (int u = 0; u < TB / 64; ++u) v += red[threadIdx.x][u];
        partial[static_cast<int64_t>(blockIdx.x) * K + threadIdx.x] = v;
    }
}

template <int K>
__global__ void __launch_bounds__(TB) k_mupdate(int64_t n, const MCoef alpha, const double2_t *p, const double2_t *q,
                                                double2_t *x, double2_t *r, float2_t *r32, double *partial) {
    constexpr int H = K / 2;
    const int64_t t = static_cast<int64_t>(blockIdx.x) * TB + threadIdx.x, stride = static_cast<int64_t>(gridDim.x) * TB;
    const int c = 2 * static_cast<int>(t % H);  // (H divides the stride)
    const double2_t al = {alpha.c[c], alpha.c[c + 1]};
    double2_t acc = {0.0, 0.0};
#pragma unroll 2
    for (int64_t e = t; e < n; e += stride) {
        x[e] = x[e] + al * p[e];
        const double2_t rv = r[e] - al * q[e];
        r[e] = rv;
        if (r32) r32[e] = float2_t{static_cast<float>(rv.x), static_cast<float>(rv.y)};
        acc += rv * rv;
    }
    mcolumns<K>(acc, partial);
}

static const double2_t *pv(const double *v) { return reinterpret_cast<const double2_t *>(v); }
static double2_t *pv(double *v) { return reinterpret_cast<double2_t *>(v); }
static const float2_t *pv(const float *v) { return reinterpret_cast<const float2_t *>(v); }
static float2_t *pv(float *v) { return reinterpret_cast<float2_t *>(v); }

void launch_mupdate(int K, int64_t nd, const MCoef &alpha, const double *p, const double *q, double *x, double *r,
                    float *r32, double *partial, double *rr, hipStream_t s) {
    const int nb = mdot_blocks(nd);
    const int64_t n = nd * K / 2;
    switch (K) {
        case 2: k_mupdate<2><<<nb, TB, 0, s>>>(n, alpha, pv(p), pv(q), pv(x), pv(r), pv(r32), partial); break;
        case 4: k_mupdate<4><<<nb, TB, 0, s>>>(n, alpha, pv(p), pv(q), pv(x), pv(r), pv(r32), partial); break;
        case 8: k_mupdate<8><<<nb, TB, 0, s>>>(n, alpha, pv(p), pv(q), pv(x), pv(r), pv(r32), partial); break;
        default: throw Error(AMG_EINVAL, "multi update: K must be 2, 4 or 8");
    }
    mreduce(nb, K, partial, rr, s);
}

// p = z + beta p (first: p = z) and, with r, the partials of <p, r>
template <int K, typename Z>
__global__ void __launch_bounds__(TB) k_mdirection(int64_t n, const MCoef beta, int first, const Z *z, double2_t *p,
                                                   const double2_t *r, double *partial) {
    constexpr int H = K / 2;
    const int64_t t = static_cast<int64_t>(blockIdx.x) * TB + threadIdx.x, stride = static_cast<int64_t>(gridDim.x) * TB;
    const int c = 2 * static_cast<int>(t % H);
    const double2_t be = {beta.c[c], beta.c[c + 1]};
    double2_t acc = {0.0, 0.0};
#pragma unroll 2
    for (int64_t e = t; e < n; e += stride) {
        const Z zv = z[e];
        double2_t pn = {static_cast<double>(zv.x), static_cast<double>(zv.y)};
        if (!first) pn += be * p[e];
        p[e] = pn;
        if (r) acc += pn * r[e];
    }
    if (r) mcolumns<K>(acc, partial);
}

template <typename T>
void launch_mdirection(int K, int64_t nd, const MCoef &beta, bool first, const T *z, double *p, const double *r,
                       double *partial, double *pr, hipStream_t s) {
    const int nb = mdot_blocks(nd), f = first ? 1 : 0;
    const int64_t n = nd * K / 2;
    switch (K) {
        case 2: k_mdirection<2><<<nb, TB, 0, s>>>(n, beta, f, pv(z), pv(p), pv(r), partial); break;
        case 4: k_mdirection<4><<<nb, TB, 0, s>>>(n, beta, f, pv(z), pv(p), pv(r), partial); break;
        case 8: k_mdirection<8><<<nb, TB, 0, s>>>(n, beta, f, pv(z), pv(p), pv(r), partial); break;
        default: throw Error(AMG_EINVAL, "multi direction: K must be 2, 4 or 8");
    }
    AMG_CHECK_LAUNCH();
    if (r) mreduce(nb, K, partial, pr, s);
}
template void launch_mdirection<double>(int, int64_t, const MCoef &, bool, const double *, double *, const double *,
                                        double *, double *, hipStream_t);
template void launch_mdirection<float>(int, int64_t, const MCoef &, bool, const float *, double *, const double *,
                                       double *, double *, hipStream_t);

// r = b - r
__global__ void k_msubtract(int64_t n, const double *b, double *r) {
    for (int64_t e = static_cast<int64_t>(blockIdx.x) * TB + threadIdx.x; e < n;
         e += static_cast<int64_t>(gridDim.x) * TB)
        r[e] = b[e] - r[e];
}

static int grid_e(int64_t n) {
    int64_t nb = (n + TB - 1) / TB;
    return static_cast<int>(nb > 8192 ? 8192 : (nb > 0 ? nb : 1));
}

void launch_msubtract(int64_t n, const double *b, double *r, hipStream_t s) {
    if (n <= 0) return;
    k_msubtract<<<grid_e(n), TB, 0, s>>>(n, b, r);
    AMG_CHECK_LAUNCH();
}

// the caller's nvec vectors <-> the interleaved block of K >= nvec (the
// block's other columns are zero going in, dropped coming out)
__global__ void k_interleave(int K, int nvec, int64_t nd, const double *src, double *dst, int to) {
    for (int64_t e = static_cast<int64_t>(blockIdx.x) * TB + threadIdx.x; e < nd * K;
         e += static_cast<int64_t>(gridDim.x) * TB) {
        const int64_t d = e / K;
        const int r = static_cast<int>(e - d * K);
        if (to)
            dst[e] = r < nvec ? src[static_cast<int64_t>(r) * nd + d] : 0.0;
        else if (r < nvec)
            dst[static_cast<int64_t>(r) * nd + d] = src[e];
    }
}

void launch_interleave(int K, int nvec, int64_t nd, const double *src, double *dst, bool to_interleaved,
                       hipStream_t s) {
    if (nd <= 0) return;
    k_interleave<<<grid_e(nd * K), TB, 0, s>>>(K, nvec, nd, src, dst, to_interleaved ? 1 : 0);
    AMG_CHECK_LAUNCH();
}

}  // namespace amgp2
