// A Gauss-Seidel sweep over all colours of a level in one launch.
//
// One launch per colour pays a launch and a chain of dependent loads (row
// pointer, column, x, values) per colour, 4 to 10 us for well under 1 us of
// bandwidth. Here the workgroups stay on the chip for the whole sweep, take
// tiles of rows from a ticket counter in colour order, and every row waits
// for its own neighbours only. Before it waits it has loaded everything that
// does not depend on them: row pointers, right-hand side, diagonal, the
// products with entries whose x the sweep has yet to change, and the columns
// and values of the others. Then there is one gather that is repeated until
// the neighbours are there, one reduction and one store: a colour costs about
// two trips to memory.
//
// Swept values go to `xg`, by colour, 4 to a node: 16-byte loads and stores
// at device scope (sc1), which the 8 XCDs see alike. An agent-scope fence
// instead would write back and invalidate an XCD's L2 (tens of us). A value
// that is not there yet holds a NaN of a fixed payload; no computed value
// has that payload (it is replaced by another NaN). There are two buffers: a
// sweep uses the one that the control words name, fills the other with the
// payload for the next sweep, and the last workgroup out turns them over.
//
// Progress: a row depends only on rows of smaller tickets (setup makes sure
// that no two rows of a colour are coupled), and a ticket is taken by a running
// workgroup, so the smallest unfinished ticket never
// waits, whatever part of the grid is resident. The wait is bounded all the
// same; past the bound the row becomes NaN, which the Krylov loops report as
// divergence.
//
// What bounds it: a colour's two trips to memory (about 2.3 us) where a colour
// is smaller than the chip, the tiles' loads where it is larger. us per sweep
// (mean of one from zero and one from an iterate), one launch per colour ->
// this kernel, elasticity:
//   16^3 level 0 (35,937 rows, 14 colours)  FP64  92 -> 48   FP32  81 -> 43
//   16^3 level 1 ( 5,217 rows, 29 colours)  FP64 178 -> 58   BF16 173 -> 54
//   32^3 level 0 (274,625 rows)             FP64 217 -> 236  FP32 147 -> 149
//   32^3 level 1 ( 39,233 rows)             FP64 200 -> 101  BF16 156 -> 70
// (with `part`, which saves half of the residual's pass after the sweep; from
// some 32^3 on, by precision, a launch per colour is faster: sweep_by_colour).
#include "common.h"
#include "sweep.h"

namespace amgp2 {

namespace {

constexpr unsigned SPIN_MAX = 1u << 21;  // a second or two of polls

template <int KIND>
struct ValueType { using V = float; };
template <>
struct ValueType<SWEEP_F64> { using V = double; };

template <typename T>
__device__ __forceinline__ T agent_load(const T *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ void agent_store(T *p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <int G, typename V>
__device__ __forceinline__ V lanes_sum(V v) {
#pragma unroll
    for (int o = G / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, G);
    return v;
}

template <int KIND, typename V>
__device__ __forceinline__ V entry(const void *val, int64_t k) {
    if constexpr (KIND == SWEEP_F64)
        return static_cast<const double *>(val)[k];
    else if constexpr (KIND == SWEEP_F32)
        return static_cast<const float *>(val)[k];
    else
        return __uint_as_float(static_cast<uint32_t>(static_cast<const uint16_t *>(val)[k]) << 16);
}

// payloads of "not there yet" (quiet NaNs)
constexpr uint32_t ABSENT32 = 0x7fdead01u;
constexpr uint64_t ABSENT64 = 0x7ffdead0beef0001ull;
__device__ __forceinline__ bool absent(float v) { return __float_as_uint(v) == ABSENT32; }
__device__ __forceinline__ bool absent(double v) {
    return static_cast<uint64_t>(__double_as_longlong(v)) == ABSENT64;
}
__device__ __forceinline__ float absent_value(float) { return __uint_as_float(ABSENT32); }
__device__ __forceinline__ double absent_value(double) { return __longlong_as_double(static_cast<long long>(ABSENT64)); }

// device-scope 16-byte loads of a swept node's components (4 to a node; the
// buffer's descriptor covers one half of xg)
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
constexpr int AUX_SC1 = 16;  // the scope bit of device-scope accesses
template <int NV, int AUX = AUX_SC1>
__device__ __forceinline__ void gather(__amdgpu_buffer_rsrc_t xg, int j, float *v) {
    if constexpr (NV == 1) {
        v[0] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(xg, 4 * j, 0, AUX));
    } else {
        const u32x4 q = __builtin_amdgcn_raw_buffer_load_b128(xg, 16 * j, 0, AUX);
        v[0] = __uint_as_float(q.x);
        v[1] = __uint_as_float(q.y);
        v[2] = __uint_as_float(q.z);
    }
}
__device__ __forceinline__ double from_words(uint32_t lo, uint32_t hi) {
    return __longlong_as_double(static_cast<long long>(static_cast<uint64_t>(hi) << 32 | lo));
}
template <int NV, int AUX = AUX_SC1>
__device__ __forceinline__ void gather(__amdgpu_buffer_rsrc_t xg, int j, double *v) {
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    if constexpr (NV == 1) {
        const u32x2 q = __builtin_amdgcn_raw_buffer_load_b64(xg, 8 * j, 0, AUX);
        v[0] = from_words(q.x, q.y);
    } else {
        const u32x4 q = __builtin_amdgcn_raw_buffer_load_b128(xg, 32 * j, 0, AUX);
        const u32x2 w = __builtin_amdgcn_raw_buffer_load_b64(xg, 32 * j + 16, 0, AUX);
        v[0] = from_words(q.x, q.y);
        v[1] = from_words(q.z, q.w);
        v[2] = from_words(w.x, w.y);
    }
}

template <int MODE, typename V>
__device__ __forceinline__ void accumulate(const V *e, const V *x, V *s) {
    if constexpr (MODE == SWEEP_BLOCK) {
        s[0] += e[0] * x[0] + e[1] * x[1] + e[2] * x[2];
        s[1] += e[3] * x[0] + e[4] * x[1] + e[5] * x[2];
        s[2] += e[6] * x[0] + e[7] * x[1] + e[8] * x[2];
    } else if constexpr (MODE == SWEEP_SCALAR3) {
        s[0] += e[0] * x[0];
        s[1] += e[0] * x[1];
        s[2] += e[0] * x[2];
    } else {
        s[0] += e[0] * x[0];
    }
}

}  // namespace

template <int MODE, int KIND, int G, int NT>
__global__ void __launch_bounds__(NT, 4) k_sweep(const SweepArgs a) {
    using V = typename ValueType<KIND>::V;
    constexpr int NV = MODE == SWEEP_SCALAR1 ? 1 : 3;   // components
    constexpr int NP = MODE == SWEEP_BLOCK ? 9 : 1;     // planes
    constexpr int XS = MODE == SWEEP_SCALAR1 ? 1 : 4;   // stride of xg
    constexpr int GROUPS = NT / G;
    // entries per lane loaded before the wait (FP64 blocks: one more would spill)
    constexpr int U = MODE == SWEEP_BLOCK && KIND == SWEEP_F64 ? 1 : 2;
    __shared__ int sh_ticket[2];
    __shared__ int sh_tpre[SWEEP_MAX_COLOURS + 1], sh_cptr[SWEEP_MAX_COLOURS + 1], sh_base[SWEEP_MAX_COLOURS + 1];
    const int tid = threadIdx.x, lane = tid % G, grp = tid / G;
    const int c3 = lane < NV ? lane : 0;
    int *const ticket = a.ctl, *const exits = a.ctl + 32, *const turn = a.ctl + 64, *const gave_up = a.ctl + 96;
    const V *const b = static_cast<const V *>(a.b);
    const V *const xo = static_cast<const V *>(a.x_old);
    V *const x = static_cast<V *>(a.x);
    const V *const dinv = static_cast<const V *>(a.dinv);
    int next = 0;
    if (tid == 0) {
        next = atomicAdd(ticket, 1);
        sh_ticket[0] = next;
        next = atomicAdd(ticket, 1);
    }
    const unsigned sweep = static_cast<unsigned>(*turn) + 1u;  // this sweep's number, from 1 on
    const int which = (sweep & 1u) == 0u;
    V *const xg = static_cast<V *>(a.xg) + (which ? a.xg_half : 0);
    V *const xfill = static_cast<V *>(a.xg) + (which ? 0 : a.xg_half);
    const __amdgpu_buffer_rsrc_t xgr =
        __builtin_amdgcn_make_buffer_rsrc(xg, 0, static_cast<int>(a.xg_half * sizeof(V)), 0x00027000);
    for (int k = tid; k <= a.ncolors; k += NT) {
        sh_tpre[k] = a.tpre[k];
        sh_cptr[k] = a.cptr[k];
        sh_base[k] = a.base[k];
    }
    __syncthreads();
    bool bad = false;
    // tile t: colour ct, this group's grouped row (-1: none)
    int ct = a.forward ? 0 : a.ncolors - 1, t = sh_ticket[0];
    auto row_of = [&](int tile) {
        if (tile >= a.ntiles) return -1;
        const int u = a.forward ? tile : a.ntiles - 1 - tile;
        if (a.forward)
            while (sh_tpre[ct + 1] <= u) ++ct;
        else
            while (sh_tpre[ct] > u) --ct;
        const int g = sh_cptr[ct] + (u - sh_tpre[ct]) * GROUPS + grp;
        return g < sh_cptr[ct + 1] ? g : -1;
    };
    int g = row_of(t), place = g < 0 ? 0 : sh_base[ct] + g - sh_cptr[ct], phase = 1;
    int4 rd = g < 0 ? make_int4(0, 0, 0, 0) : a.rows[g];
    while (t < a.ntiles) {
        if (tid == 0) sh_ticket[phase] = next;
        __syncthreads();
        const int t_next = sh_ticket[phase];
        phase ^= 1;
        if (tid == 0 && t_next < a.ntiles) next = atomicAdd(ticket, 1);
        // this row, and the next one's descriptor on its way
        const bool on = g >= 0;
        const int i = rd.w, kd = rd.y, k0 = rd.x, k1 = rd.z, here = place;
        g = row_of(t_next);
        place = g < 0 ? 0 : sh_base[ct] + g - sh_cptr[ct];
        rd = g < 0 ? make_int4(0, 0, 0, 0) : a.rows[g];
        t = t_next;
        const bool ep = on && lane < NV;
        // entries whose x this sweep changes before this row
        const int beg = a.forward ? k0 : kd + 1, end = a.forward ? kd : k1;
        int jn[U];
        V e[U][NP];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = beg + lane + u * G;
            jn[u] = k < end ? a.gcol[k] : -1;
            if (k < end) {
#pragma unroll
                for (int p = 0; p < NP; ++p) e[u][p] = entry<KIND, V>(a.val, p * a.nnz + k);
            }
        }
        V bc = V(0), own = V(0), d[NV], q[NV], base[NV];
#pragma unroll
        for (int p = 0; p < NV; ++p) {
            d[p] = base[p] = V(0);
            q[p] = V(1);
        }
        if (ep) {
            bc = b[NV * static_cast<int64_t>(i) + c3];
            if (!a.x_zero) own = xo[NV * static_cast<int64_t>(i) + c3];
            if constexpr (MODE == SWEEP_BLOCK) {
#pragma unroll
                for (int p = 0; p < NV; ++p) d[p] = dinv[(3 * c3 + p) * a.dinv_n + i];
            } else {
                d[0] = dinv[i];
            }
            if constexpr (KIND == SWEEP_BF16) {
#pragma unroll
                for (int p = 0; p < NV; ++p)
                    q[p] = MODE == SWEEP_BLOCK ? a.rscale[3 * static_cast<int64_t>(i) + p] : a.rscale[i];
            }
            xfill[static_cast<int64_t>(XS) * here + c3] = absent_value(V(0));
        }
        if (!a.x_zero) {
            // the other entries: the sweep's later side and the diagonal
            const int o0 = a.forward ? kd : k0, o1 = a.forward ? k1 : (on ? kd + 1 : 0);
            for (int ko = o0 + lane; ko < o1; ko += G) {
                const int64_t j = a.col[ko];
                V xv[NV], eo[NP];
#pragma unroll
                for (int p = 0; p < NV; ++p) xv[p] = xo[NV * j + p];
#pragma unroll
                for (int p = 0; p < NP; ++p) eo[p] = entry<KIND, V>(a.val, p * a.nnz + ko);
                accumulate<MODE>(eo, xv, base);
            }
#pragma unroll
            for (int p = 0; p < NV; ++p) base[p] = lanes_sum<G>(base[p]) * q[p];
        }

        V s[NV];
#pragma unroll
        for (int p = 0; p < NV; ++p) s[p] = V(0);
        for (int k = beg + lane; __any(k < end); k += U * G) {
            if (k != beg + lane) {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int ku = k + u * G;
                    jn[u] = ku < end ? a.gcol[ku] : -1;
                    if (ku < end) {
#pragma unroll
                        for (int p = 0; p < NP; ++p) e[u][p] = entry<KIND, V>(a.val, p * a.nnz + ku);
                    }
                }
            }
            // Most neighbours were swept a while ago: an ordinary load finds
            // them, in the L2 for its XCD's other rows (device-scope loads
            // pass by it: 21^3 level 0 FP64 87 -> 81 us, 32^3 level 1 BF16
            // 73 -> 70). Never an earlier sweep's: the launch before this one
            // filled the buffer with "absent". The others are waited for at
            // device scope.
            V xv[U][NV];
            bool got[U];
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (jn[u] >= 0) gather<NV, 0>(xgr, jn[u], xv[u]);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                got[u] = true;
                if (jn[u] >= 0) {
#pragma unroll
                    for (int p = 0; p < NV; ++p) got[u] = got[u] && !absent(xv[u][p]);
                }
            }
            unsigned n = 0;
            for (;;) {
                bool there = true;
#pragma unroll
                for (int u = 0; u < U; ++u) there = there && got[u];
                if (!there) {
                    asm volatile("" ::: "memory");  // a new load every time
#pragma unroll
                    for (int u = 0; u < U; ++u)
                        if (!got[u]) gather<NV>(xgr, jn[u], xv[u]);
                    there = true;
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        if (!got[u]) {
                            got[u] = true;
#pragma unroll
                            for (int p = 0; p < NV; ++p) got[u] = got[u] && !absent(xv[u][p]);
                        }
                        there = there && got[u];
                    }
                }
                if (__all(there)) break;
                if (bad) break;
                if ((++n & 0xfff) == 0) {
                    // a row that gives up tells the others
                    if (n > SPIN_MAX) agent_store(gave_up, static_cast<int>(sweep));
                    bad = agent_load(gave_up) == static_cast<int>(sweep);
                }
                if (n > 2) __builtin_amdgcn_s_sleep(1);
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (jn[u] >= 0) accumulate<MODE>(e[u], xv[u], s);
        }
        V res[NV];
#pragma unroll
        for (int p = 0; p < NV; ++p) {
            s[p] = lanes_sum<G>(s[p]) * q[p];
            res[p] = (NV == 1 ? bc : __shfl(bc, p, G)) - s[p] - base[p];
        }
        V dx = d[0] * (NV == 1 || c3 == 0 ? res[0] : (c3 == 1 ? res[NV / 2] : res[NV - 1]));
        if constexpr (MODE == SWEEP_BLOCK) dx = d[0] * res[0] + d[1] * res[1] + d[2] * res[2];
        V xn = own + dx;
        if (bad || absent(xn)) xn = V(__builtin_nan(""));
        if (ep) {
            agent_store(xg + static_cast<int64_t>(XS) * here + c3, xn);
            x[NV * static_cast<int64_t>(i) + c3] = xn;
        }
        if (a.part) {
            // (the diagonal entry is loaded only now: off the rows' chain)
            V ax = V(0);
            if constexpr (MODE == SWEEP_BLOCK) {
                const V x0 = __shfl(xn, 0, G), x1 = __shfl(xn, 1, G), x2 = __shfl(xn, 2, G);
                if (ep)
                    ax = entry<KIND, V>(a.val, 3 * c3 * a.nnz + kd) * x0 +
                         entry<KIND, V>(a.val, (3 * c3 + 1) * a.nnz + kd) * x1 +
                         entry<KIND, V>(a.val, (3 * c3 + 2) * a.nnz + kd) * x2;
            } else if (ep) {
                ax = entry<KIND, V>(a.val, kd) * xn;
            }
            if (ep) {
                const V sc = NV == 1 || c3 == 0 ? s[0] : (c3 == 1 ? s[NV / 2] : s[NV - 1]);
                const V qc = NV == 1 || c3 == 0 ? q[0] : (c3 == 1 ? q[NV / 2] : q[NV - 1]);
                static_cast<V *>(a.part)[NV * static_cast<int64_t>(i) + c3] = bc - sc - ax * qc;
            }
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

// r_i -= the entries of later colours times x: the residual after a forward
// sweep that left b - (the other entries) x in r. Half of the operator's
// bytes; one group of G lanes per row, two entries per lane in flight.
template <int MODE, int KIND, int G>
__global__ void __launch_bounds__(256) k_later(const SweepArgs a, int nrows) {
    using V = typename ValueType<KIND>::V;
    constexpr int NV = MODE == SWEEP_SCALAR1 ? 1 : 3;
    constexpr int NP = MODE == SWEEP_BLOCK ? 9 : 1;
    const int64_t t = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    const int g = static_cast<int>(t / G), lane = static_cast<int>(t % G);
    const bool on = g < nrows;
    const int4 rd = on ? a.rows[g] : make_int4(0, 0, 0, 0);
    const bool ep = on && lane < NV;
    const V *const x = static_cast<const V *>(a.x);
    V *const r = static_cast<V *>(a.part) + NV * static_cast<int64_t>(rd.w) + (ep ? lane : 0);
    const V old = ep ? *r : V(0);
    V q = V(1);
    if constexpr (KIND == SWEEP_BF16)
        if (ep) q = MODE == SWEEP_BLOCK ? a.rscale[3 * static_cast<int64_t>(rd.w) + lane] : a.rscale[rd.w];
    V s[NV];
#pragma unroll
    for (int p = 0; p < NV; ++p) s[p] = V(0);
    for (int k = rd.y + 1 + lane; k < rd.z; k += 2 * G) {
        const bool two = k + G < rd.z;
        const int64_t j0 = a.col[k], j1 = two ? a.col[k + G] : j0;
        V x0[NV], x1[NV], e0[NP], e1[NP];
#pragma unroll
        for (int p = 0; p < NV; ++p) {
            x0[p] = x[NV * j0 + p];
            x1[p] = two ? x[NV * j1 + p] : V(0);
        }
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            e0[p] = entry<KIND, V>(a.val, p * a.nnz + k);
            e1[p] = two ? entry<KIND, V>(a.val, p * a.nnz + k + G) : V(0);
        }
        accumulate<MODE>(e0, x0, s);
        if (two) accumulate<MODE>(e1, x1, s);
    }
#pragma unroll
    for (int p = 0; p < NV; ++p) s[p] = lanes_sum<G>(s[p]);
    if (ep) *r = old - q * (NV == 1 || lane == 0 ? s[0] : (lane == 1 ? s[NV / 2] : s[NV - 1]));
}

template <typename V>
__global__ void __launch_bounds__(256) k_absent(V *xg, int64_t n) {
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; i < n;
         i += static_cast<int64_t>(gridDim.x) * 256)
        xg[i] = absent_value(V(0));
}

void launch_sweep_absent(int kind, void *xg, int64_t n, hipStream_t s) {
    if (n <= 0) return;
    const int nb = static_cast<int>(n / 256 + 1 < 4096 ? n / 256 + 1 : 4096);
    if (kind == SWEEP_F64)
        k_absent<double><<<nb, 256, 0, s>>>(static_cast<double *>(xg), n);
    else
        k_absent<float><<<nb, 256, 0, s>>>(static_cast<float *>(xg), n);
    AMG_CHECK_LAUNCH();
}

// One wavefront per row: three passes over it, each placing its class of
// entries (earlier colours, the diagonal, later colours) by the ballot's
// prefix count, in their order.
__global__ void __launch_bounds__(256) k_split_rows(int np, int nrows, const int *order, const int *place,
                                                    const int *base, int ncolors, const int *rowptr, const int *col,
                                                    const double *val, int64_t nnz, const int *g_rowptr, int *g_col,
                                                    double *g_val, int64_t g_nnz, int4 *rows, int *gcol, int *coupled) {
    const int g = blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (g >= nrows) return;
    const int i = order[g], src = rowptr[i], end = rowptr[i + 1];
    const uint64_t below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    const int mine = place[i];
    int c = 0, over = ncolors;  // the row's colour: the last one with base[c] <= mine
    while (over - c > 1) {
        const int mid = (c + over) >> 1;
        if (base[mid] <= mine) c = mid;
        else over = mid;
    }
    const int first = base[c], last = base[c + 1] - 1;
    int dst = g_rowptr[g], diag = dst;
    bool bad = false;
    for (int cls = 0; cls < 3; ++cls) {
        if (cls == 1) diag = dst;
        for (int k0 = src; k0 < end; k0 += 64) {
            const int k = k0 + lane;
            const int j = k < end ? col[k] : -1;
            const int pj = j >= 0 ? place[j] : 0;
            const bool take = j >= 0 && (j == i ? cls == 1 : (pj < mine ? cls == 0 : cls == 2));
            bad |= j >= 0 && j != i && (pj < 0 || (pj >= first && pj <= last));
            const uint64_t mask = __ballot(take);
            if (take) {
                const int at = dst + __popcll(mask & below);
                g_col[at] = j;
                gcol[at] = pj;
                for (int p = 0; p < np; ++p) g_val[p * g_nnz + at] = val[p * nnz + k];
            }
            dst += __popcll(mask);
        }
        if (cls == 1) bad |= dst != diag + 1;
    }
    if (bad) atomicOr(coupled, 1);
    if (lane == 0) rows[g] = make_int4(g_rowptr[g], diag, dst, i);
}

void launch_split_rows(int np, int nrows, const int *order, const int *place, const int *base, int ncolors,
                       const int *rowptr, const int *col, const double *val, int64_t nnz, const int *g_rowptr,
                       int *g_col, double *g_val, int64_t g_nnz, int4 *rows, int *gcol, int *coupled, hipStream_t s) {
    if (nrows <= 0) return;
    k_split_rows<<<ceil_div(nrows, 4), 256, 0, s>>>(np, nrows, order, place, base, ncolors, rowptr, col, val, nnz,
                                                    g_rowptr, g_col, g_val, g_nnz, rows, gcol, coupled);
    AMG_CHECK_LAUNCH();
}

template <int MODE, int KIND, int G>
static void launch_g(const SweepArgs &a, const SweepShape &q, int later_rows, hipStream_t s) {
    const int grid = a.ntiles < q.grid ? a.ntiles : q.grid;
    if (later_rows > 0)
        k_later<MODE, KIND, G><<<ceil_div(static_cast<int64_t>(later_rows) * G, 256), 256, 0, s>>>(a, later_rows);
    else if (q.threads == SWEEP_THREADS_MIN)
        k_sweep<MODE, KIND, G, SWEEP_THREADS_MIN><<<grid, SWEEP_THREADS_MIN, 0, s>>>(a);
    else
        k_sweep<MODE, KIND, G, 2 * SWEEP_THREADS_MIN><<<grid, 2 * SWEEP_THREADS_MIN, 0, s>>>(a);
    AMG_CHECK_LAUNCH();
}

template <int MODE, int KIND>
static void launch_k(const SweepArgs &a, const SweepShape &q, int later_rows, hipStream_t s) {
    switch (q.G) {
        case 8: launch_g<MODE, KIND, 8>(a, q, later_rows, s); break;
        case 16: launch_g<MODE, KIND, 16>(a, q, later_rows, s); break;
        case 32: launch_g<MODE, KIND, 32>(a, q, later_rows, s); break;
        case 64: launch_g<MODE, KIND, 64>(a, q, later_rows, s); break;
        default: throw Error(AMG_EINVAL, "sweep kernel: 8, 16, 32 or 64 lanes per row");
    }
}

static void launch_any(int mode, int kind, const SweepShape &q, const SweepArgs &a, int later_rows, hipStream_t s) {
#define AMG_SWEEP_CASE(M, K) \
    if (mode == M && kind == K) return launch_k<M, K>(a, q, later_rows, s);
    AMG_SWEEP_CASE(SWEEP_BLOCK, SWEEP_F64)
    AMG_SWEEP_CASE(SWEEP_BLOCK, SWEEP_F32)
    AMG_SWEEP_CASE(SWEEP_BLOCK, SWEEP_BF16)
    AMG_SWEEP_CASE(SWEEP_SCALAR3, SWEEP_F64)
    AMG_SWEEP_CASE(SWEEP_SCALAR3, SWEEP_F32)
    AMG_SWEEP_CASE(SWEEP_SCALAR3, SWEEP_BF16)
    AMG_SWEEP_CASE(SWEEP_SCALAR1, SWEEP_F64)
    AMG_SWEEP_CASE(SWEEP_SCALAR1, SWEEP_F32)
#undef AMG_SWEEP_CASE
    throw Error(AMG_EINVAL, "sweep kernel: unsupported operator");
}

void launch_sweep(int mode, int kind, const SweepShape &q, const SweepArgs &a, hipStream_t s) {
    if (a.ntiles <= 0) return;
    AMG_REQUIRE(a.ncolors >= 1 && a.ncolors <= SWEEP_MAX_COLOURS, AMG_EINVAL, "sweep kernel: too many colours");
    AMG_REQUIRE(a.x_zero || a.x_old != a.x, AMG_EINVAL, "sweep kernel: the old iterate needs a buffer of its own");
    AMG_REQUIRE(a.forward || (!a.x_zero && !a.part), AMG_EINVAL, "sweep kernel: forward from zero or with a residual");
    launch_any(mode, kind, q, a, 0, s);
}

void launch_later(int mode, int kind, int nrows, const SweepShape &q, const SweepArgs &a, hipStream_t s) {
    if (nrows > 0) launch_any(mode, kind, q, a, nrows, s);
}

}  // namespace amgp2
