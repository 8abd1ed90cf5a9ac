// amg_solve_multi: K right-hand sides on one SPD hierarchy. The V-cycle of
// Algorithm 1 and the outer PCG / flexible CG run on interleaved blocks of K
// vectors (multi.h), so every matrix pass serves all K; each right-hand side
// keeps its own Krylov scalars, stopping test and iteration count, and one
// that has converged (or broken down) keeps its iterate while the others go
// on. Arithmetic per right-hand side is that of amg_solve up to the order of
// the floating-point sums.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <type_traits>

#include "context.h"
#include "multi.h"

namespace amgp2 {

static double mlevel_omega(amg_ctx *h, int l) {
    if (!h->level_omega.empty()) return h->level_omega[std::min<size_t>(l, h->level_omega.size() - 1)];
    return h->prm.omega;
}

// The cycle on block vectors. T = double (FP64 hierarchy) or float (the
// reduced-precision copies: FP32 finest, FP32 or BF16 below).
template <typename T>
struct MCycle {
    amg_ctx *h;
    MultiWork &W;
    int K;
    static constexpr bool RP = std::is_same<T, float>::value;

    int kind(const Level &L) const { return RP ? (L.mp.kind == VAL_BF16 ? MK_BF16 : MK_F32) : MK_F64; }
    const void *aval(const Level &L) const { return RP ? L.mp.aval() : static_cast<const void *>(L.A.val.p); }
    const void *agval(const Level &L) const { return RP ? L.mp.agval() : static_cast<const void *>(L.Ag.val.p); }
    const void *dinv(const Level &L) const {
        return RP ? static_cast<const void *>(L.mp.dinv.p) : static_cast<const void *>(L.dinv.p);
    }
    T *vx(int l) { return RP ? reinterpret_cast<T *>(W.lv[l].x32.p) : reinterpret_cast<T *>(W.lv[l].x.p); }
    T *vb(int l) { return RP ? reinterpret_cast<T *>(W.lv[l].b32.p) : reinterpret_cast<T *>(W.lv[l].b.p); }
    T *vr(int l) { return RP ? reinterpret_cast<T *>(W.lv[l].r32.p) : reinterpret_cast<T *>(W.lv[l].r.p); }
    T *vt(int l) { return RP ? reinterpret_cast<T *>(W.lv[l].t32.p) : reinterpret_cast<T *>(W.lv[l].t.p); }
    int64_t len(int l) const { return 3 * static_cast<int64_t>(h->lv[l].n) * K; }

    MRowArgs natural(const Level &L) const {
        MRowArgs a;
        a.nrows = L.n;
        a.rowptr = L.A.rowptr.p;
        a.col = L.A.col.p;
        a.val = aval(L);
        a.rscale = L.mp.scale.n ? L.mp.scale.p : nullptr;
        a.nnz = L.A.nnz;
        return a;
    }

    void fill0(T *x, int64_t n) {
        if (RP)
            launch_fill_f32(reinterpret_cast<float *>(x), 0.f, n, h->stream);
        else
            launch_fill(reinterpret_cast<double *>(x), 0.0, n, h->stream);
    }
    void copy(T *dst, const T *src, int64_t n) {
        if (RP)
            launch_copy_f32(reinterpret_cast<float *>(dst), reinterpret_cast<const float *>(src), n, h->stream);
        else
            launch_copy(reinterpret_cast<double *>(dst), reinterpret_cast<const double *>(src), n, h->stream);
    }

    // one damped Jacobi step, out of place into the other buffer of the
    // level's pair (vt, or vx when x is vt); returns the buffer with the result
    T *jacobi(int l, const T *b, T *x, bool zero) {
        Level &L = h->lv[l];
        const double om = mlevel_omega(h, l);
        if (zero) {
            launch_mjacobi_zero(L.mode, RP ? MK_F32 : MK_F64, K, L.n, dinv(L), b, om, x, h->stream);
            return x;
        }
        T *out = x == vt(l) ? vx(l) : vt(l);
        MRowArgs a = natural(L);
        a.x = x;
        a.b = b;
        a.y = out;
        a.dinv = dinv(L);
        a.dinv_n = L.n;
        a.omega = om;
        launch_mrow(L.mode, M_JACOBI, kind(L), K, a, h->stream);
        return out;
    }

    void gs(int l, const T *b, T *x, bool forward, bool x_zero) {
        Level &L = h->lv[l];
        const int ncol = static_cast<int>(L.cptr.size()) - 1;
        for (int q = 0; q < ncol; ++q) {
            const int c = forward ? q : ncol - 1 - q;
            const int r0 = L.cptr[c], r1 = L.cptr[c + 1];
            if (r1 == r0) continue;
            if (q == 0 && x_zero) {
                launch_mdiag_solve(L.mode, RP ? MK_F32 : MK_F64, K, r1 - r0, L.g_rowid.p + r0, dinv(L), L.n, b, x,
                                   h->stream);
                continue;
            }
            MRowArgs a;
            a.nrows = r1 - r0;
            a.rowptr = L.Ag.rowptr.p + r0;
            a.col = L.Ag.col.p;
            a.val = agval(L);
            a.rscale = L.mp.scale.n ? L.mp.scale.p : nullptr;
            a.nnz = L.Ag.nnz;
            a.rowid = L.g_rowid.p + r0;
            a.x = x;
            a.b = b;
            a.y = x;
            a.dinv = dinv(L);
            a.dinv_n = L.n;
            launch_mrow(L.mode, M_GS, kind(L), K, a, h->stream);
        }
    }

    T *smooth(int l, const T *b, T *x, bool pre, bool zero_init) {
        const amg_params &p = h->prm;
        const int steps = pre ? p.pre : p.post;
        if (zero_init && (steps == 0 || p.smoother != AMG_SMOOTH_JA)) fill0(x, len(l));
        for (int k = 0; k < steps; ++k) {
            if (p.smoother == AMG_SMOOTH_JA)
                x = jacobi(l, b, x, zero_init && k == 0);
            else
                gs(l, b, x, pre, pre && zero_init && k == 0);
        }
        return x;
    }

    // the coarsest level: the FP64 explicit inverse on all K columns
    void coarse(int l, const T *b, T *x) {
        const int64_t n = len(l);
        if (RP) {
            launch_to_f64(reinterpret_cast<const float *>(b), W.lv[l].b.p, n, h->stream);
            launch_mdense(MK_F64, h->coarse_inv.p, h->coarse_m, h->coarse_m, h->coarse_nc * K, W.lv[l].b.p,
                          W.lv[l].x.p, h->stream);
            launch_to_f32(W.lv[l].x.p, reinterpret_cast<float *>(x), n, h->stream);
        } else {
            launch_mdense(MK_F64, h->coarse_inv.p, h->coarse_m, h->coarse_m, h->coarse_nc * K, b, x, h->stream);
        }
    }

    // returns the buffer that holds x_l on return (Jacobi steps alternate)
    T *cycle(int l, const T *b, T *x, bool x_zero) {
        Level &L = h->lv[l];
        if (L.coarsest) {
            coarse(l, b, x);
            return x;
        }
        if (l == h->dense_start && x_zero) {
            const int nc = h->tail_nc * K;
            if (!RP)
                launch_mdense(MK_F64, h->tail_dense.p, h->tail_m, h->tail_m, nc, b, x, h->stream);
            else if (h->tail_dense16.n)
                launch_mdense(MK_BF16, h->tail_dense16.p, h->tail_m, h->tail_ld, nc, b, x, h->stream);
            else
                launch_mdense(MK_F32, h->tail_dense32.p, h->tail_m, h->tail_ld, nc, b, x, h->stream);
            return x;
        }
        x = smooth(l, b, x, true, x_zero);
        {
            MRowArgs a = natural(L);
            a.x = x;
            a.b = b;
            a.y = vr(l);
            launch_mrow(L.mode, M_RESID, kind(L), K, a, h->stream);
        }
        Level &C = h->lv[l + 1];
        {
            MRowArgs a;
            a.nrows = L.R.nrows;
            a.rowptr = L.R.rowptr.p;
            a.col = L.R.col.p;
            a.val = RP ? static_cast<const void *>(L.mp.rval.p) : static_cast<const void *>(L.R.val.p);
            a.nnz = L.R.nnz;
            a.x = vr(l);
            a.y = vb(l + 1);
            a.zero_out = vx(l + 1);
            launch_mrow(1, M_SPMV, RP ? MK_F32 : MK_F64, K, a, h->stream);
        }
        T *e = vx(l + 1);
        if (C.coarsest) {
            coarse(l + 1, vb(l + 1), e);
        } else {
            const int nu = l + 1 == h->dense_start ? 1 : std::max(1, h->prm.nu);
            for (int k = 0; k < nu; ++k) e = cycle(l + 1, vb(l + 1), e, k == 0);
        }
        {
            MRowArgs a;
            a.nrows = L.P.nrows;
            a.rowptr = L.P.rowptr.p;
            a.col = L.P.col.p;
            a.val = RP ? static_cast<const void *>(L.mp.pval.p) : static_cast<const void *>(L.P.val.p);
            a.nnz = L.P.nnz;
            a.x = e;
            a.y = x;
            launch_mrow(1, M_SPMV_ADD, RP ? MK_F32 : MK_F64, K, a, h->stream);
        }
        return smooth(l, b, x, false, false);
    }

    // M^{-1} r on blocks of the finest level, left where the cycle ends
    const T *precondition(const T *r, T *x) {
        const int cyc = std::max(1, h->prm.cycles);
        for (int k = 0; k < cyc; ++k) x = cycle(0, r, x, k == 0);
        return x;
    }
};

static void multi_alloc(amg_ctx *h, MultiWork &W, int K) {
    if (W.K == K && W.lv.size() == h->lv.size()) return;  // kept from the last call with this K
    W.K = K;
    W.lv.resize(h->lv.size());
    for (size_t l = 0; l < h->lv.size(); ++l) {
        const size_t n = 3 * static_cast<size_t>(h->lv[l].n) * K;
        MultiLevelWork &w = W.lv[l];
        if (h->mixed) {
            w.x32.alloc(n);
            w.b32.alloc(n);
            w.r32.alloc(n);
            w.t32.alloc(n);
            if (h->lv[l].coarsest) {
                w.x.alloc(n);
                w.b.alloc(n);
            }
        } else {
            w.x.alloc(n);
            w.b.alloc(n);
            w.r.alloc(n);
            w.t.alloc(n);
        }
    }
    const size_t nd = static_cast<size_t>(h->n_dof) * K;
    for (DevBuf<double> *v : {&W.B, &W.X, &W.R, &W.Z, &W.P, &W.Q}) v->alloc(nd);
    W.partial.alloc(static_cast<size_t>(mdot_blocks(h->n_dof)) * K);
    if (!W.h_dots)
        AMG_HIP(hipHostMalloc(reinterpret_cast<void **>(&W.h_dots), 2 * MULTI_MAX_K * sizeof(double),
                              hipHostMallocCoherent));
}

// y = A x on the finest level (FP64), K columns
static void mapply(amg_ctx *h, int K, const double *x, double *y) {
    Level &L = h->lv[0];
    MRowArgs a;
    a.nrows = L.n;
    a.rowptr = L.A.rowptr.p;
    a.col = L.A.col.p;
    a.val = L.A.val.p;
    a.nnz = L.A.nnz;
    a.x = x;
    a.y = y;
    launch_mrow(L.mode, M_SPMV, MK_F64, K, a, h->stream);
}

// the sums that the launches so far have left in h_dots
static void msync(amg_ctx *h) { AMG_HIP(hipStreamSynchronize(h->stream)); }

static std::vector<double> mnorms(amg_ctx *h, MultiWork &W, const double *v) {
    launch_mdot(W.K, h->n_dof, v, v, W.partial.p, W.h_dots, h->stream);
    msync(h);
    return std::vector<double>(W.h_dots, W.h_dots + W.K);
}

int solve_multi(amg_ctx *h, int nrhs, const double *B, double *X, double tol, int maxit, amg_result *res) {
    const auto t0 = std::chrono::steady_clock::now();
    AMG_REQUIRE(!h->saddle && h->nsys == 0, AMG_EINVAL, "amg_solve_multi: SPD systems only");
    AMG_REQUIRE(h->prm.krylov == AMG_KRYLOV_PCG || h->prm.krylov == AMG_KRYLOV_FCG, AMG_EINVAL,
                "amg_solve_multi: needs PCG or FCG");
    AMG_REQUIRE(!h->post_forward, AMG_EINVAL, "amg_solve_multi: needs the symmetric cycle");
    AMG_REQUIRE(nrhs >= 1 && nrhs <= MULTI_MAX_K, AMG_EINVAL, "amg_solve_multi: 1 to 8 right-hand sides");
    const int K = nrhs <= 2 ? 2 : (nrhs <= 4 ? 4 : 8);
    MultiWork &W = h->multi;
    multi_alloc(h, W, K);
    hipStream_t s = h->stream;
    const int64_t nd = h->n_dof;
    launch_interleave(K, nrhs, nd, B, W.B.p, true, s);
    launch_interleave(K, nrhs, nd, X, W.X.p, true, s);
    MCycle<double> c64{h, W, K};
    MCycle<float> c32{h, W, K};
    // z of the last preconditioner application: FP32 as a reduced-precision
    // cycle leaves it (its copy of r is r32), else FP64
    const double *z64 = nullptr;
    const float *z32 = nullptr;
    float *const r32 = h->mixed ? W.lv[0].b32.p : nullptr;
    auto prec = [&] {
        if (h->mixed)
            z32 = c32.precondition(r32, W.lv[0].x32.p);
        else
            z64 = c64.precondition(W.R.p, W.Z.p);
    };
    // sums into h_dots: dot(v) <z, v> at K; direction(r) <p, r> at K
    double *const second = W.h_dots + K;
    auto dot_z = [&](const double *v) {
        if (h->mixed)
            launch_mdot(K, nd, z32, v, W.partial.p, second, s);
        else
            launch_mdot(K, nd, z64, v, W.partial.p, second, s);
    };
    auto direction = [&](const MCoef &beta, bool first, const double *r) {
        if (h->mixed)
            launch_mdirection<float>(K, nd, beta, first, z32, W.P.p, r, W.partial.p, second, s);
        else
            launch_mdirection<double>(K, nd, beta, first, z64, W.P.p, r, W.partial.p, second, s);
    };
    // R = B - A X
    mapply(h, K, W.X.p, W.R.p);
    launch_msubtract(nd * K, W.B.p, W.R.p, s);
    if (h->mixed) launch_to_f32(W.R.p, r32, nd * K, s);
    std::vector<double> rr0 = mnorms(h, W, W.R.p);
    std::vector<int> status(K, AMG_NOT_CONVERGED), iters(K, 0), active(K, 0);
    for (int r = 0; r < K; ++r) {
        if (r >= nrhs || rr0[r] == 0.0) {
            status[r] = AMG_OK;
        } else if (!(rr0[r] == rr0[r]) || std::isinf(rr0[r])) {
            status[r] = AMG_DIVERGED;
        } else {
            active[r] = 1;
        }
    }
    auto any_active = [&]() { return std::any_of(active.begin(), active.end(), [](int a) { return a != 0; }); };
    const bool fcg = h->prm.krylov == AMG_KRYLOV_FCG;
    std::vector<double> rz(K, 0.0), pq_prev(K, 0.0);
    MCoef alpha, beta;
    int it = 0;
    if (!fcg && any_active()) {
        prec();
        dot_z(W.R.p);
        direction(beta, true, nullptr);
        msync(h);
        std::copy(second, second + K, rz.begin());
    }
    // While every running column's last relative residual is above
    // KRYLOV_AHEAD * tol, the next preconditioner application goes ahead of
    // the stopping test's read, and its dot (<r, z> for CG, <z, q> for FCG)
    // comes back in the same read: one host round trip less per iteration,
    // the same arithmetic.
    double relmin = 1.0;
    bool ahead = false;             // z of this iteration already computed
    std::vector<double> zdot(K);    // its dot, read with the last stopping test
    auto z_and_dot = [&](const double *v) {
        if (ahead) return;
        prec();
        dot_z(v);
        msync(h);
        std::copy(second, second + K, zdot.begin());
    };
    while (it < maxit && any_active()) {
        if (fcg) {
            // beta = -<z, q_prev> / <p_prev, q_prev>: p = z + beta p_prev
            if (it == 0) {
                prec();
            } else {
                z_and_dot(W.Q.p);
                for (int r = 0; r < K; ++r) beta.c[r] = active[r] && pq_prev[r] != 0.0 ? -zdot[r] / pq_prev[r] : 0.0;
            }
            direction(beta, it == 0, W.R.p);
        }
        mapply(h, K, W.P.p, W.Q.p);
        launch_mdot(K, nd, W.P.p, W.Q.p, W.partial.p, W.h_dots, s);
        msync(h);
        for (int r = 0; r < K; ++r) {
            alpha.c[r] = 0.0;
            if (!active[r]) continue;
            const double pq = W.h_dots[r];
            if (!(pq > 0.0) || !std::isfinite(pq)) {
                status[r] = (pq == pq) ? AMG_BREAKDOWN : AMG_DIVERGED;
                active[r] = 0;
                continue;
            }
            alpha.c[r] = (fcg ? second[r] : rz[r]) / pq;
            pq_prev[r] = pq;
        }
        launch_mupdate(K, nd, alpha, W.P.p, W.Q.p, W.X.p, W.R.p, r32, W.partial.p, W.h_dots, s);
        ++it;
        ahead = it < maxit && relmin > KRYLOV_AHEAD * tol;
        if (ahead) {
            prec();
            dot_z(fcg ? W.Q.p : W.R.p);
        }
        msync(h);
        const std::vector<double> rrv(W.h_dots, W.h_dots + K);
        if (ahead) std::copy(second, second + K, zdot.begin());
        relmin = 1e300;
        for (int r = 0; r < K; ++r) {
            if (!active[r]) continue;
            iters[r] = it;
            const double rr = rrv[r];
            if (!(rr == rr) || std::isinf(rr) || std::sqrt(rr / rr0[r]) > 1e3) {
                status[r] = AMG_DIVERGED;
                active[r] = 0;
            } else if (std::sqrt(rr / rr0[r]) <= tol) {
                status[r] = AMG_OK;
                active[r] = 0;
            } else {
                relmin = std::min(relmin, std::sqrt(rr / rr0[r]));
            }
        }
        if (!fcg && it < maxit && any_active()) {
            z_and_dot(W.R.p);
            for (int r = 0; r < K; ++r) {
                beta.c[r] = active[r] && rz[r] != 0.0 ? zdot[r] / rz[r] : 0.0;
                if (active[r]) rz[r] = zdot[r];
            }
            direction(beta, false, nullptr);
        }
    }
    // true residuals
    mapply(h, K, W.X.p, W.R.p);
    launch_msubtract(nd * K, W.B.p, W.R.p, s);
    std::vector<double> rr = mnorms(h, W, W.R.p);
    launch_interleave(K, nrhs, nd, W.X.p, X, false, s);
    AMG_HIP(hipStreamSynchronize(s));
    const double ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
    int worst = AMG_OK;
    for (int r = 0; r < nrhs; ++r) {
        const double rel = rr0[r] > 0.0 ? std::sqrt(rr[r] / rr0[r]) : 0.0;
        int st = status[r];
        if (st == AMG_OK && !(rel == rel)) st = AMG_DIVERGED;
        if (res) {
            res[r].iters = iters[r];
            res[r].status = st;
            res[r].relres = rel;
            res[r].solve_ms = ms;
        }
        worst = std::max(worst, st);
    }
    return worst;
}

}  // namespace amgp2
