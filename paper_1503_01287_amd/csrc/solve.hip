// amg_solve: Algorithm 1 (the basic AMG iteration) and the outer Krylov
// drivers. Every vector operation runs on the GPU; Krylov scalars stay in a
// device array, and the host reads one residual norm per iteration for the
// stopping test.
#include <chrono>
#include <cmath>

#include "context.h"

namespace amgp2 {

// ---------------------------------------------------------------- profiling
ProfScope::ProfScope(amg_ctx *hh, const std::string &cls, double bytes) : h(hh), idx(0) {
    if (!h->prof) return;
    if (h->prof_finest_only && cls.size() > 3 && cls.compare(cls.size() - 3, 3, ".L0") != 0) return;
    amg_ctx::Pending pe;
    pe.cls = cls;
    pe.bytes = bytes;
    // timing-only events: no system-scope fence (its L2 writeback and
    // invalidate would lengthen the interval and slow the next kernel);
    // profile_collect synchronises the stream before reading them
    for (hipEvent_t *e : {&pe.a, &pe.b}) {
        if (!h->event_pool.empty()) {
            *e = h->event_pool.back();
            h->event_pool.pop_back();
        } else {
            AMG_HIP(hipEventCreateWithFlags(e, hipEventDisableSystemFence));
        }
    }
    AMG_HIP(hipEventRecord(pe.a, h->stream));
    h->pending.push_back(pe);
    idx = h->pending.size();
}

ProfScope::~ProfScope() {
    if (!h->prof || idx == 0) return;
    (void)hipEventRecord(h->pending[idx - 1].b, h->stream);
}

void profile_collect(amg_ctx *h) {
    if (h->pending.empty()) return;
    AMG_HIP(hipStreamSynchronize(h->stream));
    for (auto &pe : h->pending) {
        float ms = 0.f;
        AMG_HIP(hipEventElapsedTime(&ms, pe.a, pe.b));
        ProfStat &st = h->stats[pe.cls];
        st.launches += 1;
        st.ms += ms;
        st.bytes += pe.bytes;
        h->event_pool.push_back(pe.a);
        h->event_pool.push_back(pe.b);
    }
    h->pending.clear();
}

// algorithmic bytes of one pass over rows [.., ..) of a block operator
static double row_bytes(const DMat &m, int64_t nnz, int nrows) {
    return static_cast<double>(nnz) * (m.np * 8.0 + 4.0) + nrows * 4.0;
}

static RowArgs row_args(const DMat &m) {
    RowArgs a;
    a.nrows = m.nrows;
    a.rowptr = m.rowptr.p;
    a.col = m.col.p;
    a.val = m.val.p;
    a.nnz = m.nnz;
    return a;
}

static std::string tag(const char *cls, int l) { return std::string(cls) + ".L" + std::to_string(l); }

// The level's operator in tiles, where it has them.
static bool in_tiles(const Level &L) { return L.tiles.v64.n > 0 && !L.by_rows; }

// ---------------------------------------------------------------- level ops
void apply_level(amg_ctx *h, int l, const double *x, double *y) {
    Level &L = h->lv[l];
    if (in_tiles(L) && x != y) {
        TileArgs a = L.tiles.args(TILE_F64);
        a.x = x;
        a.y = y;
        ProfScope ps(h, tag("spmv", l), L.tiles.bytes(TILE_F64, L.A.nnz) + 3.0 * L.n * 16.0);
        launch_tile(TILE_SPMV, TILE_F64, a, h->stream);
        return;
    }
    RowArgs a = row_args(L.A);
    a.x = x;
    a.y = y;
    ProfScope ps(h, tag("spmv", l), row_bytes(L.A, L.A.nnz, L.n) + 3.0 * L.n * 16.0);
    a.trip = L.trip;
    launch_row(L.mode, OP_SPMV, L.G, a, h->stream);
}

// r = b - A x on the level's first `rows` rows (all of them: -1)
static void residual(amg_ctx *h, int l, const double *b, const double *x, double *r, int rows = -1) {
    Level &L = h->lv[l];
    if (in_tiles(L) && (rows < 0 || rows == L.n)) {
        TileArgs a = L.tiles.args(TILE_F64);
        a.x = x;
        a.b = b;
        a.y = r;
        ProfScope ps(h, tag("resid", l), L.tiles.bytes(TILE_F64, L.A.nnz) + 3.0 * L.n * 24.0);
        launch_tile(TILE_RESID, TILE_F64, a, h->stream);
        return;
    }
    RowArgs a = row_args(L.A);
    if (rows >= 0) a.nrows = rows;
    a.x = x;
    a.b = b;
    a.y = r;
    ProfScope ps(h, tag("resid", l), row_bytes(L.A, L.A.nnz, L.n) + 3.0 * L.n * 24.0);
    a.trip = L.trip;
    launch_row(L.mode, OP_RESID, L.G, a, h->stream);
}

static double level_omega(amg_ctx *h, int l) {
    if (!h->level_omega.empty())
        return h->level_omega[std::min<size_t>(l, h->level_omega.size() - 1)];
    return h->prm.omega;
}

// (on the level's leading nA rows: the systems of a batch that continue
// below the level; every row outside batches)
static void jacobi_step(amg_ctx *h, int l, const double *b, double *x, bool zero_init) {
    Level &L = h->lv[l];
    const double om = level_omega(h, l);
    const int nb = L.mode == 3 ? 9 : 1;
    if (zero_init) {
        ProfScope ps(h, tag("jacobi0", l), 3.0 * L.n * 16.0 + nb * 8.0 * L.n);
        launch_jacobi_zero(L.mode, L.nA, L.dinv.p, L.n, b, om, x, h->stream);
        return;
    }
    RowArgs a = row_args(L.A);
    a.nrows = L.nA;
    a.x = x;
    a.b = b;
    a.y = L.t.p;
    a.dinv = L.dinv.p;
    a.dinv_n = L.n;
    a.omega = om;
    if (in_tiles(L) && L.nA == L.n) {
        TileArgs q = L.tiles.args(TILE_F64);
        q.x = x;
        q.b = b;
        q.y = L.t.p;
        q.dinv = L.dinv.p;
        q.omega = om;
        ProfScope ps(h, tag("jacobi", l), L.tiles.bytes(TILE_F64, L.A.nnz) + 3.0 * L.n * 24.0 + 8.0 * L.n);
        launch_tile(TILE_JACOBI, TILE_F64, q, h->stream);
    } else {
        ProfScope ps(h, tag("jacobi", l), row_bytes(L.A, L.A.nnz, L.n) + 3.0 * L.n * 24.0 + nb * 8.0 * L.n);
        a.trip = L.trip;
        launch_row(L.mode, OP_JACOBI, L.G, a, h->stream);
    }
    launch_copy(x, L.t.p, 3 * static_cast<int64_t>(L.nA), h->stream);
}

// One block Gauss-Seidel sweep by colours. x_zero: x is zero on entry (and
// its buffer holds the zeros), so the first colour's rows see only zero
// neighbours: x_i = D_i^{-1} b_i without reading their matrix rows.
// in_t: the iterate on entry is in L.t (one-launch sweeps read it there).
// part: see SweepArgs::part (one-launch forward sweeps).
static SweepArgs sweep_args(Level &L, const double *b, double *x, bool forward, bool x_zero, double *part) {
    SweepArgs a;
    L.sweep.fill(a, L.shape, L.sweep.f64);
    a.col = L.Ag.col.p;
    a.val = L.Ag.val.p;
    a.nnz = L.Ag.nnz;
    a.dinv = L.dinv.p;
    a.dinv_n = L.n;
    a.b = b;
    a.x_old = L.t.p;
    a.x = x;
    a.part = part;
    a.forward = forward ? 1 : 0;
    a.x_zero = x_zero ? 1 : 0;
    return a;
}

static void gs_sweep(amg_ctx *h, int l, const double *b, double *x, bool forward, bool x_zero, bool in_t,
                     double *part) {
    Level &L = h->lv[l];
    if (one_launch_sweeps(h, L, false)) {
        if (!x_zero && !in_t) launch_copy(L.t.p, x, 3 * static_cast<int64_t>(L.nA), h->stream);
        const double rows = L.Ag.nrows;
        ProfScope ps(h, tag("gs", l), row_bytes(L.Ag, x_zero ? L.Ag.nnz / 2 : L.Ag.nnz, L.Ag.nrows) +
                                          rows * (8.0 + 24.0 + 48.0 + (L.mode == 3 ? 72.0 : 8.0)));
        launch_sweep(L.mode, SWEEP_F64, L.shape, sweep_args(L, b, x, forward, x_zero, part), h->stream);
        return;
    }
    const int ncol = static_cast<int>(L.cptr.size()) - 1;
    const int nb = L.mode == 3 ? 9 : 1;
    for (int q = 0; q < ncol; ++q) {
        const int c = forward ? q : ncol - 1 - q;
        const int r0 = L.cptr[c], r1 = L.cptr[c + 1];
        if (r1 == r0) continue;
        if (q == 0 && x_zero) {
            ProfScope ps(h, tag("gs", l), (r1 - r0) * (4.0 + 48.0 + nb * 8.0));
            launch_diag_solve(L.mode, r1 - r0, L.g_rowid.p + r0, L.dinv.p, L.n, b, x, h->stream);
            continue;
        }
        RowArgs a;
        a.nrows = r1 - r0;
        a.rowptr = L.Ag.rowptr.p + r0;
        a.col = L.Ag.col.p;
        a.val = L.Ag.val.p;
        a.nnz = L.Ag.nnz;
        a.rowid = L.g_rowid.p + r0;
        a.x = x;
        a.b = b;
        a.y = x;
        a.dinv = L.dinv.p;
        a.dinv_n = L.n;
        a.xcd_chunks = L.gs_xcd;
        // matrix rows of this colour + row pointer, row id, b_i, x_i read and
        // write, inverted diagonal block
        const double bytes = static_cast<double>(L.colour_nnz[c]) * (L.Ag.np * 8.0 + 4.0) +
                             a.nrows * (8.0 + 24.0 + 48.0 + nb * 8.0);
        ProfScope ps(h, tag("gs", l), bytes);
        a.trip = L.tripg;
        launch_row(L.mode, OP_GS, L.Gg, a, h->stream);
    }
}

// zero_init: x is zero on entry; filled: its buffer already holds the zeros;
// in_t: the iterate on entry is in L.t; part: written by the last sweep
static void smooth_from(amg_ctx *h, int l, const double *b, double *x, bool pre, bool zero_init, bool filled,
                        bool in_t, double *part) {
    const amg_params &p = h->prm;
    const int steps = pre ? p.pre : p.post;
    Level &L = h->lv[l];
    const bool need_fill =
        zero_init && !filled && (steps == 0 || (p.smoother != AMG_SMOOTH_JA && !(pre && one_launch_sweeps(h, L, false))));
    if (need_fill) launch_fill(x, 0.0, 3 * static_cast<int64_t>(L.nA), h->stream);
    for (int k = 0; k < steps; ++k) {
        if (p.smoother == AMG_SMOOTH_JA)
            jacobi_step(h, l, b, x, zero_init && k == 0);
        else
            gs_sweep(h, l, b, x, pre || h->post_forward, pre && zero_init && k == 0, in_t && k == 0,
                     k == steps - 1 ? part : nullptr);
    }
}

void smooth(amg_ctx *h, int l, const double *b, double *x, bool pre, bool zero_init, bool filled) {
    smooth_from(h, l, b, x, pre, zero_init, filled, false, nullptr);
}

static void coarse_solve(amg_ctx *h, const double *b, double *x) {
    ProfScope ps(h, "coarse", static_cast<double>(h->coarse_m) * h->coarse_m * 8.0);
    launch_dense_gemv(h->coarse_inv.p, h->coarse_m, h->coarse_nc, b, x, h->stream);
}

// a batch of SPD systems: the systems ending on level l (its rows past nA)
// by their explicit inverses
static void ending_systems(amg_ctx *h, int l, const double *b, double *x) {
    Level &L = h->lv[l];
    if (L.dseg.count == 0) return;
    ProfScope ps(h, "coarse", L.dseg.bytes);
    launch_dense_segs<double>(L.dseg.view(), b, b, x, x, h->stream);
}

static void run_dense_tail(amg_ctx *h, const double *b, double *x) {
    ProfScope ps(h, "dense_tail", static_cast<double>(h->tail_m) * h->tail_m * 8.0);
    launch_dense_gemv(h->tail_dense.p, h->tail_m, h->tail_nc, b, x, h->stream);
}

// Algorithm 1: AMG(K_l, x_l, b_l). x_zero: x_l is zero on entry (the first
// Jacobi step then needs no operator pass); filled: its buffer holds the zeros.
static void cycle(amg_ctx *h, int l, const double *b, double *x, bool x_zero, bool filled) {
    Level &L = h->lv[l];
    if (h->nsys > 0) ending_systems(h, l, b, x);
    if (L.coarsest) {
        if (h->nsys == 0) coarse_solve(h, b, x);
        return;
    }
    if (l == h->dense_start && x_zero) {
        run_dense_tail(h, b, x);
        return;
    }
    if (h->prm.pre > 0 && one_launch_sweeps(h, L, false)) {
        // the last pre-smoothing sweep leaves all of the residual but the
        // entries of later colours
        smooth_from(h, l, b, x, true, x_zero, filled, false, L.r.p);
        ProfScope ps(h, tag("resid", l), row_bytes(L.Ag, L.Ag.nnz / 2, L.Ag.nrows) + 3.0 * L.Ag.nrows * 24.0);
        launch_later(L.mode, SWEEP_F64, L.Ag.nrows, L.shape, sweep_args(L, b, x, true, x_zero, L.r.p), h->stream);
    } else {
        smooth_from(h, l, b, x, true, x_zero, filled, false, nullptr);
        residual(h, l, b, x, L.r.p, L.nA);
    }
    Level &C = h->lv[l + 1];
    {
        // b_{l+1} = P^T r; the same pass zeroes x_{l+1} for the recursion
        RowArgs a = row_args(L.R);
        a.x = L.r.p;
        a.y = C.b.p;
        a.zero_out = C.x.p;
        ProfScope ps(h, tag("restrict", l), row_bytes(L.R, L.R.nnz, L.R.nrows) + 3.0 * (L.n + 2 * C.n) * 8.0);
        launch_row(1, OP_SPMV, L.Gr, a, h->stream);
    }
    if (C.coarsest) {
        if (h->nsys > 0) ending_systems(h, l + 1, C.b.p, C.x.p);
        else coarse_solve(h, C.b.p, C.x.p);
    } else {
        // x_{l+1} = 0, then nu recursive calls (nu = 1: V-cycle, 2: W-cycle;
        // the assembled coarse end covers all of them)
        const int nu = l + 1 == h->dense_start ? 1 : std::max(1, h->prm.nu);
        for (int k = 0; k < nu; ++k) cycle(h, l + 1, C.b.p, C.x.p, k == 0, k == 0);
    }
    // one-launch sweeps read their iterate from L.t: the prolongation puts it there
    const bool to_t = h->prm.post > 0 && one_launch_sweeps(h, L, false);
    {
        RowArgs a = row_args(L.P);
        a.x = C.x.p;
        a.base = x;
        a.y = to_t ? L.t.p : x;
        ProfScope ps(h, tag("prolong", l), row_bytes(L.P, L.P.nnz, L.P.nrows) + 3.0 * (2.0 * L.n + C.n) * 8.0);
        launch_row(1, OP_SPMV_ADD, L.Gp, a, h->stream);
    }
    smooth_from(h, l, b, x, false, false, false, to_t, nullptr);
}

void vcycle(amg_ctx *h, int l, const double *b, double *x) { cycle(h, l, b, x, true, false); }

// z = M^{-1} r: `cycles` successive applications of Algorithm 1 on the
// finest level, the first from z = 0, each further one from the current z.
static void precondition_eager(amg_ctx *h, const double *r, double *z) {
    if (h->saddle) {
        saddle_precondition(h, r, z);
        return;
    }
    if (h->mixed) {
        precondition_mp(h, r, z);
        return;
    }
    const int cyc = std::max(1, h->prm.cycles);
    for (int k = 0; k < cyc; ++k) cycle(h, 0, r, z, k == 0, false);
}

// Launches recorded once into a HIP graph and replayed: one launch call
// instead of hundreds. The recording runs on a stream of the library's own (a
// capture cannot run on the legacy default stream) and contains kernels only:
// no host synchronisation, no memset or copy nodes, no event records
// (profiling runs eagerly).
template <typename F>
static hipGraphExec_t record_graph(amg_ctx *h, F &&launches) {
    hipStream_t cs = nullptr;
    AMG_HIP(hipStreamCreateWithFlags(&cs, hipStreamNonBlocking));
    // the capture stream must see everything ordered before it on the caller's stream
    hipEvent_t ev;
    AMG_HIP(hipEventCreateWithFlags(&ev, hipEventDisableTiming));
    AMG_HIP(hipEventRecord(ev, h->stream));
    AMG_HIP(hipStreamWaitEvent(cs, ev, 0));
    const hipStream_t saved = h->stream;
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    h->stream = cs;
    AMG_HIP(hipStreamBeginCapture(cs, hipStreamCaptureModeRelaxed));
    try {
        launches();
    } catch (...) {
        (void)hipStreamEndCapture(cs, &graph);
        if (graph) (void)hipGraphDestroy(graph);
        h->stream = saved;
        (void)hipStreamDestroy(cs);
        (void)hipEventDestroy(ev);
        throw;
    }
    h->stream = saved;
    AMG_HIP(hipStreamEndCapture(cs, &graph));
    AMG_HIP(hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0));
    AMG_HIP(hipGraphDestroy(graph));
    AMG_HIP(hipStreamSynchronize(cs));
    AMG_HIP(hipStreamDestroy(cs));
    AMG_HIP(hipEventDestroy(ev));
    return exec;
}

// the preconditioner's graph, one per (r, z) pair
static hipGraphExec_t graph_for(amg_ctx *h, const double *r, double *z) {
    for (const auto &g : h->graphs)
        if (g.kind == GRAPH_PRECONDITION && g.r == r && g.z == z) return g.exec;
    if (h->graphs.size() >= 8) return nullptr;
    h->graphs.push_back({GRAPH_PRECONDITION, r, z, record_graph(h, [&] { precondition_eager(h, r, z); })});
    return h->graphs.back().exec;
}

// z = M^{-1} r for pointers that stay the same from call to call
static void precondition_impl(amg_ctx *h, const double *r, double *z) {
    if (h->prm.graph && !h->prof) {
        if (hipGraphExec_t g = graph_for(h, r, z)) {
            AMG_HIP(hipGraphLaunch(g, h->stream));
            return;
        }
    }
    precondition_eager(h, r, z);
}

// the reduced-precision cycle from mp.b of the finest level, as a graph where
// the solver records them; its result is at cg_z, the same buffer every time
static void cycle_f32_eager(amg_ctx *h) { h->cg_z = h->saddle ? saddle_precondition_f32(h) : precondition_f32(h); }
static void cycle_f32(amg_ctx *h) {
    if (h->prm.graph && !h->prof) {
        for (const auto &g : h->graphs)
            if (g.kind == GRAPH_CYCLE_F32) {
                AMG_HIP(hipGraphLaunch(g.exec, h->stream));
                return;
            }
        if (h->graphs.size() < 8) {
            h->graphs.push_back({GRAPH_CYCLE_F32, nullptr, nullptr, record_graph(h, [&] { cycle_f32_eager(h); })});
            AMG_HIP(hipGraphLaunch(h->graphs.back().exec, h->stream));
            return;
        }
    }
    cycle_f32_eager(h);
}

// z = M^{-1} r for pointers that change from call to call (the flexible
// GMRES basis): through staging vectors so that one recording serves all
// A reduced-precision cycle starts and ends in FP32 vectors of its own, so the
// conversions stand outside its recording and no staging is needed: two
// launches and two copies of a vector (4-12 us each) less. With in_b32 the
// cycle's right-hand side mp.b holds r already.
void precondition_step(amg_ctx *h, const double *r, double *z, bool in_b32) {
    if (h->mixed) {
        Level &L = h->lv[0];
        if (!in_b32) launch_to_f32(r, L.mp.b.p, L.vlen(), h->stream);
        cycle_f32(h);
        launch_to_f64(h->cg_z, z, L.vlen(), h->stream);
        return;
    }
    if (!h->prm.graph || h->prof) {
        precondition_eager(h, r, z);
        return;
    }
    if (h->g_in.n != static_cast<size_t>(h->n_dof)) {
        h->g_in.alloc(h->n_dof);
        h->g_out.alloc(h->n_dof);
    }
    launch_copy(h->g_in.p, r, h->n_dof, h->stream);
    precondition_impl(h, h->g_in.p, h->g_out.p);
    launch_copy(z, h->g_out.p, h->n_dof, h->stream);
}

void precondition(amg_ctx *h, const double *r, double *z) { precondition_impl(h, r, z); }

}  // namespace amgp2

// ---------------------------------------------------------------- Krylov
namespace amgp2 {

static double read_scalar(amg_ctx *h, int idx) {
    AMG_HIP(hipMemcpyAsync(h->h_sc, h->sc.p, SC_COUNT * sizeof(double), hipMemcpyDeviceToHost, h->stream));
    AMG_HIP(hipStreamSynchronize(h->stream));
    return h->h_sc[idx];
}

// The stopping test's scalars, which the update's reduction has written to
// pinned host memory, waited on separately (scalars_wait), so that work
// enqueued in between overlaps the host's round trip.
static void scalars_begin(amg_ctx *h) {
    if (!h->sc_ready) AMG_HIP(hipEventCreateWithFlags(&h->sc_ready, hipEventDisableTiming));
    AMG_HIP(hipEventRecord(h->sc_ready, h->stream));
}
static void scalars_wait(amg_ctx *h) { AMG_HIP(hipEventSynchronize(h->sc_ready)); }

// CG's stopping test waits for the scalars of iteration k on the host; while
// the last test's relative residual is still above KRYLOV_AHEAD * tol, the
// next preconditioner application, which only reads r and writes z, is
// enqueued before that wait, so the round trip overlaps the GPU's cycle. If
// the test then stops the solve, that application has changed nothing else.

template <typename T>
static void dot_into(amg_ctx *h, const T *a, const double *b, int dst, int post = RED_NONE) {
    ProfScope ps(h, "blas", h->n_dof * (8.0 + sizeof(T)));
    const int nb = launch_dot_partial(a, b, h->n_dof, h->partial.p, h->stream);
    launch_reduce(h->partial.p, nb, h->sc.p, dst, h->stream, post);
}

// q = A p on the finest level and <p, q> into sc[SC_PQ]
static void spmv_dot(amg_ctx *h, const double *p, double *q, int post) {
    Level &L = h->lv[0];
    RowArgs a = row_args(L.A);
    a.x = p;
    a.y = q;
    a.partial = h->partial.p;
    int nb = row_blocks(L.n, L.G);
    if (in_tiles(L)) {
        TileArgs t = L.tiles.args(TILE_F64);
        t.x = p;
        t.y = q;
        t.partial = h->partial.p;
        nb = ceil_div(L.n, TILE_ROWS);
        ProfScope ps(h, "spmv.L0", L.tiles.bytes(TILE_F64, L.A.nnz) + 3.0 * L.n * 16.0);
        launch_tile(TILE_SPMV_DOT, TILE_F64, t, h->stream);
    } else {
        ProfScope ps(h, "spmv.L0", row_bytes(L.A, L.A.nnz, L.n) + 3.0 * L.n * 16.0);
        a.trip = L.trip;
        launch_row(L.mode, OP_SPMV_DOT, L.G, a, h->stream);
    }
    launch_reduce(h->partial.p, nb, h->sc.p, SC_PQ, h->stream, post);
}

// A reduced-precision cycle inside CG: its copy of r is written by the update
// and its z read as it is, in FP32.
static bool cg_f32(const amg_ctx *h) { return h->mixed && !h->saddle; }

// x += alpha p, r -= alpha q, <r, r> into sc[SC_RR] and, with <p, q>, into
// the host's copy
static void cg_update(amg_ctx *h, double *x, double *r, const double *p, const double *q) {
    float *r32 = cg_f32(h) ? h->lv[0].mp.b.p : nullptr;
    ProfScope ps(h, "blas", h->n_dof * (r32 ? 52.0 : 48.0));
    const int nb = launch_cg_update(x, r, p, q, h->sc.p, h->n_dof, h->partial.p, r32, h->stream);
    launch_reduce(h->partial.p, nb, h->sc.p, SC_RR, h->stream, RED_NONE, h->h_sc);
}

// Whether CG launches the cycle's kernels one by one although graphs are on. A
// graph takes about 14 us of the stream until its first kernel, and its
// kernels follow each other 2 to 3 us apart instead of 4: it pays where many
// kernels are shorter than that (launches per colour, Jacobi steps on several
// small levels), not for the few of a cycle of one level or one that ends in
// the assembled map, nor for sweeps of a launch each. us per solve, graph / one
// by one:
//   Laplacian  4^3 GS-1-1 FP64   1249 /  683   elasticity 12^3 JA-1-1 FP64  6319 /  6019
//             12^3 JA-1-1 FP64   1933 / 1738              12^3 GS-1-1 MIXED 4542 /  4344
//             48^3 GS-1-1 MIXED 28489 / 28370             32^3 GS-1-1 MIXED 27317 / 27045
//   W-cycles: Laplacian 8^3 JA-1-1 MIXED 2266 / 2712, 16^3 FP64 3319 / 3410,
//             elasticity 12^3 GS-1-1 MIXED 23904 / 23850
//   a launch per colour: elasticity 8^3 GS-1-1 MIXED 5149 / 5595
// (Two graphs of the whole iteration, 0.96 to 1.05 of the time with a graph of
// the cycle, were slower than single launches everywhere.)
static bool cycle_launched(const amg_ctx *h) {
    const int last = static_cast<int>(h->lv.size()) - 1, top = h->dense_start >= 0 ? h->dense_start : last;
    if (h->prm.smoother == AMG_SMOOTH_GS) {
        for (int l = 0; l < top; ++l)
            if (!one_launch_sweeps(h, h->lv[l], h->mixed)) return false;
        return true;
    }
    return top <= 1 || (h->dense_start >= 0 && h->prm.nu == 1);
}

// One iteration in two halves. cg_step: up to the stopping test's scalars;
// cg_cycle and cg_next_direction: the next direction, which may go ahead of
// that test (it leaves x and r alone).
static void cg_step(amg_ctx *h, bool fcg, double *x) {
    double *r = h->kr.p, *p = h->kp.p, *q = h->kq.p;
    spmv_dot(h, p, q, fcg ? RED_FCG_ALPHA : RED_CG_ALPHA);
    cg_update(h, x, r, p, q);
}
static void cg_cycle(amg_ctx *h, bool launched) {
    if (cg_f32(h))
        launched ? cycle_f32_eager(h) : cycle_f32(h);
    else
        launched ? precondition_eager(h, h->kr.p, h->kz.p) : precondition_impl(h, h->kr.p, h->kz.p);
}
template <typename T>
static void cg_direction_from(amg_ctx *h, bool fcg, bool first, const T *z) {
    double *r = h->kr.p, *p = h->kp.p, *q = h->kq.p;
    // PCG: p = z + (<r, z> / <r, z>_prev) p; FCG: p = z - (<z, q> / <p, q>) p
    if (!fcg)
        dot_into(h, z, r, first ? SC_RZ : SC_TMP, first ? RED_NONE : RED_CG_BETA);
    else if (!first)
        dot_into(h, z, q, SC_TMP, RED_FCG_BETA);
    ProfScope ps(h, "blas", h->n_dof * (16.0 + sizeof(T) + (fcg ? 8.0 : 0.0)));
    const int nb = launch_cg_direction(p, z, h->sc.p, first, h->n_dof, fcg ? r : nullptr, h->partial.p, h->stream);
    if (fcg) launch_reduce(h->partial.p, nb, h->sc.p, SC_PR, h->stream);
}
static void cg_next_direction(amg_ctx *h, bool fcg, bool first = false) {
    if (cg_f32(h))
        cg_direction_from(h, fcg, first, h->cg_z);
    else
        cg_direction_from(h, fcg, first, static_cast<const double *>(h->kz.p));
}

double true_relres(amg_ctx *h, const double *b, const double *x, double r0norm) {
    residual(h, 0, b, x, h->kw.p);
    dot_into(h, h->kw.p, h->kw.p, SC_TMP);
    const double rr = read_scalar(h, SC_TMP);
    return r0norm > 0.0 ? std::sqrt(rr) / r0norm : 0.0;
}

static int finish(amg_ctx *h, const double *b, const double *x, double r0, int it, int status,
                  std::chrono::steady_clock::time_point t0, amg_result *res) {
    const double rel = true_relres(h, b, x, r0);
    if (status == AMG_OK && !(rel == rel)) status = AMG_DIVERGED;
    if (res) {
        res->iters = it;
        res->status = status;
        res->relres = rel;
        res->solve_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
    }
    profile_collect(h);
    return status;
}

// classify the recursive residual: converged, diverged, or continue (-1)
static int check(double rr, double rr0, double tol) {
    if (!(rr == rr) || std::isinf(rr)) return AMG_DIVERGED;
    const double rel = std::sqrt(rr / rr0);
    if (rel > 1e3) return AMG_DIVERGED;
    if (rel <= tol) return AMG_OK;
    return -1;
}

static int solve_cg(amg_ctx *h, bool fcg, const double *b, double *x, double tol, int maxit, amg_result *res) {
    const auto t0 = std::chrono::steady_clock::now();
    const int64_t n = h->n_dof;
    double *r = h->kr.p;
    residual(h, 0, b, x, r);
    dot_into(h, r, r, SC_RR);
    const double rr0 = read_scalar(h, SC_RR);
    const double r0 = std::sqrt(rr0);
    if (rr0 == 0.0) return finish(h, b, x, r0, 0, AMG_OK, t0, res);
    if (!(rr0 == rr0)) return finish(h, b, x, r0, 0, AMG_DIVERGED, t0, res);
    if (maxit <= 0) return finish(h, b, x, r0, 0, AMG_NOT_CONVERGED, t0, res);
    const bool launched = cycle_launched(h);
    if (cg_f32(h)) launch_to_f32(r, h->lv[0].mp.b.p, n, h->stream);
    cg_cycle(h, launched);
    cg_next_direction(h, fcg, true);
    int it = 0, status = AMG_NOT_CONVERGED;
    double rel = 1.0;
    while (it < maxit) {
        cg_step(h, fcg, x);
        ++it;
        scalars_begin(h);
        const bool ahead = it < maxit && rel > KRYLOV_AHEAD * tol;
        auto go = [&] {
            cg_cycle(h, launched);
            cg_next_direction(h, fcg);
        };
        if (ahead) go();
        scalars_wait(h);
        const double rr = h->h_sc[SC_RR];
        if (!(h->h_sc[SC_PQ] > 0.0)) { status = AMG_BREAKDOWN; break; }
        const int c = check(rr, rr0, tol);
        if (c >= 0) { status = c; break; }
        rel = std::sqrt(rr / rr0);
        if (!ahead && it < maxit) go();
    }
    return finish(h, b, x, r0, it, status, t0, res);
}

int solve_pcg(amg_ctx *h, const double *b, double *x, double tol, int maxit, amg_result *res) {
    return solve_cg(h, false, b, x, tol, maxit, res);
}

int solve_fcg(amg_ctx *h, const double *b, double *x, double tol, int maxit, amg_result *res) {
    return solve_cg(h, true, b, x, tol, maxit, res);
}

// Stand-alone AMG: repeated Algorithm 1 from the current iterate.
int solve_stationary(amg_ctx *h, const double *b, double *x, double tol, int maxit, amg_result *res) {
    const auto t0 = std::chrono::steady_clock::now();
    double *r = h->kr.p;
    residual(h, 0, b, x, r);
    dot_into(h, r, r, SC_RR);
    const double rr0 = read_scalar(h, SC_RR);
    const double r0 = std::sqrt(rr0);
    if (rr0 == 0.0) return finish(h, b, x, r0, 0, AMG_OK, t0, res);
    int it = 0, status = AMG_NOT_CONVERGED;
    const int cyc = std::max(1, h->prm.cycles);
    while (it < maxit) {
        for (int k = 0; k < cyc; ++k) cycle(h, 0, b, x, false, false);
        residual(h, 0, b, x, r);
        dot_into(h, r, r, SC_RR);
        ++it;
        const int c = check(read_scalar(h, SC_RR), rr0, tol);
        if (c >= 0) { status = c; break; }
    }
    return finish(h, b, x, r0, it, status, t0, res);
}

}  // namespace amgp2
