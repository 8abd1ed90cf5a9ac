"""Performance cases: what a program has this library do, each call with the
sizes, smoothers, precisions and systems of the model problems it is made for
(vector Laplacian, elasticity, mixed elasticity, batches of Stokes cavities).

A case is a dict of plain values: the `call` (solve, multi, batch, precondition
or setup), the `problem`, its mesh size `n` and the solver's options. Systems
are assembled here on the GPU, on cube meshes whose inner vertices are moved a
little, so that no coupling vanishes by symmetry. The element integrals are
multiples of a power of two, so their sums are exact whatever the order. A
system's operator goes with (problem, n) and is made once; right-hand sides
(and the material of a `setup` case) go with the seed.
"""
import functools
import random

import numpy as np
import torch

import paper_1503_01287_amd as amg
from paper_1503_01287_amd.problems import LinearSystem, cube_mesh

TOL = 1e-8
DEV = "cuda"

# edges of a tetrahedron that carry the quadratic basis functions
EDGES = ((0, 1), (1, 2), (2, 3), (0, 2), (0, 3), (1, 3))


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # the smallest system in use: latency and the number of launches
        dict(name="laplace-4 PCG", call="solve", problem="laplace", n=4, smoother="GS-1-1", krylov="PCG", precision="FP64"),
        # a small odd mesh with W-cycles and two smoothing steps
        dict(name="elasticity-9 W PCG", call="solve", problem="elasticity", n=9, smoother="GS-2-2", krylov="PCG", precision="FP64", nu=2),
        # a mid-size odd mesh in FP64 throughout
        dict(name="elasticity-21 PCG", call="solve", problem="elasticity", n=21, smoother="GS-1-1", krylov="PCG", precision="FP64"),
        # the benchmark's elasticity system, reduced-precision cycle
        dict(name="elasticity-32 mixed FCG", call="solve", problem="elasticity", n=32, smoother="GS-1-1", krylov="FCG", precision="MIXED"),
        # the benchmark's Laplacian, the largest single system
        dict(name="laplace-48 mixed FCG", call="solve", problem="laplace", n=48, smoother="JA-1-1-0.5", krylov="FCG", precision="MIXED"),
        # several data sets of one system at once
        dict(name="laplace-32 x8 mixed", call="multi", problem="laplace", n=32, smoother="JA-1-1-0.5", krylov="FCG", precision="MIXED", rhs=8),
        # the benchmark's saddle point system, segregated smoother
        dict(name="mixed-elasticity-24 sGS", call="solve", problem="mixed", n=24, smoother="sGS-1-1", krylov="FGMRES", precision="MIXED"),
        # the strongest saddle smoother, FP64
        dict(name="mixed-elasticity-12 Vanka", call="solve", problem="mixed", n=12, smoother="Vanka-1-1", krylov="FGMRES", precision="FP64"),
        # a batch of cavities of unlike sizes, merged
        dict(name="cavities x16 BS", call="batch", problem="cavity", n=16, n_min=8, count=16, smoother="BS-1-1", krylov="FGMRES", precision="FP32"),
        # many small elastic bodies at once
        dict(name="elasticity x24 PCG", call="batch", problem="elasticity", n=10, n_min=4, count=24, smoother="GS-1-1", krylov="PCG", precision="FP64"),
        # a caller with a Krylov loop of its own: one FP64 V-cycle
        dict(name="elasticity-24 V-cycle", call="precondition", problem="elasticity", n=24, smoother="GS-1-1", krylov="PCG", precision="FP64"),
        # one system, one solve: the whole setup counts
        dict(name="elasticity-16 setup", call="setup", problem="elasticity", n=16, smoother="GS-1-1", krylov="FCG", precision="MIXED"),
    ]


def draw(rng: random.Random):
    def size(a, b):
        return min(b, int(round(a * (b / a) ** rng.random())))

    kind = rng.choice(("solve", "solve", "saddle", "saddle", "multi", "batch", "precondition", "setup"))
    if kind == "saddle":
        smoother = rng.choice(("sGS-1-1", "sGS-1-1", "BS-1-1", "Vanka-1-1"))
        precision = "FP64" if smoother.startswith("Vanka") else rng.choice(("MIXED", "FP64"))
        return dict(call="solve", problem="mixed", n=size(4, 12 if smoother.startswith("Vanka") else 20),
                    smoother=smoother, krylov="FGMRES", precision=precision)
    if kind == "batch":
        if rng.random() < 0.5:
            hi = rng.randint(6, 14)
            return dict(call="batch", problem="cavity", n=hi, n_min=rng.randint(4, hi - 1), count=rng.randint(3, 15),
                        smoother="BS-1-1", krylov="FGMRES", precision=rng.choice(("FP32", "FP64")))
        precision = rng.choice(("FP64", "MIXED"))
        hi = rng.randint(5, 12)
        return dict(call="batch", problem=rng.choice(("elasticity", "laplace")), n=hi, n_min=rng.randint(3, hi - 1),
                    count=rng.randint(3, 23), smoother="GS-1-1", krylov="PCG" if precision == "FP64" else "FCG",
                    precision=precision)
    problem = rng.choice(("elasticity", "laplace"))
    precision = rng.choice(("FP64", "MIXED", "MIXED", "FP32"))
    if kind == "precondition":
        precision = "FP64"
    top = {"multi": 28, "setup": 18}.get(kind, 30 if problem == "elasticity" else 40)
    case = dict(call=kind, problem=problem, n=size(4, top), smoother=rng.choice(("GS-1-1", "GS-1-1", "GS-2-2", "JA-1-1-0.5")),
                krylov="PCG" if precision == "FP64" else "FCG", precision=precision)
    if kind == "multi":
        case["rhs"] = rng.randint(2, 8)
    if kind == "solve" and rng.random() < 0.25:
        case["nu"] = 2
    return case


# ----------------------------------------------------------------- the systems
@functools.lru_cache(maxsize=None)
def _mesh(n: int, mirrored: bool):
    return cube_mesh(n, mirrored=mirrored)


def _basis(mesh, moved):
    """g[t, k, i] with grad phi_k = sum_i lambda_i g[t, k, i] / det on
    tetrahedron t, and the determinants, in units of the mesh width: exact,
    the places being multiples of 1/64."""
    X = torch.from_numpy(moved).to(DEV)[torch.from_numpy(mesh.tet).to(DEV)]
    J = X[:, 1:] - X[:, :1]
    a, b, c = J[:, 0], J[:, 1], J[:, 2]
    det = (a * torch.linalg.cross(b, c)).sum(1)
    G = torch.stack([torch.linalg.cross(b, c), torch.linalg.cross(c, a), torch.linalg.cross(a, b)], 1)
    G = torch.cat([-G.sum(1, keepdim=True), G], 1)
    g = torch.zeros(X.shape[0], 10, 4, 3, dtype=torch.float64, device=DEV)
    g[:, :4] = G[:, :, None]
    for e, (p, q) in enumerate(EDGES):
        g[:, 4 + e, p] = 4 * G[:, q]
        g[:, 4 + e, q] = 4 * G[:, p]
    return g, det


# the integrals of lambda_i lambda_j over a tetrahedron, times 120 / |det|
MASS = torch.ones(4, 4, dtype=torch.float64) + torch.eye(4, dtype=torch.float64)


def _pattern(rows, cols, nrows, ncols):
    key, where = torch.unique((rows[:, :, None] * ncols + cols[:, None, :]).reshape(-1), return_inverse=True)
    r = key // ncols
    rowptr = torch.searchsorted(r, torch.arange(nrows + 1, device=DEV))
    return r, key % ncols, rowptr, where


def _sum_entries(where, values, nnz):
    """Multiples of 2^-32, summed per entry: exact in any order."""
    return torch.stack([torch.zeros(nnz, dtype=torch.float64, device=DEV).index_add_(0, where, v) for v in values], 1)


def _host(t, dtype):
    return np.ascontiguousarray(t.cpu().numpy().astype(dtype, copy=False))


@functools.lru_cache(maxsize=None)
def _system(problem: str, n: int):
    """The system with a zero right-hand side, the free nodes, the nodes'
    places and, for a cavity, the right-hand side of a lid of speed 1."""
    mesh = _mesh(n, problem == "cavity")
    N, nv, h = mesh.nv + mesh.ne, mesh.nv, 1.0 / n
    T, V = torch.from_numpy(mesh.tnode).to(DEV), torch.from_numpy(mesh.tet).to(DEV)
    xyz = mesh.xyz
    pos = np.concatenate([xyz, 0.5 * (xyz[mesh.edge[:, 0]] + xyz[mesh.edge[:, 1]])])
    on = np.any((xyz == 0.0) | (xyz == 1.0), axis=1) if problem == "cavity" else xyz[:, 0] == 0.0
    fixed = np.concatenate([on, on[mesh.edge[:, 0]] & on[mesh.edge[:, 1]]])
    gpu_fixed = torch.from_numpy(fixed).to(DEV)

    moved = np.rint(xyz * n)
    inside = np.all((moved > 0) & (moved < n), axis=1)
    moved[inside] += np.random.default_rng([n, 11]).integers(-9, 10, (int(inside.sum()), 3)) / 64.0
    g, det = _basis(mesh, moved)
    mg = torch.einsum("ij,tkjc->tkic", MASS.to(DEV), g)
    rows, cols, rowptr, where = _pattern(T, T, N, N)
    nnz = rows.numel()

    def product(c, d):
        K = torch.matmul(g[..., c].contiguous(), mg[..., d].transpose(1, 2).contiguous()) / det.abs()[:, None, None]
        return torch.round(K * 2.0 ** 32).reshape(-1) / 2.0 ** 32

    off = (gpu_fixed[rows] | gpu_fixed[cols]) & (rows != cols)
    if problem == "laplace":
        full = _sum_entries(where, [product(0, 0) + product(1, 1) + product(2, 2)], nnz) * (h / 120.0)
    else:
        H = _sum_entries(where, (product(c, d) for c in range(3) for d in range(3)), nnz).view(nnz, 3, 3)
        # elasticity: E = 1, Poisson ratio 0.3; mixed: 0.49999; cavity: viscosity 0.5
        ratio = {"elasticity": 0.3, "mixed": 0.49999, "cavity": 0.0}[problem]
        mu, lam = 0.5 / (1.0 + ratio), ratio / ((1.0 + ratio) * (1.0 - 2.0 * ratio))
        lap = torch.diagonal(H, dim1=1, dim2=2).sum(1)
        full = mu * (lap[:, None, None] * torch.eye(3, dtype=torch.float64, device=DEV) + H.transpose(1, 2))
        if problem == "elasticity":
            full = full + lam * H
        full = (full * (h / 120.0)).reshape(nnz, 9)
        del H
    lid = np.zeros(0)
    if problem == "cavity":
        inner = np.all((pos[:, :2] > 0.0) & (pos[:, :2] < 1.0), axis=1) & (pos[:, 2] == 1.0)
        inner[nv:] = False  # the lid's velocity is carried by its inner vertices
        drive = torch.zeros(N, 3, dtype=torch.float64)
        drive[:, 0] = torch.from_numpy(inner.astype(np.float64))
        y = torch.zeros(N, 3, dtype=torch.float64)
        from_lid = torch.from_numpy(inner).to(DEV)[cols].nonzero()[:, 0].cpu()
        y.index_add_(0, rows.cpu()[from_lid], -full.cpu()[from_lid].view(-1, 3, 3)[:, :, 0])
        y[torch.from_numpy(fixed)] = 0.0
        lid = y.reshape(-1).numpy()
    full[off] = 0.0
    sysm = LinearSystem(problem, n, nv, mesh.ne, 0, 1 if problem == "laplace" else 3, _host(rowptr, np.int32),
                        _host(cols, np.int32), _host(full.reshape(-1), np.float64), np.zeros(3 * N), np.zeros((N, 3)))
    if problem in ("mixed", "cavity"):
        brow, bcol, bptr, bwhere = _pattern(V, T, nv, N)
        B = -_sum_entries(bwhere, ((mg[..., c] * det.sign()[:, None, None]).transpose(1, 2).reshape(-1) for c in range(3)), brow.numel()) * (h * h / 120.0)
        if problem == "cavity":
            from_lid = torch.from_numpy(inner).to(DEV)[bcol].nonzero()[:, 0].cpu()
            q = torch.zeros(nv, dtype=torch.float64).index_add_(0, brow.cpu()[from_lid], -B.cpu()[from_lid, 0])
            lid = np.concatenate([lid, q.numpy()])
            sysm.pressure_kernel = True
        B[gpu_fixed[bcol]] = 0.0
        sysm.n_pres, sysm.B_rowptr, sysm.B_col = nv, _host(bptr, np.int32), _host(bcol, np.int32)
        sysm.B_val = _host(B.reshape(-1), np.float64)
        sysm.rhs = np.zeros(3 * N + nv)
        if problem == "mixed":
            crow, ccol, cptr, cwhere = _pattern(V, V, nv, nv)
            C = _sum_entries(cwhere, [(MASS.to(DEV) * det.abs()[:, None, None]).reshape(-1)], crow.numel()) * (h ** 3 / 120.0 / lam)
            sysm.C_rowptr, sysm.C_col, sysm.C_val = _host(cptr, np.int32), _host(ccol, np.int32), _host(C.reshape(-1), np.float64)
    return sysm, ~fixed, pos, lid


def _rhs(problem: str, n: int, rng) -> np.ndarray:
    """A smooth body force (lumped), and a cavity's lid at a speed in [0.5, 2]."""
    sysm, free, pos, lid = _system(problem, n)
    f = np.zeros((free.size, 3))
    for c in range(3):
        for _ in range(3):
            k, phase = rng.integers(0, 3, 3), rng.uniform(0.0, 2.0 * np.pi, 3)
            f[:, c] += rng.normal() * np.prod(np.cos(np.pi * k * pos + phase), axis=1)
    f[: sysm.n_lin] *= 4.0
    f[~free] = 0.0
    b = np.concatenate([(f * (0.25 / n ** 3)).ravel(), np.zeros(sysm.n_pres)])
    return b + rng.uniform(0.5, 2.0) * lid if problem == "cavity" else b


def _sizes(case):
    rng = random.Random("%d %d %d" % (case["n_min"], case["n"], case["count"]))
    return [case["n"]] + [rng.randint(case["n_min"], case["n"]) for _ in range(case["count"] - 1)]


def _options(case):
    return dict(smoother=case["smoother"], krylov=case["krylov"], precision=case["precision"], nu=case.get("nu", 1))


def _material(case, seed):
    """A setup case's stiffness."""
    return float(np.random.default_rng([7, seed]).uniform(0.5, 2.0))


def _right_hand_sides(case, seed):
    rng = np.random.default_rng([3, seed])
    ns = _sizes(case) if case["call"] == "batch" else [case["n"]] * case.get("rhs", 1)
    return [_rhs(case["problem"], n, rng) for n in ns]


# -------------------------------------------------------------------- the calls
def prepare(case, seed):
    call, problem = case["call"], case["problem"]
    b = torch.from_numpy(np.concatenate(_right_hand_sides(case, seed))).to(DEV)
    st = dict(case=case, b=b, x=torch.zeros_like(b))
    if call == "batch":
        systems = [_system(problem, n)[0] for n in _sizes(case)]
        st["solver"] = amg.BatchedSolver(systems, **_options(case))
        if problem == "cavity":
            parts, at = [], 0
            for k, s in enumerate(systems):
                parts.append((at + 3 * s.nodes, s.n_pres, k))
                at += s.dofs
            st["p_at"] = torch.cat([torch.arange(a, a + m) for a, m, _ in parts]).to(DEV)
            st["p_of"] = torch.cat([torch.full((m,), k) for _, m, k in parts]).to(DEV)
            st["p_n"] = torch.tensor([float(m) for _, m, _ in parts], dtype=torch.float64, device=DEV)
    elif call == "setup":
        sysm = _system(problem, case["n"])[0]
        st["system"] = LinearSystem(**{**vars(sysm), "A_val": sysm.A_val * _material(case, seed)})
    else:
        st["solver"] = amg.AMGSolver(_system(problem, case["n"])[0], **_options(case))
        if call == "multi":
            st["b"], st["x"] = b.view(case["rhs"], -1), torch.zeros_like(b).view(case["rhs"], -1)
    return st


def run(st):
    case, b, x = st["case"], st["b"], st["x"]
    if case["call"] == "precondition":
        st["solver"].precondition(b, x)
        return x
    x.zero_()
    if case["call"] == "setup":
        solver = amg.AMGSolver(st["system"], **_options(case))
        r = solver.solve(b, x, tol=TOL)
        solver.close()
        return {"x": x, "iters": r.iters}
    if case["call"] == "solve":
        return {"x": x, "iters": st["solver"].solve(b, x, tol=TOL).iters}
    if case["call"] == "multi":
        return {"x": x, "iters": np.array([r.iters for r in st["solver"].solve_multi(b, x, tol=TOL)])}
    iters = np.array([r.iters for r in st["solver"].solve(b, x, tol=TOL)])
    if case["problem"] == "cavity":  # a cavity's pressure is known up to a constant: of mean zero
        p = x[st["p_at"]]
        mean = torch.zeros_like(st["p_n"]).index_add_(0, st["p_of"], p) / st["p_n"]
        x[st["p_at"]] = p - mean[st["p_of"]]
    return {"x": x, "iters": iters}


# ------------------------------------------------------------- what a pass needs
def work(case):
    """The operator's entries and the vectors, read once per use that the
    method cannot do without: one FP64 product per iteration and, in the
    cycle's precision, one pass before and one after the coarse correction
    (a smoothing step and the residual after it share a pass from a zero
    guess). Iterations are those that the method needs about."""
    saddle = case["problem"] in ("mixed", "cavity")
    blk = 1 if case["problem"] == "laplace" else 9
    entries = nodes = pres = 0
    for n in _sizes(case) if case["call"] == "batch" else [case["n"]]:
        nodes += (2 * n + 1) ** 3
        entries += 28 * (2 * n + 1) ** 3
        pres += (n + 1) ** 3 if saddle else 0
    k = case.get("rhs", 1)
    its = 60 if case["smoother"].startswith("sGS") else 35 if saddle else 25
    steps = 2 if "-2-2" in case["smoother"] else 1
    vb = {"FP64": 8, "MIXED": 4, "FP32": 4}[case["precision"]]
    vec = 8 * k * (3 * nodes + pres)
    outer = entries * (blk * 8 + 4) + pres * 65 * 28 * 2 + 4 * vec
    cycle = (2 * steps) * (entries * (blk * vb + 4) + pres * 65 * (3 * vb + 4) * 2 + 2 * vec * vb // 8)
    flops = 2 * (9 if blk == 9 else 3) * entries * k + 12 * 65 * pres
    if case["smoother"].startswith("Vanka"):
        its, cycle = 12, cycle + 2 * 8 * pres * 196 * 196
        flops += 4 * pres * 196 * 196
    if case["call"] == "precondition":
        return {"bytes": cycle, "flops": 2 * steps * flops}
    return {"bytes": its * (outer + cycle) + (entries * (blk * 8 + 4) if case["call"] == "setup" else 0),
            "flops": its * (1 + 2 * steps) * flops}


# --------------------------------------------------------- solutions in 64 bits
def _scalar_csr(sysm):
    """The velocity operator as a scalar sparse matrix."""
    ptr, col = torch.from_numpy(sysm.A_rowptr).long(), torch.from_numpy(sysm.A_col).long()
    val = torch.from_numpy(sysm.A_val).to(DEV)
    row = torch.repeat_interleave(torch.arange(sysm.nodes), ptr.diff()).to(DEV)
    col = col.to(DEV)
    m = sysm.nodes
    if sysm.bs == 3:
        c = torch.arange(3, device=DEV)
        row, col = (3 * row[:, None, None] + c[:, None]).expand(-1, 3, 3), (3 * col[:, None, None] + c).expand(-1, 3, 3)
        row, col, m = row.reshape(-1), col.reshape(-1), 3 * m
    diag = torch.zeros(m, dtype=torch.float64, device=DEV)
    at = row == col
    diag[row[at]] = val[at]
    return torch.sparse_coo_tensor(torch.stack([row, col]), val, (m, m)).coalesce().to_sparse_csr(), diag


def _cg(A, diag, b):
    """Columns of b solved by conjugate gradients with the diagonal, to 1e-13."""
    x, r = torch.zeros_like(b), b.clone()
    z = r / diag[:, None]
    p, rz = z.clone(), (r * z).sum(0)
    stop = 1e-13 * b.norm(dim=0)
    for k in range(6000):
        q = A @ p
        a = rz / (p * q).sum(0).clamp_min(1e-300)
        x += a * p
        r -= a * q
        if k % 20 == 0 and bool((r.norm(dim=0) <= stop).all()):
            break
        z = r / diag[:, None]
        new = (r * z).sum(0)
        p = z + (new / rz.clamp_min(1e-300)) * p
        rz = new
    return x


def exact(case, seed):
    """The solutions; a V-cycle's result and a large saddle point system's
    solution are left out."""
    if case["call"] == "precondition" or case["problem"] == "cavity":
        return None
    rhs = _right_hand_sides(case, seed)
    if case["problem"] == "mixed":
        s = _system("mixed", case["n"])[0]
        if s.dofs > 6000:
            return None
        K = torch.zeros(s.dofs, s.dofs, dtype=torch.float64, device=DEV)
        u = 3 * s.nodes
        A, _ = _scalar_csr(s)
        K[:u, :u] = A.to_dense()
        for ptr, col, val, w in ((s.B_rowptr, s.B_col, s.B_val, 3), (s.C_rowptr, s.C_col, s.C_val, 1)):
            row = torch.from_numpy(np.repeat(np.arange(s.n_pres), np.diff(ptr))).to(DEV)
            col = torch.from_numpy(col).long().to(DEV)
            val = torch.from_numpy(val).view(-1, w).to(DEV)
            for c in range(w):
                if w == 3:
                    K[u + row, 3 * col + c] = val[:, c]
                    K[3 * col + c, u + row] = val[:, c]
                else:
                    K[u + row, u + col] = -val[:, 0]
        return {"x": torch.linalg.solve(K, torch.from_numpy(rhs[0]).to(DEV)), "iters": None}
    ns = _sizes(case) if case["call"] == "batch" else [case["n"]]
    if case["call"] != "batch":
        rhs = [np.stack(rhs)]
    out = {}
    for at, n in enumerate(ns):
        if n not in out:
            out[n] = _scalar_csr(_system(case["problem"], n)[0])
        A, diag = out[n]
        b = torch.from_numpy(np.atleast_2d(rhs[at])).to(DEV)
        k = b.shape[0]
        if case["problem"] == "laplace":  # one scalar operator for the three components
            x = _cg(A, diag, b.view(k, -1, 3).permute(1, 0, 2).reshape(-1, 3 * k).contiguous())
            x = x.view(-1, k, 3).permute(1, 0, 2).reshape(k, -1)
        else:
            x = _cg(A, diag, b.t().contiguous()).t()
        rhs[at] = x.reshape(-1)
    x = torch.cat(rhs)
    if case["call"] == "setup":
        x = x / _material(case, seed)
    return {"x": x.view(case["rhs"], -1) if case["call"] == "multi" else x, "iters": None}
