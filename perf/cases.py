"""What this library's speed is measured on: solves, batches and the single
operations of the spectral-element Poisson solver, each through the Python
binding's public calls.

A case is one call (or, for "setup", the three calls that prepare a solve) on
a box of deformed hexahedra whose vertices and right-hand side are drawn from
the seed.  Meshes come in rows, as a structured generator numbers them, or
shuffled (elements in random order, every local frame rotated), as an
unstructured one does.  CG cases run a fixed number of iterations: long
enough that the iteration and not the set-up is what counts, short enough
that FP32 rounding does not yet separate two correct runs.  Mixed-precision
cases run to a true residual of 1e-10.
"""
from __future__ import annotations

import itertools
import math

import numpy as np
import torch

import paper_2108_12188_amd as sem

PREC = {"fp32": sem.FP32, "fp64": sem.FP64, "mixed": sem.MIXED}
GEOM = {"pre": sem.PRECOMPUTED, "otf": sem.ON_THE_FLY}
TOL_MIXED = 1e-10


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------
def _cg(name, nx, ny, nz, N, prec, geom, iters, precond="none", numbering="rows"):
    return {"name": name, "call": "cg", "nx": nx, "ny": ny, "nz": nz, "N": N, "prec": prec,
            "geom": geom, "iters": iters, "precond": precond, "numbering": numbering}


def listed():
    return [
        # the smallest solve in use (FP64, 64 elements): one iteration is a
        # handful of dependent launches, so latency is everything
        _cg("cg_fp64_4cube_N7", 4, 4, 4, 7, "fp64", "pre", 64),
        # a small FP32 solve with no round size: launches still dominate
        _cg("cg_fp32_7x6x5_N7", 7, 6, 5, 7, "fp32", "otf", 40),
        # an ordinary FP32 solve whose vectors fit the cache
        _cg("cg_fp32_16cube_N7", 16, 16, 16, 7, "fp32", "otf", 50),
        # the largest: the benchmark's own mesh, a tenth of its iterations
        _cg("cg_fp32_32cube_N7", 32, 32, 32, 7, "fp32", "otf", 50),
        # precomputed factors on an unstructured numbering
        _cg("cg_fp32_pre_24x23x25_N5", 24, 23, 25, 5, "fp32", "pre", 50, numbering="shuffled"),
        # FP64 with the factors recomputed
        _cg("cg_fp64_20cube_N7", 20, 20, 20, 7, "fp64", "otf", 30),
        # Jacobi-preconditioned, an even order (the per-point gather table)
        _cg("pcg_fp32_13x12x14_N8", 13, 12, 14, 8, "fp32", "otf", 50, precond="jacobi"),
        # a whole mixed-precision solve to 1e-10
        {"name": "mixed_10x11x9_N9", "call": "mixed", "nx": 10, "ny": 11, "nz": 9, "N": 9,
         "geom": "otf", "numbering": "rows"},
        # many small problems solved together, orders and sizes mixed
        {"name": "batch_10_mixed", "call": "batch", "count": 10, "lo": 64, "hi": 1000,
         "geom": "otf", "mix": 4},
        # the local operator alone (a user's own Krylov loop or smoother)
        {"name": "ax_fp32_otf_21x20x19_N9", "call": "ax", "nx": 21, "ny": 20, "nz": 19, "N": 9,
         "prec": "fp32", "geom": "otf", "numbering": "rows"},
        # the gather-scatter alone, with its mask
        {"name": "gs_fp64_24x23x22_N7", "call": "gs", "nx": 24, "ny": 23, "nz": 22, "N": 7,
         "prec": "fp64", "numbering": "rows"},
        # what precedes a solve: coordinates, right-hand side, diagonal
        {"name": "setup_16x17x15_N7", "call": "setup", "nx": 16, "ny": 17, "nz": 15, "N": 7,
         "prec": "fp32", "numbering": "rows"},
    ]


# local points up to which each kind of call is drawn; the smallest meshes
# have a few dozen elements
_MOST = {("cg", "fp32"): 1 << 23, ("cg", "fp64"): 1 << 22, "mixed": 1 << 20, "ax": 1 << 23,
         "gs": 1 << 23, "setup": 1 << 22}


def _box(rng, N, most):
    """A near-cubic box of the order, its points log-uniform up to `most`."""
    P3 = (N + 1) ** 3
    lo, hi = math.log(27.0), math.log(most / P3)
    side = math.exp(rng.uniform(lo, hi) / 3.0)
    n = [max(1, round(side * rng.uniform(0.9, 1.1))) for _ in range(3)]
    while n[0] * n[1] * n[2] * P3 > most:
        n[n.index(max(n))] -= 1
    return n


def draw(rng):
    call = rng.choice(["cg", "cg", "cg", "cg", "cg", "cg", "mixed", "batch", "ax", "ax", "gs",
                       "setup"])
    # the orders of the batched and served workloads most, all built ones some
    N = rng.choice([5, 7, 7, 9, rng.randint(3, 11)])
    geom = rng.choice(["otf", "otf", "pre"])
    if call == "batch":
        case = {"call": "batch", "count": rng.randint(4, 12), "lo": 64, "hi": rng.randint(200, 1000),
                "geom": geom, "mix": rng.randrange(1 << 20)}
        while work(case)["bytes"] > 9e10:                    # no more than the listed batch
            case["count"] -= 1
        return case
    prec = rng.choice(["fp32", "fp32", "fp64"])
    nx, ny, nz = _box(rng, N, _MOST.get(call) or _MOST[(call, prec)])
    case = {"call": call, "nx": nx, "ny": ny, "nz": nz, "N": N,
            "numbering": rng.choice(["rows", "rows", "shuffled"])}
    if call != "mixed":
        case["prec"] = prec
    if call in ("cg", "mixed", "ax"):
        case["geom"] = geom
    if call == "cg":
        # on a small mesh FP32 rounding separates the iterates sooner
        case["iters"] = min(rng.randint(30, 60), max(12, int(0.8 * max(nx, ny, nz) * N)))
        case["precond"] = rng.choice(["none", "none", "none", "jacobi"])
    return case


# ---------------------------------------------------------------------------
# inputs (host): meshes, right-hand sides
# ---------------------------------------------------------------------------
def _rotations():
    """The 24 proper rotations of the cube as (axis permutation, signs)."""
    out = []
    for perm in itertools.permutations(range(3)):
        parity = sum(perm[a] > perm[b] for a in range(3) for b in range(a + 1, 3)) % 2
        for signs in itertools.product((1, -1), repeat=3):
            if signs[0] * signs[1] * signs[2] == (-1 if parity else 1):
                out.append((perm, signs))
    return out


def _rotated_index(P, perm, signs):
    """Local index before the rotation of every local point after it."""
    t = np.arange(P)
    new = np.meshgrid(t, t, t, indexing="ij")[::-1]          # i, j, k of point i + P (j + P k)
    old = [new[perm[d]] if signs[d] > 0 else P - 1 - new[perm[d]] for d in range(3)]
    return (old[0] + P * (old[1] + P * old[2])).ravel()


def _mesh(nx, ny, nz, N, numbering, graded, seed):
    """(vertices [E][8][3], global ids [E][P^3], Dirichlet flags [E][P^3], global points)."""
    rng = np.random.Generator(np.random.PCG64(seed))
    P = N + 1
    axes = [np.linspace(0.0, 1.0, n + 1) for n in (nx, ny, nz)]
    grid = np.stack(np.meshgrid(axes[2], axes[1], axes[0], indexing="ij")[::-1], axis=-1)
    h = np.array([1.0 / nx, 1.0 / ny, 1.0 / nz])
    inner = (slice(1, -1),) * 3
    grid[inner] += rng.uniform(-0.1, 0.1, grid[inner].shape) * h
    if graded:                                               # thin elements next to z = 0
        z = grid[..., 2]
        grid[..., 2] = (z + 3.0 * z ** 3) / 4.0
    grid = grid.astype(np.float32).astype(np.float64)
    ez, ey, ex = (a.ravel() for a in np.meshgrid(np.arange(nz), np.arange(ny), np.arange(nx),
                                                 indexing="ij"))
    vert = np.stack([grid[ez + c, ey + b, ex + a] for c in (0, 1) for b in (0, 1)
                     for a in (0, 1)], axis=1)
    t = np.arange(P)
    kk, jj, ii = (a.ravel() for a in np.meshgrid(t, t, t, indexing="ij"))
    gx, gy, gz = nx * N + 1, ny * N + 1, nz * N + 1
    first = (ex * N + gx * (ey * N + gy * (ez * N))).astype(np.int64)
    gid = first[:, None] + (ii + gx * (jj + gy * kk))[None, :]
    onb = np.zeros((gz, gy, gx), dtype=np.uint8)
    for d in range(3):
        edge = [slice(None)] * 3
        for side in (0, -1):
            edge[d] = side
            onb[tuple(edge)] = 1
    dirichlet = onb.ravel()[gid]
    if numbering == "shuffled":
        turn = rng.integers(0, 24, size=vert.shape[0])
        for r, (perm, signs) in enumerate(_rotations()):
            sel = np.nonzero(turn == r)[0]
            vert[sel] = vert[sel][:, _rotated_index(2, perm, signs)]
            gid[sel] = gid[sel][:, _rotated_index(P, perm, signs)]
            dirichlet[sel] = dirichlet[sel][:, _rotated_index(P, perm, signs)]
        order = rng.permutation(vert.shape[0])
        vert, gid, dirichlet = vert[order], gid[order], dirichlet[order]
    return vert, gid, dirichlet, gx * gy * gz


def _case_mesh(case, seed):
    return _mesh(case["nx"], case["ny"], case["nz"], case["N"], case["numbering"],
                 case.get("precond") == "jacobi", seed)


def _random_global(n_glob, seed):
    """One value U[-1, 1] per global point, representable in FP32."""
    rng = np.random.Generator(np.random.PCG64(seed + 12188))
    return torch.from_numpy(rng.uniform(-1.0, 1.0, n_glob).astype(np.float32))


def _source(xyz, seed):
    """A smooth forcing, a few sine modes of random weight, at points xyz [3][n]."""
    rng = np.random.Generator(np.random.PCG64(seed + 30000))
    f = torch.zeros_like(xyz[0])
    for _ in range(3):
        kx, ky, kz = (float(v) for v in rng.integers(1, 4, 3))
        amp = float(rng.uniform(0.5, 1.5)) * math.pi ** 2 * (kx * kx + ky * ky + kz * kz)
        f += amp * torch.sin(kx * math.pi * xyz[0]) * torch.sin(ky * math.pi * xyz[1]) \
            * torch.sin(kz * math.pi * xyz[2])
    return f.contiguous()


def _batch_boxes(case):
    """(nx, ny, nz, N) of a batch's problems: element counts log-uniform, orders 5, 7 and 9."""
    rng = np.random.Generator(np.random.PCG64(case["mix"]))
    out = []
    for _ in range(case["count"]):
        e = math.exp(rng.uniform(math.log(case["lo"]), math.log(case["hi"])))
        n = max(1, round(e ** (1.0 / 3.0)))
        out.append((n, n, max(1, round(e / (n * n))), int(rng.choice([5, 7, 9]))))
    return out


def _local(glob, gid, dirichlet, dtype):
    """Masked local copies on the device of one value per global point."""
    ids = torch.from_numpy(gid).cuda().view(-1)
    v = glob.cuda()[ids]
    v[torch.from_numpy(dirichlet).cuda().view(-1) != 0] = 0
    return v.to(dtype)


# ---------------------------------------------------------------------------
# prepare, run
# ---------------------------------------------------------------------------
def _handle(mesh, N, prec, geom):
    vert, gid, dirichlet, _ = mesh
    pre = geom == "pre"
    return sem.Mesh(vert, gid, dirichlet, N, g_fp32=pre and prec != "fp64",
                    g_fp64=pre and prec == "fp64")


def prepare(case, seed):
    call = case["call"]
    if call == "batch":
        meshes, bs = [], []
        for q, (nx, ny, nz, N) in enumerate(_batch_boxes(case)):
            m = _handle(_mesh(nx, ny, nz, N, "rows", False, seed + 7919 * q), N, "mixed",
                        case["geom"])
            bs.append(m.rhs(_source(m.coords(), seed + 7919 * q)))
            meshes.append(m)
        return {"case": case, "batch": sem.Batch(meshes), "bs": bs}
    mesh = _case_mesh(case, seed)
    vert, gid, dirichlet, n_glob = mesh
    prec = case.get("prec", "mixed")
    m = _handle(mesh, case["N"], prec, case.get("geom", "otf"))
    st = {"case": case, "mesh": m}
    dtype = torch.float32 if prec == "fp32" else torch.float64
    if call == "cg":
        st["b"] = _local(_random_global(n_glob, seed), gid, dirichlet, dtype)
    elif call == "mixed":
        st["b"] = m.rhs(_source(m.coords(), seed))
    elif call == "ax":
        st["u"] = _local(_random_global(n_glob, seed), gid, dirichlet, dtype)
        st["w"] = torch.empty_like(st["u"])
    elif call == "gs":
        # values of one element each, as the local operator leaves them
        st["u"] = torch.from_numpy(np.random.Generator(np.random.PCG64(seed)).uniform(
            -1.0, 1.0, m.n).astype(np.float32)).cuda().to(dtype)
        st["w"] = torch.empty_like(st["u"])
    else:
        st["f"] = _source(m.coords(), seed)
    return st


def run(state):
    case = state["case"]
    call = case["call"]
    if call == "cg":
        x, info = state["mesh"].cg_solve(
            state["b"], prec=PREC[case["prec"]], geom=GEOM[case["geom"]],
            fixed_iters=case["iters"],
            precond=sem.PRECOND_JACOBI if case["precond"] == "jacobi" else sem.PRECOND_NONE)
        return {"x": x, "iters": info["iters"]}
    if call == "mixed":
        x, info = state["mesh"].cg_solve(state["b"], prec=sem.MIXED, geom=GEOM[case["geom"]],
                                         tol=TOL_MIXED)
        return {"x": x, "converged": info["converged"]}
    if call == "batch":
        xs, infos = state["batch"].solve(state["bs"], prec=sem.MIXED, geom=GEOM[case["geom"]],
                                         tol=TOL_MIXED)
        return {"x": xs, "converged": [i["converged"] for i in infos]}
    m = state["mesh"]
    if call == "ax":
        return m.ax(state["u"], state["w"], geom=GEOM[case["geom"]])
    if call == "gs":
        # in place, so the values are put there first (a device copy)
        return m.gs(state["w"].copy_(state["u"]))
    return {"xyz": m.coords(), "b": m.rhs(state["f"], prec=PREC[case["prec"]]), "diag": m.diag()}


# ---------------------------------------------------------------------------
# work
# ---------------------------------------------------------------------------
def _points(nx, ny, nz, N):
    return nx * ny * nz * (N + 1) ** 3


def _iteration(n, N, size, geom, jacobi):
    """(bytes, flops) of one CG iteration: r, p, x and w each read and
    written (r once more for the next direction), the factors if they are
    stored, M^-1 and z with the preconditioner."""
    words = 9 + (6 if geom == "pre" else 0) + (3 if jacobi else 0)
    return n * words * size, n * (12 * (N + 1) + 15 + 12 + (60 if geom == "otf" else 0))


def _inner_iterations(nx, ny, nz, N):
    """About what a mixed solve to 1e-10 takes on these meshes."""
    return 1.2 * max(nx, ny, nz) * N * N


def work(case):
    call = case["call"]
    if call in ("batch", "mixed"):
        boxes = _batch_boxes(case) if call == "batch" else [(case["nx"], case["ny"], case["nz"],
                                                             case["N"])]
        b = f = 0.0
        for box in boxes:
            ib, fl = _iteration(_points(*box), box[3], 4, case["geom"], False)
            b += ib * _inner_iterations(*box)
            f += fl * _inner_iterations(*box)
        return {"bytes": b, "flops": f}
    N = case["N"]
    n = _points(case["nx"], case["ny"], case["nz"], N)
    size = 4 if case["prec"] == "fp32" else 8
    if call == "cg":
        b, f = _iteration(n, N, size, case["geom"], case["precond"] == "jacobi")
        return {"bytes": b * case["iters"], "flops": f * case["iters"]}
    if call == "ax":
        pre = case["geom"] == "pre"
        return {"bytes": n * size * (8 if pre else 2),
                "flops": n * (12 * (N + 1) + 15 + (0 if pre else 60))}
    if call == "gs":
        # the copy in, then every value read and written once
        return {"bytes": n * size * 4, "flops": n}
    # coordinates out; source in, right-hand side out; diagonal out
    return {"bytes": n * (24 + 8 + size + 8), "flops": n * (24 + 4 + 6 * (N + 1) + 90)}


# ---------------------------------------------------------------------------
# exact: the same results in 64 bits, in plain torch on one value per global
# point (Algorithm 1 does not depend on the copies)
# ---------------------------------------------------------------------------
def _gll(N):
    """Gauss-Lobatto-Legendre points, weights and the derivative matrix."""
    leg = np.polynomial.legendre.Legendre.basis(N)
    xi = np.concatenate([[-1.0], np.sort(leg.deriv().roots().real), [1.0]])
    for _ in range(3):                                      # polish the interior points
        xi[1:-1] -= leg.deriv()(xi[1:-1]) / leg.deriv(2)(xi[1:-1])
    w = 2.0 / (N * (N + 1) * leg(xi) ** 2)
    D = np.zeros((N + 1, N + 1))
    for i in range(N + 1):
        for j in range(N + 1):
            if i != j:
                D[i, j] = leg(xi[i]) / leg(xi[j]) / (xi[i] - xi[j])
    D[0, 0], D[N, N] = -N * (N + 1) / 4.0, N * (N + 1) / 4.0
    return xi, w, D


class _Exact:
    """The discrete Poisson operator of a mesh in FP64 torch."""

    def __init__(self, mesh, N):
        vert, gid, dirichlet, self.n_glob = mesh
        dev = "cuda" if torch.cuda.is_available() else "cpu"
        xi, w, D = _gll(N)
        self.P, self.E, self.dev = N + 1, vert.shape[0], dev
        self.gid = torch.from_numpy(gid).to(dev).view(-1)
        self.free = torch.ones(self.n_glob, dtype=torch.float64, device=dev)
        self.free[self.gid[torch.from_numpy(dirichlet).to(dev).view(-1) != 0]] = 0.0
        self.D = torch.from_numpy(D).to(dev)
        self.Dt = self.D.t().contiguous()
        x1 = torch.from_numpy(xi).to(dev)
        wt = torch.from_numpy(w).to(dev)
        v = torch.from_numpy(vert).to(dev)
        x, y, z = x1.view(1, 1, 1, -1), x1.view(1, 1, -1, 1), x1.view(1, -1, 1, 1)
        f = [((1 - x) / 2, (1 + x) / 2), ((1 - y) / 2, (1 + y) / 2), ((1 - z) / 2, (1 + z) / 2)]
        s = (-0.5, 0.5)
        shape = (self.E, self.P, self.P, self.P)
        self.xyz, J = [], []
        for d in range(3):
            q = [0.0, 0.0, 0.0, 0.0]
            for c, b, a in itertools.product((0, 1), repeat=3):
                vd = v[:, a + 2 * b + 4 * c, d].view(-1, 1, 1, 1)
                q[0] = q[0] + vd * f[0][a] * f[1][b] * f[2][c]
                q[1] = q[1] + vd * s[a] * f[1][b] * f[2][c]
                q[2] = q[2] + vd * f[0][a] * s[b] * f[2][c]
                q[3] = q[3] + vd * f[0][a] * f[1][b] * s[c]
            q = [t.expand(shape) for t in q]
            self.xyz.append(q[0].reshape(-1))
            J.append(q[1:])
        col = [[J[d][a] for d in range(3)] for a in range(3)]     # x_xi, x_eta, x_gamma

        def cross(a, b):
            return [a[1] * b[2] - a[2] * b[1], a[2] * b[0] - a[0] * b[2], a[0] * b[1] - a[1] * b[0]]

        def dot(a, b):
            return a[0] * b[0] + a[1] * b[1] + a[2] * b[2]
        r = [cross(col[1], col[2]), cross(col[2], col[0]), cross(col[0], col[1])]
        det = dot(col[0], r[0])
        wq = wt.view(1, 1, 1, -1) * wt.view(1, 1, -1, 1) * wt.view(1, -1, 1, 1)
        self.mass = (wq * det).reshape(-1)
        self.G = {(a, b): (wq / det * dot(r[a], r[b])).contiguous()
                  for a in range(3) for b in range(a, 3)}

    def diff(self, u, d, M):
        """M applied along direction d (0: i, the fastest) of u [E][P][P][P]."""
        P = self.P
        if d == 0:
            return (u.reshape(-1, P) @ M.t()).view(u.shape)
        t = u.transpose(3, 3 - d).contiguous()
        return (t.view(-1, P) @ M.t()).view(t.shape).transpose(3, 3 - d).contiguous()

    def ax(self, u):
        """The local operator on a local vector."""
        u = u.view(self.E, self.P, self.P, self.P)
        g = [self.diff(u, d, self.D) for d in range(3)]
        out = 0.0
        for a in range(3):
            v = sum(self.G[(min(a, b), max(a, b))] * g[b] for b in range(3))
            out = out + self.diff(v, a, self.Dt)
        return out.reshape(-1)

    def assemble(self, w):
        g = torch.zeros(self.n_glob, dtype=torch.float64, device=self.dev)
        return g.index_add_(0, self.gid, w)

    def apply(self, ug):
        return self.assemble(self.ax(ug[self.gid])) * self.free

    def diag_local(self):
        D2 = (self.D ** 2).t().contiguous()
        s = sum(self.diff(self.G[(a, a)], a, D2) for a in range(3))
        dd = torch.diagonal(self.D)
        pos = [dd.view(1, 1, 1, -1), dd.view(1, 1, -1, 1), dd.view(1, -1, 1, 1)]
        for a, b in ((0, 1), (0, 2), (1, 2)):
            s = s + 2.0 * pos[a] * pos[b] * self.G[(a, b)]
        return s.reshape(-1)

    def cg(self, b, iters, minv=None, tol=0.0):
        x = torch.zeros_like(b)
        r = b.clone()
        z = r if minv is None else minv * r
        p = z.clone()
        rz = torch.dot(r, z)
        stop = float(torch.dot(r, r)) * tol * tol
        for it in range(iters):
            w = self.apply(p)
            alpha = rz / torch.dot(p, w)
            x += alpha * p
            r -= alpha * w
            z = r if minv is None else minv * r
            new = torch.dot(r, z)
            p = z + (new / rz) * p
            rz = new
            if tol and it % 16 == 15 and float(torch.dot(r, r)) <= stop:
                break
        return x

    def solve(self, b, most):
        """A x = b as far as FP64 CG goes: one solve and one correction."""
        x = self.cg(b, most, tol=1e-12)
        return x + self.cg(b - self.apply(x), most, tol=1e-3)

    def rhs(self, f):
        return self.assemble(self.mass * f) * self.free


def _exact_solve(mesh, box, seed):
    e = _Exact(mesh, box[3])
    f = _source(torch.stack(e.xyz), seed)
    return e.solve(e.rhs(f), int(3 * _inner_iterations(*box)) + 100)[e.gid]


def exact(case, seed):
    call = case["call"]
    if call == "batch":
        xs = [_exact_solve(_mesh(*box, "rows", False, seed + 7919 * q), box, seed + 7919 * q)
              for q, box in enumerate(_batch_boxes(case))]
        return {"x": xs, "converged": [None] * len(xs)}
    mesh = _case_mesh(case, seed)
    box = (case["nx"], case["ny"], case["nz"], case["N"])
    if call == "mixed":
        return {"x": _exact_solve(mesh, box, seed), "converged": None}
    e = _Exact(mesh, case["N"])
    if call in ("cg", "ax"):
        u = _random_global(mesh[3], seed).to(e.dev).double() * e.free
        if call == "ax":
            return e.ax(u[e.gid])
        minv = None
        if case["precond"] == "jacobi":
            minv = e.free / e.assemble(e.diag_local())
        return {"x": e.cg(u, case["iters"], minv)[e.gid], "iters": None}
    if call == "gs":
        u = torch.from_numpy(np.random.Generator(np.random.PCG64(seed)).uniform(
            -1.0, 1.0, e.gid.numel()).astype(np.float32)).to(e.dev).double()
        return (e.assemble(u) * e.free)[e.gid]
    xyz = torch.stack(e.xyz)
    return {"xyz": xyz, "b": e.rhs(_source(xyz, seed))[e.gid], "diag": e.assemble(e.diag_local())[e.gid]}
