"""Performance cases: what users of this framework have it do, from a few
thousand cells (where launches and latency count) to a few million (where HBM
bandwidth does).

Meshes are jittered tetrahedral unit cubes of 6 n^3 cells (each hex cut into
its 6 Kuhn tetrahedra), the kind the tests and the benchmark use; odd n give
ragged tiles and slices.  A user preprocesses a mesh once and keeps it, so a
mesh is kept here per size; states (device workspace, tables) and inputs are
made anew for every `prepare`.

Kinds of case:
  step      RK3 steps of the convection-diffusion equation, FP64 or FP32,
            launched directly (with or without a CFL evaluation before each)
            or replayed as a captured graph; zero-flux or mixed walls.
  poisson   one cold solve of Laplace(P) = f to `tol`: Jacobi-CG matrix-free
            or on the stored matrix, the FP32-refined form, or flexible CG
            with the multigrid W-cycle.
  streamer  coupled steps: Poisson solve, field, drift, ionisation, transport.
  batch     many uneven meshes in one state: every step an RK3 step of each
            mesh at its own CFL bound, then each mesh's warm-started solve.
"""
import math
from collections import OrderedDict
from types import SimpleNamespace

import numpy as np
import torch

from paper_2203_00925_amd import binding as B

D_SCALAR = 1e-3
CFL = 0.4
TAGS = 6                                   # walls x0, x1, y0, y1, z0, z1
ZERO, NEU, DIR = B.ZERO_FLUX, B.NEUMANN, B.DIRICHLET
# wall kinds and values: the benchmark's closed box, and one of every kind
WALLS = {"closed": ([ZERO] * 6, [0.0] * 6),
         "mixed": ([DIR, NEU, ZERO, ZERO, NEU, DIR], [0.5, 0.0, 0.0, 0.0, 0.1, 0.25])}
# the potential: grounded on every wall, or between two electrodes
POTENTIAL = {"grounded": ([DIR] * 6, [0.0] * 6),
             "electrodes": ([DIR, DIR, NEU, NEU, NEU, NEU], [1.0, 0.0, 0.0, 0.0, 0.0, 0.0])}
STREAMER = dict(mobility=1.0, charge_scale=40.0, alpha_a=2.0, alpha_b=0.3, cfl=CFL, tol=1e-12)
BATCH_TOL = 1e-10


def listed():
    return [
        # one step at a time with its own CFL bound on the smallest mesh of
        # real use: all launches and latency
        dict(name="step_3k_cfl", kind="step", n=8, prec="fp64", walls="mixed", steps=1, how="cfl"),
        # the paper-sized small configuration: ten captured steps, 48,000 cells
        dict(name="step_48k_graph", kind="step", n=20, prec="fp64", walls="closed", steps=10, how="graph"),
        # an odd-sized middle mesh, walls of every kind, direct launches
        dict(name="step_304k", kind="step", n=37, prec="fp64", walls="mixed", steps=4, how="direct"),
        # the benchmark's step beyond the last-level cache: 3.07M cells
        dict(name="step_3m_graph", kind="step", n=80, prec="fp64", walls="closed", steps=2, how="graph"),
        # the reduced-precision form of the step, 1.57M cells
        dict(name="step32_1m6_graph", kind="step", n=64, prec="fp32", walls="closed", steps=3, how="graph"),
        # small matrix-free solve: 48,000 cells, a chain of small kernels
        dict(name="solve_48k", kind="poisson", n=20, method="plain", matrix_free=True, pot="grounded", tol=1e-10),
        # the benchmark's solve at one eighth of its mesh: 1.3M cells
        dict(name="solve_1m3", kind="poisson", n=60, method="plain", matrix_free=True, pot="grounded", tol=1e-10),
        # the assembled system, as the paper's solvers take it (odd size)
        dict(name="solve_stored_179k", kind="poisson", n=31, method="plain", matrix_free=False, pot="electrodes",
             tol=1e-11),
        # FP32 inner iterations inside FP64 refinement
        dict(name="solve_refined_619k", kind="poisson", n=47, method="refined", matrix_free=True, pot="grounded",
             tol=1e-10),
        # the fastest solver: flexible CG around the multigrid W-cycle
        dict(name="solve_multigrid_750k", kind="poisson", n=50, method="multigrid", matrix_free=True,
             pot="grounded", tol=1e-10),
        # two coupled streamer steps, 83k cells, from a cold potential
        dict(name="streamer_83k", kind="streamer", n=24, steps=2),
        # eight uneven meshes (about 0.5M cells), two steps and solves each
        dict(name="batch_8_meshes", kind="batch", count=8, n_lo=12, n_hi=29, steps=2, mesh_seed=4),
    ]


def draw(rng):
    def size(lo, hi):                      # spread over the logarithm of the cell count
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    pick = rng.random()
    if pick < 0.45:
        prec = rng.choice(["fp64", "fp64", "fp32"])
        n = size(8, 80)
        how = rng.choice(["cfl", "direct", "graph"])
        return dict(kind="step", n=n, prec=prec, walls=rng.choice(["closed", "mixed"]),
                    steps=1 if how == "cfl" else rng.randint(1, 10 if n <= 40 else 3), how=how)
    if pick < 0.80:
        method, free, hi = rng.choice([("plain", True, 60), ("plain", True, 60), ("plain", False, 36),
                                       ("refined", True, 55), ("multigrid", True, 52)])
        # between electrodes the right-hand side is large beside the potential:
        # the tighter tolerance keeps the same accuracy of P
        pot, tol = rng.choice([("grounded", 1e-10), ("electrodes", 1e-11)])
        return dict(kind="poisson", n=size(9, hi), method=method, matrix_free=free, pot=pot, tol=tol)
    if pick < 0.90:
        return dict(kind="streamer", n=size(8, 30), steps=rng.randint(1, 3))
    return dict(kind="batch", count=rng.randint(3, 10), n_lo=size(8, 14), n_hi=size(16, 29), steps=rng.randint(1, 2),
                mesh_seed=rng.randint(1, 10 ** 6))


# ---- meshes ---------------------------------------------------------------------

def cube(n, seed):
    """Vertices, tetrahedra and tagged boundary triangles of a jittered cube."""
    n1 = n + 1
    g = np.arange(n)
    corner = np.stack([a.ravel() for a in np.meshgrid(g, g, g, indexing="ij")][::-1], axis=1)
    eye = np.eye(3, dtype=np.int64)
    perms = [(0, 1, 2), (0, 2, 1), (1, 0, 2), (1, 2, 0), (2, 0, 1), (2, 1, 0)]
    offs = np.stack([np.stack([np.zeros(3, np.int64), eye[p[0]], eye[p[0]] + eye[p[1]], np.ones(3, np.int64)])
                     for p in perms])
    lat = (corner[:, None, None, :] + offs[None]).reshape(-1, 4, 3)
    tets = (lat[..., 0] + n1 * (lat[..., 1] + n1 * lat[..., 2])).astype(np.int32)
    g1 = np.arange(n1)
    ijk = np.stack([a.ravel() for a in np.meshgrid(g1, g1, g1, indexing="ij")][::-1], axis=1)
    jit = np.random.default_rng(seed).uniform(-0.2 / n, 0.2 / n, ijk.shape)
    jit[(ijk == 0) | (ijk == n)] = 0.0     # the domain stays the unit cube
    tris, tags = [], []
    for f in ([1, 2, 3], [0, 2, 3], [0, 1, 3], [0, 1, 2]):
        for axis in range(3):
            for side, at in ((0, 0), (1, n)):
                hit = (lat[:, f, axis] == at).all(axis=1)
                tris.append(tets[hit][:, f])
                tags.append(np.full(int(hit.sum()), 2 * axis + side, np.int32))
    return SimpleNamespace(xyz=ijk / n + jit, tets=tets, btris=np.concatenate(tris), btags=np.concatenate(tags),
                           nv=len(ijk), nc=len(tets))


_kept = OrderedDict()                      # the last few meshes: what a program keeps for its runs
_KEEP = 16


def kept(key, make):
    if key not in _kept:
        _kept[key] = make()
        while len(_kept) > _KEEP:
            _kept.popitem(last=False)
    _kept.move_to_end(key)
    return _kept[key]


def cell_points(c):
    return torch.from_numpy(c.xyz).cuda()[torch.from_numpy(c.tets).cuda().long()].mean(dim=1)


def mesh_of(n, stored):
    def make():
        c = cube(n, 2)
        return SimpleNamespace(raw=c, mesh=B.Mesh.from_cube(c, no_matrix=not stored), pts=cell_points(c))
    return kept((n, stored), make)


def batch_sizes(case):
    r = np.random.default_rng(case["mesh_seed"])
    lo, hi = math.log(case["n_lo"]), math.log(case["n_hi"])
    return [int(round(math.exp(x))) for x in r.uniform(lo, hi, case["count"])]


def batch_of(case):
    def make():
        raws = [cube(n, 1000 + k) for k, n in enumerate(batch_sizes(case))]
        return SimpleNamespace(raws=raws, mesh=B.Mesh.from_batch(raws, no_matrix=True),
                               pts=[cell_points(c) for c in raws])
    return kept(("batch", case["count"], case["n_lo"], case["n_hi"], case["mesh_seed"]), make)


# ---- inputs -----------------------------------------------------------------------

def pulse(pts, rng):
    """A Gaussian pulse, its centre and width from the seed."""
    centre = torch.tensor(rng.uniform(0.35, 0.65, 3), dtype=torch.float64, device=pts.device)
    sigma = float(rng.uniform(0.1, 0.2))
    return torch.exp(-((pts - centre) ** 2).sum(1) / sigma ** 2)


def velocity(pts, rng):
    """The rotating field (sin pi y, sin pi z, sin pi x), scaled per axis."""
    a = rng.uniform(0.7, 1.3, 3)
    s = torch.sin(math.pi * pts)
    return torch.stack([a[0] * s[:, 1], a[1] * s[:, 2], a[2] * s[:, 0]])


def inputs(case, seed):
    rng = np.random.default_rng(seed)
    if case["kind"] == "batch":
        pts = batch_of(case).pts
        u = torch.cat([pulse(p, rng) for p in pts])
        return dict(u=u, vel=torch.cat([velocity(p, rng) for p in pts], dim=1),
                    D=[float(x) for x in rng.uniform(1e-4, 1e-2, len(pts))])
    pts = mesh_of(case["n"], needs_matrix(case)).pts
    if case["kind"] == "step":
        return dict(u=pulse(pts, rng), vel=velocity(pts, rng))
    if case["kind"] == "poisson":
        return dict(f=pulse(pts, rng))
    ne = pulse(pts, rng) + 1e-2
    return dict(ne=ne, ion=ne * (1.0 + 0.02 * torch.sin(2 * math.pi * pts[:, 1])))


def needs_matrix(case):
    """The stored pattern: the assembled solve, and the multigrid setup."""
    return case["kind"] == "poisson" and (not case["matrix_free"] or case["method"] == "multigrid")


# ---- the passes -------------------------------------------------------------------

def prepare(case, seed):
    x = inputs(case, seed)
    s = SimpleNamespace(case=case, **x)
    kind = case["kind"]
    if kind == "batch":
        s.state = st = B.State(batch_of(case).mesh)
        st.set_mesh_diffusivity(x["D"])
        st.set_bcs(B.VAR_SCALAR, [ZERO] * TAGS)
        st.set_bcs(B.VAR_POTENTIAL, [DIR] * TAGS)
        st.set_field(B.FIELD_VEL, x["vel"].ravel())
        st.cfl_dt(CFL)
        s.zero = torch.zeros_like(x["u"])
        # one launch per kernel for all meshes: the schedule the tuner picks at these sizes
        s.batch = B.Batch(st, policy=B.BQ_LAUNCHES)
        return s
    m = mesh_of(case["n"], needs_matrix(case))
    st = s.state = B.State(m.mesh, diffusivity=D_SCALAR,
                           precision=B.FP32 if case.get("prec") == "fp32" else B.FP64)
    if kind == "step":
        st.set_bcs(B.VAR_SCALAR, *WALLS[case["walls"]])
        st.set_field(B.FIELD_VEL, x["vel"].ravel())
        st.set_field(B.FIELD_U, x["u"])
        s.dt = st.cfl_dt(CFL)
        s.dtype = torch.float32 if case["prec"] == "fp32" else torch.float64
    elif kind == "poisson":
        st.set_bcs(B.VAR_POTENTIAL, *POTENTIAL[case["pot"]])
        s.zero = torch.zeros_like(x["f"])
        if needs_matrix(case):
            st.poisson_assemble()
        s.opts = dict(tol=case["tol"], matrix_free=case["matrix_free"])
        if case["method"] == "refined":
            s.opts.update(method=B.SOLVE_IR_FP32)
        elif case["method"] == "multigrid":
            st.amg_build(theta=0.4, omega=0.8, cycle=B.CYCLE_W)
            s.opts.update(method=B.SOLVE_AMG, graph=1, chunk=8)
    else:
        st.set_bcs(B.VAR_SCALAR, [NEU] * TAGS)
        st.set_bcs(B.VAR_POTENTIAL, *POTENTIAL["electrodes"])
        s.zero = torch.zeros_like(x["ne"])
    return s


def run(s):
    case, st = s.case, s.state
    kind = case["kind"]
    if kind == "step":
        if case["how"] == "cfl":
            for _ in range(case["steps"]):
                st.step(1, st.cfl_dt(CFL))
        elif case["how"] == "graph":
            st.step_graph(case["steps"], s.dt)
        else:
            st.step(case["steps"], s.dt)
        return st.get_field(B.FIELD_U, dtype=s.dtype)
    if kind == "poisson":
        st.set_field(B.FIELD_P, s.zero)
        st.poisson_solve(s.f, **s.opts)
        return st.get_field(B.FIELD_P)
    if kind == "streamer":
        st.set_field(B.FIELD_U, s.ne)
        st.set_field(B.FIELD_ION, s.ion)
        st.set_field(B.FIELD_P, s.zero)
        st.streamer_step(case["steps"], matrix_free=True, **STREAMER)
        return {"ne": st.get_field(B.FIELD_U), "ion": st.get_field(B.FIELD_ION), "P": st.get_field(B.FIELD_P),
                "E": st.get_field(B.FIELD_EFIELD)}
    st.set_field(B.FIELD_U, s.u)
    st.set_field(B.FIELD_P, s.zero)
    s.batch.run(case["steps"], tol=BATCH_TOL)
    return {"u": st.get_field(B.FIELD_U), "P": st.get_field(B.FIELD_P)}


# ---- what a pass cannot do without --------------------------------------------------

def step_work(nc, prec):
    """One RK3 step: three stages, each over the geometry and fields once.
    Per cell: the least-squares inverse (6), 2 faces' coefficients (3),
    velocity flux and centroid (3), volume, centre (3), u^n, u, source and the
    new u as reals; vertex ids (4), 2 faces' cells and vertices (5) and the
    shared-edge neighbours (13.8) as 32-bit ids.  Operations: gradient sums
    over ~70 neighbours (9 each), limiter, vertex values, fluxes."""
    b = 4 if prec == "fp32" else 8
    per_cell = b * (6 + 2 * 7 + 8) + 4 * (4 + 2 * 5 + 13.8)
    return 3 * nc * per_cell, 3 * nc * 900.0


def iteration_work(nc, b=8):
    """One Jacobi-CG iteration with the matrix-free product: vertex lists (4
    ids and weights), 4 vertex and 4 face weights, 8 ids, and the vectors x,
    r, p, q and D^-1 with x, r, p, q written."""
    return nc * (4 * (4 + b) + 8 * b + 8 * 4 + 9 * b), nc * 45.0


def stored_work(nc):
    """One Jacobi-CG iteration on the stored matrix: 70 values and 16-bit
    local columns per row, and the vectors."""
    return nc * (70 * 10 + 72), nc * 160.0


def work(case):
    kind = case["kind"]
    if kind == "step":
        nc = 6 * case["n"] ** 3
        b, f = step_work(nc, case["prec"])
        return {"bytes": case["steps"] * b, "flops": case["steps"] * f}
    if kind == "poisson":
        n, nc = case["n"], 6 * case["n"] ** 3
        if case["method"] == "multigrid":          # about 50 cycles, two products each and one outside
            b, f = iteration_work(nc)
            return {"bytes": 50 * 3 * b, "flops": 50 * 3 * f}
        b, f = (iteration_work(nc, 4 if case["method"] == "refined" else 8) if case["matrix_free"]
                else stored_work(nc))
        return {"bytes": 16 * n * b, "flops": 16 * n * f}      # about 16 n iterations from zero
    if kind == "streamer":
        n, nc = case["n"], 6 * case["n"] ** 3
        b, f = iteration_work(nc)
        bs, fs = step_work(nc, "fp64")
        return {"bytes": 16 * n * b + case["steps"] * bs, "flops": 16 * n * f + case["steps"] * fs}
    total = {"bytes": 0.0, "flops": 0.0}
    for n in batch_sizes(case):
        nc = 6 * n ** 3
        b, f = iteration_work(nc)
        bs, fs = step_work(nc, "fp64")
        total["bytes"] += 16 * n * b + case["steps"] * bs
        total["flops"] += 16 * n * f + case["steps"] * fs
    return total


# ---- the same results in 64 bits, in plain torch --------------------------------------

def dot(a, b):
    return (a * b).sum(-1)


class Reference:
    """The discretisation on one mesh: least-squares gradients over every
    cell and ghost sharing a vertex, Barth-Jespersen limiting over the face
    neighbours, upwind MUSCL fluxes, diamond diffusion with least-squares
    vertex values, mirrored ghosts."""

    def __init__(self, raw):
        dev = "cuda"
        x = torch.from_numpy(raw.xyz).to(dev)
        t = torch.from_numpy(raw.tets).to(dev).long()
        nc, nv = len(t), len(x)
        p = x[t]
        self.nc, self.nv = nc, nv
        self.vol = dot(p[:, 1] - p[:, 0], torch.linalg.cross(p[:, 2] - p[:, 0], p[:, 3] - p[:, 0])).abs() / 6
        centre = p.mean(1)
        # faces: sorted vertex triples; the first cell (lower number) is L
        tri = torch.sort(t[:, [[1, 2, 3], [0, 2, 3], [0, 1, 3], [0, 1, 2]]].reshape(-1, 3), dim=1).values
        key = (tri[:, 0] * nv + tri[:, 1]) * nv + tri[:, 2]
        uniq, inv, cnt = torch.unique(key, return_inverse=True, return_counts=True)
        nf = len(uniq)
        owner = torch.arange(nc, device=dev).repeat_interleave(4)
        order = torch.argsort(inv, stable=True)
        first = torch.cumsum(cnt, 0) - cnt
        L = owner[order][first]
        inner = cnt == 2
        bf = torch.nonzero(~inner)[:, 0]
        nb = len(bf)
        R = torch.empty(nf, dtype=torch.long, device=dev)
        R[inner] = owner[order][first[inner] + 1]
        R[bf] = nc + torch.arange(nb, device=dev)
        abc = tri[order][first]
        A, Bv, C = x[abc[:, 0]], x[abc[:, 1]], x[abc[:, 2]]
        self.fx = (A + Bv + C) / 3
        S = torch.linalg.cross(Bv - A, C - A) / 2
        flip = dot(S, self.fx - centre[L]) < 0
        S = torch.where(flip[:, None], -S, S)
        abc = torch.where(flip[:, None], abc[:, [0, 2, 1]], abc)
        A, Bv, C = x[abc[:, 0]], x[abc[:, 1]], x[abc[:, 2]]
        self.S, self.area, self.abc, self.L, self.R, self.inner = S, S.norm(dim=1), abc, L, R, inner
        self.cf = inv.reshape(nc, 4)
        self.sign = torch.where(L[self.cf] == torch.arange(nc, device=dev)[:, None], 1.0, -1.0).double()
        # ghosts: mirrored centres, tags of their triangles
        nrm = S[bf] / self.area[bf][:, None]
        xg = centre[L[bf]] + 2 * dot(self.fx[bf] - centre[L[bf]], nrm)[:, None] * nrm
        self.xc = torch.cat([centre, xg])
        self.gowner, self.gdist, self.bf = L[bf], (xg - centre[L[bf]]).norm(dim=1), bf
        bt = torch.sort(torch.from_numpy(raw.btris).to(dev).long(), dim=1).values
        at = torch.searchsorted(uniq, (bt[:, 0] * nv + bt[:, 1]) * nv + bt[:, 2])
        tag = torch.zeros(nf, dtype=torch.long, device=dev)
        tag[at] = torch.from_numpy(raw.btags).to(dev).long()
        self.gtag = tag[bf]
        # diamond coefficients of S . grad: kAC (uA - uC) + kBC (uB - uC) + kRL (uR - uL)
        c = self.xc[R] - self.xc[L]
        mu3 = dot(S, c)
        self.kAC = dot(torch.linalg.cross(Bv - C, c), S) / (2 * mu3)
        self.kBC = dot(torch.linalg.cross(c, A - C), S) / (2 * mu3)
        self.kRL = dot(S, S) / mu3
        # vertex -> cells and ghosts, least-squares weights of the vertex value
        ne = nc + nb
        vk = torch.cat([t.reshape(-1), abc[bf].reshape(-1)]) * ne
        vk += torch.cat([owner, (nc + torch.arange(nb, device=dev)).repeat_interleave(3)])
        vk = torch.sort(vk).values
        self.v, self.e = vk // ne, vk % ne
        a = torch.cat([torch.ones(len(vk), 1, dtype=torch.float64, device=dev), self.xc[self.e] - x[self.v]], dim=1)
        M = torch.zeros(nv, 16, dtype=torch.float64, device=dev)
        M.index_add_(0, self.v, (a[:, :, None] * a[:, None, :]).reshape(-1, 16))
        rhs = torch.zeros(nv, 4, 1, dtype=torch.float64, device=dev)
        rhs[:, 0] = 1
        self.alpha = dot(a, torch.linalg.solve(M.reshape(nv, 4, 4), rhs)[:, :, 0][self.v])
        self.t, self.vk_ptr = t, torch.searchsorted(self.v.contiguous(), torch.arange(nv + 1, device=dev))
        self.stencil = None

    def make_stencil(self):
        """Pairs (cell, entity sharing a vertex), M^-1 of the gradient."""
        nc, ne = self.nc, len(self.xc)
        deg = self.vk_ptr[1:] - self.vk_ptr[:-1]
        keys = []
        for k in range(4):                              # one vertex slot at a time bounds the scratch
            v = self.t[:, k]
            n = deg[v]
            row = torch.arange(nc, device=v.device).repeat_interleave(n)
            start = torch.cumsum(n, 0) - n
            pos = torch.arange(len(row), device=v.device) - start[row] + self.vk_ptr[v][row]
            keys.append(row * ne + self.e[pos])
        key = torch.unique(torch.cat(keys))
        row, col = key // ne, key % ne
        off = col != row
        self.row, self.col = row[off], col[off]
        d = self.xc[self.col] - self.xc[self.row]
        M = torch.zeros(nc, 9, dtype=torch.float64, device=d.device)
        M.index_add_(0, self.row, (d[:, :, None] * d[:, None, :]).reshape(-1, 9))
        self.Minv, self.stencil = torch.linalg.inv(M.reshape(nc, 3, 3)), True

    def walls(self, kinds, vals):
        k = torch.tensor(kinds, device=self.gtag.device)[self.gtag]
        v = torch.tensor(vals, dtype=torch.float64, device=self.gtag.device)[self.gtag]
        gs = torch.where(k == DIR, -1.0, 1.0).double()
        gt = torch.where(k == DIR, 2 * v, torch.where(k == NEU, v * self.gdist, torch.zeros_like(v)))
        fk = torch.full((len(self.L),), DIR, device=k.device)
        fk[self.bf] = k
        fv = torch.zeros(len(self.L), dtype=torch.float64, device=k.device)
        fv[self.bf] = v
        return SimpleNamespace(gs=gs, gt=gt, kind=fk, val=fv)

    def extend(self, u, w):
        return torch.cat([u, w.gs * u[self.gowner] + w.gt])

    def gradient(self, ue):
        if not self.stencil:
            self.make_stencil()
        J = torch.zeros(self.nc, 3, dtype=torch.float64, device=ue.device)
        J.index_add_(0, self.row, (self.xc[self.col] - self.xc[self.row]) * (ue[self.col] - ue[self.row])[:, None])
        return (self.Minv * J[:, None, :]).sum(-1)

    def vertices(self, ue):
        return torch.zeros(self.nv, dtype=torch.float64, device=ue.device).index_add_(0, self.v, self.alpha * ue[self.e])

    def diffusion(self, ue, w):
        un = self.vertices(ue)[self.abc]
        f = self.kAC * (un[:, 0] - un[:, 2]) + self.kBC * (un[:, 1] - un[:, 2]) + self.kRL * (ue[self.R] - ue[self.L])
        return torch.where(w.kind == NEU, w.val * self.area, torch.where(w.kind == ZERO, torch.zeros_like(f), f))

    def phi(self, vel):
        R = torch.where(self.inner, self.R, self.L)
        return dot((vel[self.L] + vel[R]) / 2, self.S)

    def residual(self, u, phi, D, w, src=None):
        ue = self.extend(u, w)
        g = self.gradient(ue)
        nbr = torch.where(self.sign > 0, self.R[self.cf], self.L[self.cf])
        un = ue[nbr]
        hi, lo = torch.maximum(u, un.amax(1)) - u, torch.minimum(u, un.amin(1)) - u
        delta = (g[:, None, :] * (self.fx[self.cf] - self.xc[:self.nc, None, :])).sum(-1)
        one = torch.ones_like(delta)
        lim = torch.where(delta > 0, torch.minimum(one, hi[:, None] / delta),
                          torch.where(delta < 0, torch.minimum(one, lo[:, None] / delta), one))
        psi = lim.amin(1)
        up = torch.where(phi >= 0, self.L, self.R)
        cell = up < self.nc
        uc = torch.where(cell, up, self.L)
        face = ue[up] + torch.where(cell, psi[uc] * dot(g[uc], self.fx - self.xc[uc]), torch.zeros_like(phi))
        F = torch.where(w.kind == ZERO, torch.zeros_like(phi), face * phi - D * self.diffusion(ue, w))
        res = -(self.sign * F[self.cf]).sum(1) / self.vol
        return res if src is None else res + src

    def cfl(self, phi, D, w):
        rate = torch.where(w.kind == ZERO, torch.zeros_like(phi), phi.abs() + D * self.kRL)
        return CFL * float((self.vol / rate[self.cf].sum(1)).min())

    def step(self, u, dt, phi, D, w, src=None):
        uk = u
        for a in (0.5, 0.5, 1.0):
            uk = u + a * dt * self.residual(uk, phi, D, w, src)
        return uk

    def solve(self, f, w, x, tol=1e-13, maxit=6000):
        """K x = b with K x = -(linear part of the summed face fluxes), by
        Jacobi-preconditioned BiCGSTAB from x."""
        h = SimpleNamespace(gs=w.gs, gt=torch.zeros_like(w.gt), kind=w.kind, val=torch.zeros_like(w.val))

        def flux_sum(v, wall):
            return (self.sign * self.diffusion(self.extend(v, wall), wall)[self.cf]).sum(1)

        b = -self.vol * f + flux_sum(torch.zeros_like(f), w)
        # the diagonal's two-point part is a good enough scaling
        krl = torch.where((w.kind == DIR), self.kRL, torch.zeros_like(self.kRL)) * torch.where(self.inner, 1.0, 2.0)
        dinv = 1 / krl[self.cf].sum(1)
        bn = float(b.norm())
        for _ in range(4):                              # reopened from the true residual
            r = b + flux_sum(x, h)
            if float(r.norm()) <= tol * bn:
                break
            r0, p, v = r.clone(), torch.zeros_like(r), torch.zeros_like(r)
            rho = alpha = omega = torch.ones((), dtype=torch.float64, device=f.device)
            for it in range(maxit):
                rho1 = r0 @ r
                p = r + (rho1 / rho) * (alpha / omega) * (p - omega * v)
                ph = dinv * p
                v = -flux_sum(ph, h)
                alpha, rho = rho1 / (r0 @ v), rho1
                s = r - alpha * v
                sh = dinv * s
                t = -flux_sum(sh, h)
                omega = (t @ s) / (t @ t)
                x = x + alpha * ph + omega * sh
                r = s - omega * t
                if it % 10 == 9 and not float(r.norm()) > tol * bn:
                    break
        return x


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        return exact_batch(case, seed)
    x = inputs(case, seed)
    ref = Reference(mesh_of(case["n"], needs_matrix(case)).raw)
    if kind == "poisson":
        w = ref.walls(*POTENTIAL[case["pot"]])
        return ref.solve(x["f"], w, torch.zeros_like(x["f"]))
    if kind == "step":
        w = ref.walls(*WALLS[case["walls"]])
        phi = ref.phi(x["vel"].T)
        dt, u = ref.cfl(phi, D_SCALAR, w), x["u"]
        for _ in range(case["steps"]):
            u = ref.step(u, dt, phi, D_SCALAR, w)
        return u
    w, wp = ref.walls([NEU] * TAGS, [0.0] * TAGS), ref.walls(*POTENTIAL["electrodes"])
    ne, ion, P = x["ne"], x["ion"], torch.zeros_like(x["ne"])
    for _ in range(case["steps"]):
        P = ref.solve(STREAMER["charge_scale"] * (ne - ion), wp, P)
        E = -ref.gradient(ref.extend(P, wp))
        v = -STREAMER["mobility"] * E
        src = STREAMER["alpha_a"] * torch.exp(-STREAMER["alpha_b"] / E.norm(dim=1)) * v.norm(dim=1) * ne
        phi = ref.phi(v)
        dt = ref.cfl(phi, D_SCALAR, w)
        ne = ref.step(ne, dt, phi, D_SCALAR, w, src)
        ion = ion + dt * src
    return {"ne": ne, "ion": ion, "P": P, "E": E.T.reshape(-1)}


def exact_batch(case, seed):
    x = inputs(case, seed)
    us, ps, at = [], [], 0
    for raw, D in zip(batch_of(case).raws, x["D"]):
        ref = Reference(raw)
        u, vel = x["u"][at:at + raw.nc], x["vel"][:, at:at + raw.nc]
        at += raw.nc
        w, wp = ref.walls([ZERO] * TAGS, [0.0] * TAGS), ref.walls([DIR] * TAGS, [0.0] * TAGS)
        phi = ref.phi(vel.T)
        dt, P = ref.cfl(phi, D, w), torch.zeros_like(u)
        for _ in range(case["steps"]):
            u = ref.step(u, dt, phi, D, w)
        us.append(u)
        ps.append(ref.solve(u, wp, P))
    return {"u": torch.cat(us), "P": torch.cat(ps)}
