"""The kernels that a rule on sizes chooses between, at the sizes on both
sides of each rule: the CG iteration against a host CG on the general
matrix-free product, the multigrid cycle on grids of many slices against the
oracle's, and the step that replays its stages against direct launches."""
import numpy as np
import pytest
import scipy.sparse as sp

import synth
from conftest import cube
from oracle import amg, poisson
from oracle.geometry import DIRICHLET, NEUMANN, ZERO_FLUX, build_geometry

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
B = pytest.importorskip("paper_2203_00925_amd.binding")
from mapping import Mapped  # noqa: E402

KINDS = [DIRICHLET, NEUMANN, ZERO_FLUX, DIRICHLET, NEUMANN, ZERO_FLUX]


@pytest.fixture(scope="module", autouse=True)
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)


def dev(a):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


def joined(sizes):
    """Two cubes that share the corner vertex (1, 1, 1): the arrays of two meshes."""
    a, b = (cube(n, 1000 + n) for n in sizes)
    at = int(np.argmin(np.abs(a.xyz - 1.0).sum(1)))
    own = int(np.argmin(np.abs(b.xyz).sum(1)))
    ids = np.arange(b.nv) + a.nv - (np.arange(b.nv) > own)
    ids[own] = at
    xyz = np.concatenate([a.xyz, np.delete(b.xyz + 1.0, own, axis=0)])
    return (xyz, np.concatenate([a.tets, ids[b.tets]]).astype(np.int32),
            np.concatenate([a.btris, ids[b.btris]]).astype(np.int32), np.concatenate([a.btags, b.btags]))


def meshes(sizes, shared=False):
    if shared:
        return B.Mesh(*joined(sizes), mesh_cell_start=np.cumsum([0] + [6 * n ** 3 for n in sizes]))
    if len(sizes) == 1:
        return B.Mesh.from_cube(cube(sizes[0], 1000 + sizes[0]))
    return B.Mesh.from_batch([cube(n, 1000 + n) for n in sizes])


def host_cg(apply, b, dinv, off, its):
    """x after `its` Jacobi-CG iterations from zero, the scalars per mesh."""
    sums = lambda v: np.repeat(np.add.reduceat(v, off[:-1]), np.diff(off))
    x, r = np.zeros_like(b), b.copy()
    z = dinv * r
    p, rz = z.copy(), sums(r * z)
    for _ in range(its):
        q = apply(p)
        a = rz / sums(p * q)
        x, r = x + a * p, r - a * q
        z = dinv * r
        new = sums(r * z)
        p, rz = z + new / rz * p, new
    return x


# cells: 6 n^3.  One mesh: 384 (the last tile half full), 118,098 and 131,712
# (below and above the product by tiles, its last tile half full), 279,936 (two
# rows a thread of the vector kernels).  Meshes: ends inside blocks; 262,656
# cells, two rows a thread; meshes with a common vertex (the six-kernel form).
CG = {"n4": ((4,), False), "n27": ((27,), False), "n28": ((28,), False), "n36": ((36,), False),
      "batch": ((4, 5, 6), False), "batch_wide": ((28, 24, 20), False), "shared_vertex": ((4, 5), True)}


@pytest.mark.parametrize("matrix_free", [True, False])
@pytest.mark.parametrize("case", list(CG))
def test_cg_iterates_equal_host_cg(case, matrix_free):
    """x after 12 iterations, from direct launches and from replayed chunks.
    An iteration's sums of about 30 terms a row round to 30 x 2.2e-16 of
    their largest; 12 iterations, each amplifying an earlier one's error by at
    most about ten: 1e-12 of the largest x.  The preconditioner is read off the
    first iterate (x_1 = alpha D^-1 b; the iteration does not depend on a mesh's alpha)."""
    sizes, shared = CG[case]
    print(f"[gpu] cg iterates {case} matrix_free={matrix_free}", flush=True)
    mesh = meshes(sizes, shared)
    off = np.cumsum([0] + [6 * n ** 3 for n in sizes])
    st = B.State(mesh)
    st.set_bcs(B.VAR_POTENTIAL, KINDS, [1.0, 0.5, 0.0, -2.0, 0.1, 0.0])
    st.poisson_assemble()
    f = np.random.default_rng(5).normal(size=mesh.info.nc)
    b = host(st.poisson_rhs(dev(f)))

    def iterate(its, **kw):
        st.set_field(B.FIELD_P, dev(np.zeros(mesh.info.nc)))
        info = st.poisson_solve(dev(f), tol=1e-30, maxit=its, allow_not_converged=True, matrix_free=matrix_free, **kw)
        assert info["iterations"] == its
        return host(st.get_field(B.FIELD_P))

    if shared:                             # K couples the meshes: the scale of D^-1 counts
        dinv = 1.0 / poisson.assemble(build_geometry(*joined(sizes)), KINDS, [0.0] * 6)[0].diagonal()
    else:
        dinv = iterate(1) / b
    assert np.all(dinv > 0)
    ref = host_cg(lambda p: host(st.poisson_apply_free(dev(p))), b, dinv, off, 12)
    scale = np.repeat([np.abs(ref[s:e]).max() for s, e in zip(off[:-1], off[1:])], np.diff(off))
    for kw in (dict(chunk=12, graph=0), dict(chunk=4), dict(chunk=4, graph=1)):
        err = float((np.abs(iterate(12, **kw) - ref) / scale).max())
        print(f"[gpu] {kw}: {err:.2e}", flush=True)
        assert err < 1e-12
    if matrix_free:                        # the FP32 inner iterations of the same product
        st.set_field(B.FIELD_P, dev(np.zeros(mesh.info.nc)))
        info = st.poisson_solve(dev(f), tol=1e-10, method=B.SOLVE_IR_FP32, inner_tol=1e-2, matrix_free=True)
        assert info["status"] == B.OK
        r = b - host(st.poisson_apply_free(st.get_field(B.FIELD_P)))
        for s, e in zip(off[:-1], off[1:]):
            assert np.linalg.norm(r[s:e]) <= 1.01e-10 * np.linalg.norm(b[s:e])
        # each outer step gains 1e-2, and FP32 rounding costs no more than two
        assert info["outer"] <= 7


@pytest.mark.parametrize("cycle, coarse_max", [("v", 1024), ("v", 300), ("w", 16)])
def test_multigrid_cycle_equals_oracle(cycle, coarse_max):
    """16,464 cells: coarse rows over several slices and blocks, two levels and
    more.  1e-10 relative, as for the smaller grid's cycle."""
    print(f"[gpu] multigrid cycle {cycle} {coarse_max}", flush=True)
    mp = Mapped(14, 4)
    K = sp.csr_matrix(poisson.assemble(mp.geo, KINDS, [0.0] * 6)[0])
    K = sp.csr_matrix(K[mp.cp][:, mp.cp])
    K.sort_indices()
    st = B.State(mp.lib)
    st.set_bcs(B.VAR_POTENTIAL, KINDS, [0.0] * 6)
    st.poisson_assemble()
    info = st.amg_build(coarse_max=coarse_max, cycle=B.CYCLE_W if cycle == "w" else 0)
    levels, cinv = amg.build(K, coarse_max=coarse_max)
    assert info["rows"] == [A.shape[0] for A, _ in levels]
    r = np.random.default_rng(3).normal(size=mp.geo.nc)
    ref = np.empty_like(r)
    ref[mp.cp] = amg.v_cycle(levels, cinv, r[mp.cp], gamma=2 if cycle == "w" else 1)
    assert np.abs(host(st.amg_apply(dev(r))) - ref).max() < 1e-10 * np.abs(ref).max()


@pytest.mark.parametrize("precision", [B.FP64, B.FP32])
@pytest.mark.parametrize("n", [4, 27, 28])
def test_step_after_a_wait_equals_direct_launches(n, precision):
    """A step that follows a CFL evaluation replays its stages (to 131,072
    cells: n = 27 below, n = 28 above); bitwise the direct launches', over
    several replays with other work and a change of the walls between them,
    and inside a caller's own capture."""
    print(f"[gpu] step after a wait n={n} precision={precision}", flush=True)
    m = cube(n, 1000 + n)
    mesh = B.Mesh.from_cube(m, no_matrix=True)
    vel = dev(synth.rotating_velocity(m).T.ravel())

    def state():
        st = B.State(mesh, diffusivity=1e-3, precision=precision)
        st.set_bcs(B.VAR_SCALAR, [ZERO_FLUX] * 6)
        st.set_field(B.FIELD_VEL, vel)
        st.set_field(B.FIELD_U, dev(synth.gaussian_field(m)))
        return st

    a, b = state(), state()
    dt = a.cfl_dt(0.4)
    for rep in range(5):
        a.cfl_dt(0.4)
        a.step(1, dt)                      # replayed from the second on
        b.step(1, dt)                      # nothing waited for: direct
        if rep == 2:
            for st in (a, b):
                st.set_bcs(B.VAR_SCALAR, KINDS, [0.3, 0.1, 0.0, -0.2, 0.2, 0.0])
        assert np.array_equal(host(a.get_field(B.FIELD_U)), host(b.get_field(B.FIELD_U)))
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    a.conservation()                       # a wait, then a step under the caller's capture
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        a.step(1, dt, stream=s)
    for _ in range(3):
        g.replay()
        torch.cuda.synchronize()
        b.step(1, dt)
        assert a.conservation() == b.conservation()
        assert np.array_equal(host(a.get_field(B.FIELD_U)), host(b.get_field(B.FIELD_U)))


@pytest.mark.parametrize("precision, tol", [(B.FP64, 1e-12), (B.FP32, 1e-5)])
@pytest.mark.parametrize("n", [30, 32])
def test_vertex_values_by_slices_equal_oracle(n, precision, tol):
    """29,791 vertices (465 slices: the direct form) and 35,937 (562 slices,
    the last of 33 vertices: staged): the vertex values of a residual evaluation
    against the sum of the lists, alpha from the mesh's export.  A value is a sum
    of about 24 terms of size one: 1e-12 in FP64, 1e-5 in FP32."""
    print(f"[gpu] vertex values n={n} precision={precision}", flush=True)
    m = cube(n, 1000 + n)
    mesh = B.Mesh.from_cube(m, no_matrix=True)
    st = B.State(mesh, diffusivity=1e-3, precision=precision)
    st.set_bcs(B.VAR_SCALAR, [ZERO_FLUX] * 6)
    st.set_field(B.FIELD_VEL, dev(synth.rotating_velocity(m).T.ravel()))
    u = np.random.default_rng(2).normal(size=m.nc)
    st.set_field(B.FIELD_U, dev(u))
    got = host(st.residual()["u_node"])
    ptr, idx, alpha = (mesh.export(k) for k in ("node_ptr", "node_idx", "node_alpha"))
    ghost_owner = mesh.export("ghost_owner")
    cells = np.where(idx < m.nc, idx, ghost_owner[np.maximum(idx - m.nc, 0)])
    ui = u[mesh.export("cell_perm")]
    ref = np.add.reduceat(alpha * ui[cells], ptr[:-1])
    out = np.empty_like(ref)
    out[mesh.export("vert_perm")] = ref
    assert np.abs(got - out).max() < tol * np.abs(out).max()
