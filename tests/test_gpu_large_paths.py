"""The kernels and block orders that only meshes above two million cells
reach, and CG iterations over restarts.

n = 71: 2,147,466 cells in 8,389 tiles (the last of 122 cells), 373,248
vertices in 5,832 slices.  The tiled product takes its tiles in two rounds and
the step's and the vertices' kernels their blocks in windows, the stored
product two tiles a block, the vector kernels 512 threads of five rows."""
import numpy as np
import pytest

import synth
from conftest import cube, cube_geometry
from oracle import poisson
from oracle.geometry import DIRICHLET, NEUMANN, ZERO_FLUX

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
B = pytest.importorskip("paper_2203_00925_amd.binding")

N = 71
KINDS = [DIRICHLET, NEUMANN, ZERO_FLUX, DIRICHLET, NEUMANN, ZERO_FLUX]
VALS = [1.0, 0.5, 0.0, -2.0, 0.1, 0.0]


@pytest.fixture(scope="module", autouse=True)
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)


@pytest.fixture(scope="module")
def big():
    print(f"[gpu] large paths: building the n={N} mesh", flush=True)
    m = synth.jittered_cube(N, 6)
    return m, B.Mesh.from_cube(m)


def cg(apply, b, dinv, its, restart=0):
    """x after `its` Jacobi-CG iterations from zero, reopened from the true
    residual every `restart`."""
    x, r = torch.zeros_like(b), b.clone()
    for k in range(its):
        if k == 0 or (restart and k % restart == 0):
            if k:
                r = b - apply(x)
            z = dinv * r
            p, rz = z.clone(), r @ z
        q = apply(p)
        a = rz / (p @ q)
        x, r = x + a * p, r - a * q
        z = dinv * r
        new = r @ z
        p, rz = z + new / rz * p, new
    return x


def iterate(st, f, its, **kw):
    st.set_field(B.FIELD_P, torch.zeros_like(f))
    info = st.poisson_solve(f, tol=1e-30, maxit=its, allow_not_converged=True, **kw)
    assert info["iterations"] == its
    return st.get_field(B.FIELD_P)


def test_large_cg_iterates(big):
    """Twelve iterations, launched and replayed, matrix-free and stored: 1e-12
    of the largest x, as for the smaller meshes (sums of 30 terms a row, each
    iteration amplifying an earlier one's error by at most about ten); the
    scale of D^-1 drops out.  The refined form by its true residual."""
    m, mesh = big
    st = B.State(mesh)
    st.set_bcs(B.VAR_POTENTIAL, KINDS, VALS)
    st.poisson_assemble()
    f = torch.from_numpy(np.random.default_rng(5).normal(size=m.nc)).cuda()
    b = st.poisson_rhs(f)
    ref = None
    for free in (True, False):
        if ref is None:
            ref = cg(st.poisson_apply_free, b, iterate(st, f, 1, matrix_free=True) / b, 12)
        for kw in (dict(chunk=12, graph=0), dict(chunk=4)):
            err = float((iterate(st, f, 12, matrix_free=free, **kw) - ref).abs().max() / ref.abs().max())
            print(f"[gpu] large CG matrix_free={free} {kw}: {err:.2e}", flush=True)
            assert err < 1e-12
    st.set_field(B.FIELD_P, torch.zeros_like(f))
    info = st.poisson_solve(f, tol=1e-7, method=B.SOLVE_IR_FP32, inner_tol=1e-2, matrix_free=True)
    r = b - st.poisson_apply_free(st.get_field(B.FIELD_P))
    assert info["status"] == B.OK and float(r.norm()) <= 1.01e-7 * float(b.norm())


@pytest.mark.parametrize("precision, tol", [(B.FP64, 1e-13), (B.FP32, 1e-5)])
def test_large_step_equals_its_residuals(big, precision, tol):
    """A step, launched and captured, against u + a dt Res(u) from the residual
    evaluation's own face kernel.  A stage adds dt times a sum of four fluxes,
    CFL 0.4 of u at most, each a few tens of roundings: 3 x 0.4 x 40 x 1.1e-16
    is 5e-15, with the rounding of u 1e-14 in FP64, 3e-6 in FP32.  The vertex
    values against the sum of their lists."""
    m, mesh = big
    st = B.State(mesh, diffusivity=1e-3, precision=precision)
    st.set_bcs(B.VAR_SCALAR, KINDS, VALS)
    st.set_field(B.FIELD_VEL, torch.from_numpy(np.ascontiguousarray(synth.rotating_velocity(m).T.ravel())))
    dtype = torch.float32 if precision == B.FP32 else torch.float64
    u = torch.from_numpy(synth.gaussian_field(m)).cuda().to(dtype)
    st.set_field(B.FIELD_U, u)
    dt = st.cfl_dt(0.4)
    uk = u
    for k, a in enumerate((0.5, 0.5, 1.0)):
        st.set_field(B.FIELD_U, uk)
        out = st.residual()
        if k == 0:                         # 16-bit halo numbers, windows of slices
            ptr, idx, alpha = (mesh.export(x) for x in ("node_ptr", "node_idx", "node_alpha"))
            ui = u.double().cpu().numpy()[mesh.export("cell_perm")]
            inner = np.add.reduceat((idx >= m.nc).astype(np.int8), ptr[:-1]) == 0
            ref = np.add.reduceat(alpha * ui[np.where(idx < m.nc, idx, 0)], ptr[:-1])
            got = out["u_node"].cpu().numpy()[mesh.export("vert_perm")]
            err = np.abs(got - ref)[inner].max() / np.abs(ref).max()
            print(f"[gpu] large vertex values precision={precision}: {err:.2e}", flush=True)
            assert err < tol
        uk = (u.double() + a * dt * out["res"]).to(dtype)
    for captured in (False, True):
        st.set_field(B.FIELD_U, u)
        st.step_graph(1, dt) if captured else st.step(1, dt)
        if captured:                       # the first call launches, this one replays
            st.set_field(B.FIELD_U, u)
            st.step_graph(1, dt)
        err = float((st.get_field(B.FIELD_U, dtype=dtype) - uk).abs().max() / uk.abs().max())
        print(f"[gpu] large step precision={precision} captured={captured}: {err:.2e}", flush=True)
        assert err < tol


@pytest.mark.parametrize("matrix_free", [True, False])
def test_cg_iterates_over_restarts(matrix_free):
    """24 iterations reopened every 8 against the same on the host side, D^-1
    from the oracle's matrix: a reopening forgets the error of the iterations
    before it, eight amplify rounding to 1e-12 of x, three times that here."""
    print(f"[gpu] CG over restarts matrix_free={matrix_free}", flush=True)
    m = cube(12, 3)
    st = B.State(B.Mesh.from_cube(m))
    st.set_bcs(B.VAR_POTENTIAL, KINDS, VALS)
    st.poisson_assemble()
    K = poisson.assemble(cube_geometry(12, 3), KINDS, [0.0] * 6)[0]
    dinv = 1.0 / torch.from_numpy(K.diagonal()).cuda()
    f = torch.from_numpy(np.random.default_rng(5).normal(size=m.nc)).cuda()
    b = st.poisson_rhs(f)
    ref = cg(st.poisson_apply_free, b, dinv, 24, restart=8)
    for kw in (dict(chunk=8, graph=0), dict(chunk=5)):
        got = iterate(st, f, 24, restart=8, matrix_free=matrix_free, **kw)
        assert float((got - ref).abs().max()) < 3e-12 * float(ref.abs().max())


def test_vertex_recurrence_does_not_drift():
    """500 iterations without a reopening, far past convergence: the recurrence's
    residual vanishes and the true one is what the two have drifted apart.  The
    vertex values of p follow a recurrence of their own, one rounding an
    iteration beside the dozen of a direct sum: within four times the drift of
    the same iteration with direct products."""
    print("[gpu] CG residual gap", flush=True)
    m = cube(12, 3)
    st = B.State(B.Mesh.from_cube(m))
    st.set_bcs(B.VAR_POTENTIAL, [DIRICHLET] * 6, VALS)
    K = poisson.assemble(cube_geometry(12, 3), [DIRICHLET] * 6, [0.0] * 6)[0]
    dinv = 1.0 / torch.from_numpy(K.diagonal()).cuda()
    f = torch.from_numpy(np.random.default_rng(5).normal(size=m.nc)).cuda()
    st.poisson_assemble()
    b = st.poisson_rhs(f)
    its = 500

    def gap(x, r):
        return float((b - st.poisson_apply_free(x) - r).norm() / b.norm())

    x, r = torch.zeros_like(b), b.clone()
    z = dinv * r
    p, rz = z.clone(), r @ z
    for _ in range(its):
        q = st.poisson_apply_free(p)
        a = rz / (p @ q)
        x, r = x + a * p, r - a * q
        z = dinv * r
        new = r @ z
        p, rz = z + new / rz * p, new
    direct = gap(x, r)
    st.set_field(B.FIELD_P, torch.zeros_like(f))
    info = st.poisson_solve(f, tol=1e-30, maxit=its, restart=0, chunk=its, history=4, matrix_free=True,
                            allow_not_converged=True)
    true = float((b - st.poisson_apply_free(st.get_field(B.FIELD_P))).norm() / b.norm())
    print(f"[gpu] recurrence {info['history'][1]:.1e}, true {true:.2e}, direct products {direct:.2e}", flush=True)
    assert info["history"][1] < 1e-2 * true <= 4e-2 * direct
