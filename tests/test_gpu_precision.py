"""Vertex values and gradients of the residual evaluation beside the same sums
taken directly in 64 bits, both measured from extended precision: the star
form regroups the sums and must not cost digits."""
import numpy as np
import pytest

from conftest import cube
from oracle.geometry import DIRICHLET, ZERO_FLUX

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
B = pytest.importorskip("paper_2203_00925_amd.binding")
X = np.longdouble


@pytest.fixture(scope="module", autouse=True)
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)


def solve(A, b):
    """Batched Gaussian elimination with partial pivoting (A [m, n, n], b [m, n])."""
    A, b, at = A.copy(), b.copy(), np.arange(len(A))
    n = A.shape[1]
    for c in range(n):
        p = np.abs(A[:, c:, c]).argmax(1) + c
        A[at, p], A[:, c] = A[:, c].copy(), A[at, p].copy()
        b[at, p], b[:, c] = b[:, c].copy(), b[at, p].copy()
        for k in range(c + 1, n):
            m = A[:, k, c] / A[:, c, c]
            A[:, k] -= m[:, None] * A[:, c]
            b[:, k] -= m * b[:, c]
    for c in range(n - 1, -1, -1):
        for k in range(c + 1, n):
            b[:, c] -= A[:, c, k] * b[:, k]
        b[:, c] /= A[:, c, c]
    return b


def rms(a):
    return float(np.sqrt((a.astype(X) ** 2).mean()))


# 8,000 cells; 48,000; 196,608 (35,937 vertices: the moments by slices)
@pytest.mark.parametrize("walls", ["closed", "half"])
@pytest.mark.parametrize("n, gradient", [(11, True), (20, True), (32, False)])
def test_star_sums_cost_no_digits(n, gradient, walls):
    """The direct sums add products of weights and values in list order; the
    star form has as many roundings of the same size, summed in another order:
    within 1.2 of the direct sums' distance from the exact ones (root mean
    square over 1,700 vertices or 8,000 cells and more)."""
    print(f"[gpu] star sums n={n} {walls}", flush=True)
    mesh = B.Mesh.from_cube(cube(n, 7), no_matrix=True)
    i = mesh.info
    st = B.State(mesh)
    kind, val = (ZERO_FLUX, 0.0) if walls == "closed" else (DIRICHLET, 0.5)
    st.set_bcs(B.VAR_SCALAR, [kind] * 6, [val] * 6)
    xc, owner = mesh.export("centre").T, mesh.export("ghost_owner")
    u = np.exp(-((xc[:i.nc] - 0.45) ** 2).sum(1) / 0.03)
    user = np.empty(i.nc)
    user[mesh.export("cell_perm")] = u
    st.set_field(B.FIELD_U, torch.from_numpy(user))
    st.set_field(B.FIELD_VEL, torch.zeros(3 * i.nc, dtype=torch.float64))
    got = {k: v.cpu().numpy() for k, v in st.residual().items()}
    ue = np.concatenate([u, u[owner] if walls == "closed" else 2 * val - u[owner]])

    # vertex values: the least-squares weights of each list
    ptr, idx, alpha = (mesh.export(k) for k in ("node_ptr", "node_idx", "node_alpha"))
    v = np.repeat(np.arange(i.nv), np.diff(ptr))
    xv = cube(n, 7).xyz[mesh.export("vert_perm")]
    a = np.concatenate([np.ones((len(v), 1), X), xc[idx].astype(X) - xv[v]], axis=1)
    sums = lambda t: np.add.reduceat(t, ptr[:-1], axis=0)
    w = solve(sums((a[:, :, None] * a[:, None, :]).reshape(-1, 16)).reshape(-1, 4, 4),
              np.tile(np.array([1, 0, 0, 0], X), (i.nv, 1)))
    exact = sums((a * w[v]).sum(1) * ue[idx])
    lib = got["u_node"][mesh.export("vert_perm")]
    here, direct = rms(lib - exact), rms(sums(alpha * ue[idx]) - exact)
    print(f"[gpu] vertex values {here:.2e}, direct {direct:.2e}", flush=True)
    assert here <= 1.2 * direct
    if not gradient:
        return
    # gradients: least squares over the stencil
    ptr, idx, minv = (mesh.export(k) for k in ("stencil_ptr", "stencil_idx", "minv"))
    r = np.repeat(np.arange(i.nc), np.diff(ptr))
    sums = lambda t: np.add.reduceat(t, ptr[:-1], axis=0)
    d = xc[idx].astype(X) - xc[r]
    exact = solve(sums((d[:, :, None] * d[:, None, :]).reshape(-1, 9)).reshape(-1, 3, 3),
                  sums(d * (ue[idx].astype(X) - ue[r])[:, None]))
    J = sums((xc[idx] - xc[r]) * (ue[idx] - ue[r])[:, None])
    full = minv[[0, 1, 2, 1, 3, 4, 2, 4, 5]].T.reshape(-1, 3, 3)
    lib = got["grad"].T[mesh.export("cell_perm")]
    here, direct = rms(lib - exact), rms((full * J[:, None, :]).sum(-1) - exact)
    print(f"[gpu] gradients {here:.2e}, direct {direct:.2e}", flush=True)
    assert here <= 1.2 * direct
