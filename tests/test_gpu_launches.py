"""How many kernels and copies a call enqueues, counted by capturing it: small
meshes are bound by their launches."""
import ctypes as C

import numpy as np
import pytest

import synth
from conftest import cube
from oracle.geometry import DIRICHLET, NEUMANN, ZERO_FLUX

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
B = pytest.importorskip("paper_2203_00925_amd.binding")

KINDS = [DIRICHLET, NEUMANN, ZERO_FLUX, DIRICHLET, NEUMANN, ZERO_FLUX]


@pytest.fixture(scope="module", autouse=True)
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)


def hip():
    """The HIP runtime this process has loaded."""
    with open("/proc/self/maps") as f:
        paths = {line.split()[-1] for line in f if "libamdhip64" in line}
    assert len(paths) == 1, paths
    return C.CDLL(paths.pop())


def nodes(call):
    """Nodes of the graph that capturing call(stream) makes; the graph is not run."""
    h, s = hip(), torch.cuda.Stream()
    call(s)                                # warm: tables, torch's pools
    torch.cuda.synchronize()
    q, g, n = C.c_void_p(s.cuda_stream), C.c_void_p(), C.c_size_t()
    assert h.hipStreamBeginCapture(q, 2) == 0          # relaxed
    try:
        call(s)
    finally:
        rc = h.hipStreamEndCapture(q, C.byref(g))
    assert rc == 0
    assert h.hipGraphGetNodes(g, None, C.byref(n)) == 0
    assert h.hipGraphDestroy(g) == 0
    return n.value


def state(n=8, **kw):
    m = cube(n, 1000 + n)
    st = B.State(B.Mesh.from_cube(m), diffusivity=1e-3, **kw)
    st.set_bcs(B.VAR_SCALAR, KINDS, [0.3, 0.1, 0.0, -0.2, 0.2, 0.0])
    st.set_bcs(B.VAR_POTENTIAL, KINDS, [1.0, 0.5, 0.0, -2.0, 0.1, 0.0])
    st.set_field(B.FIELD_VEL, torch.from_numpy(np.ascontiguousarray(synth.rotating_velocity(m).T.ravel())))
    st.set_field(B.FIELD_U, torch.from_numpy(synth.gaussian_field(m)))
    return st


def test_residual_launches():
    """Ghosts, moments, gradient, face fluxes; the cells' parts in the caller's
    order, the vertex values, the fluxes: no more than the nine of the one-kernel
    gradient."""
    st = state()
    print("[gpu] launches of a residual evaluation", flush=True)
    assert nodes(lambda s: st.residual(stream=s)) <= 9
