"""What a call costs beside another that does the same work: calls that are
bound by launches and graph captures, compared by their times in turn (the
smallest of several medians)."""
import time

import numpy as np
import pytest

import synth
from conftest import cube
from oracle.geometry import DIRICHLET, NEUMANN, ZERO_FLUX

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
B = pytest.importorskip("paper_2203_00925_amd.binding")

KINDS = [DIRICHLET, NEUMANN, ZERO_FLUX, DIRICHLET, NEUMANN, ZERO_FLUX]
VALS = [1.0, 0.5, 0.0, -2.0, 0.1, 0.0]


@pytest.fixture(scope="module", autouse=True)
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)


def times(*calls, reps=15, rounds=5):
    """Microseconds of each call, waited for, the calls taken in turn."""
    out = [[] for _ in calls]
    for _ in range(rounds):
        for k, call in enumerate(calls):
            one = []
            for _ in range(reps):
                torch.cuda.synchronize()
                t = time.perf_counter()
                call()
                torch.cuda.synchronize()
                one.append(time.perf_counter() - t)
            out[k].append(float(np.median(one)) * 1e6)
    best = [min(o) for o in out]
    print("[gpu] " + ", ".join(f"{b:.1f} us" for b in best), flush=True)
    return best


def state(n=8, **kw):
    m = cube(n, 1000 + n)
    st = B.State(B.Mesh.from_cube(m), diffusivity=1e-3, **kw)
    st.set_bcs(B.VAR_SCALAR, KINDS, VALS)
    st.set_bcs(B.VAR_POTENTIAL, KINDS, VALS)
    st.set_field(B.FIELD_VEL, torch.from_numpy(np.ascontiguousarray(synth.rotating_velocity(m).T.ravel())))
    st.set_field(B.FIELD_U, torch.from_numpy(synth.gaussian_field(m)))
    return st, torch.from_numpy(np.random.default_rng(5).normal(size=m.nc)).cuda()


@pytest.mark.parametrize("method", [B.SOLVE_PLAIN, B.SOLVE_IR_FP32])
def test_converged_matrix_free_solve_costs_its_residual(method):
    """A solve that is converged on entry opens the loop and ends: two kernels
    more than on the stored matrix (the product), none for an iteration that
    does not follow.  3,072 cells: the stored matrix's product is as long as
    one of them, so no more than a quarter longer."""
    st, f = state()
    st.poisson_assemble()
    st.poisson_solve(f, tol=1e-11)
    free = lambda: st.poisson_solve(f, tol=1e-8, matrix_free=True, method=method)
    stored = lambda: st.poisson_solve(f, tol=1e-8, method=method)
    assert free()["iterations"] == 0 and stored()["iterations"] == 0
    a, b = times(free, stored)
    assert a < 1.25 * b
