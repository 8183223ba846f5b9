"""Float iterations keep F itself between the steps of a call, at its own
rounding: nothing that depends on F depends on where a call ends.

- The residuals of n iterations in one call are those of n calls of one
  iteration, whose fields are stored and read back: the same sums of the same
  floats, in the same order. Bound 1e-12 (the kernels for the end of a call may
  contract an expression of the double sums otherwise).
- F, u and Lambda after admm_solve are those of admm_step with as many
  iterations: F bit for bit, also where the closed form does not apply;
  Lambda to one unit of float rounding.
"""
import numpy as np
import pytest

from paper_2010_06697_amd import admm, microstructure as M
from parity_util import gpu_solver, random_state, rel

pytestmark = pytest.mark.gpu

# a stiff phase at a small penalty: Lambda / rho is many times F - I
MATS = [M.neohooke(100.0, 400.0), M.neohooke(1.0, 4.0)]


def say(*a):
    print(*a, flush=True)


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def solver(shape, negative, n):
    phase = M.random_two_phase(shape, 0.4, seed=21)
    s = gpu_solver([phase], MATS, [M.random_fbar(0.04, seed=22)], "fp32", rho0=3.0, mu_ref=25.0,
                   tol_p=0.0, tol_d=0.0, max_iter=n, check_every=n)
    if negative:  # det A < 0 on a third of the voxels in the first iteration
        u, F, L = random_state(shape, seed=23)
        rng = np.random.default_rng(24)
        neg = rng.random(shape) < 1.0 / 3.0
        L[8][neg] = -3.0 * rng.uniform(1.2, 1.6, size=int(neg.sum()))
        s.set_state(0, u=u, F=F, Lambda=L)
    return s


# one workgroup per CU at most, and beyond
@pytest.mark.parametrize("negative", [0, 1])
@pytest.mark.parametrize("shape", [(12, 16, 24), (36, 48, 48)])
def test_residuals_do_not_depend_on_where_calls_end(shape, negative):
    say("residuals over calls", shape, negative)
    hist = []
    for calls in ([6], [1] * 6):
        s = solver(shape, negative, 6)
        for n in calls:
            assert s.step(n)[0] == admm.OK
        hist.append(s.history(0))
        s.close()
    err = [float(np.max(np.abs(a / b - 1.0))) for a, b in zip(*hist)]
    say("  r_p r_d rho", err)
    assert max(err) <= 1e-12


# n = 1: the voxels outside the closed form's range end the call
@pytest.mark.parametrize("negative,n", [(0, 4), (1, 1), (1, 3)])
@pytest.mark.parametrize("shape", [(12, 16, 24), (36, 48, 48)])
def test_solve_leaves_what_steps_leave(shape, negative, n):
    say("solve against steps", shape, negative, n)
    s = solver(shape, negative, n)
    assert s.step(n)[0] == admm.OK
    a = s.state(0)
    s.close()
    s = solver(shape, negative, n)
    assert s.solve()[0] == admm.NOT_CONVERGED
    assert s.info(0)[0] == n
    b = s.state(0)
    s.close()
    same = [np.array_equal(a[f], b[f]) for f in ("u", "F")]
    say("  u F same", same, "F", rel(b["F"], a["F"]), "Lambda", rel(b["Lambda"], a["Lambda"]))
    assert all(same)
    assert rel(b["Lambda"], a["Lambda"]) <= 1.2e-7
