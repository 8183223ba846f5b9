"""GPU parity of the iterations that keep F and Lambda implicit (neo-Hookean
cells, exact local step) and of the two-step transforms, at the sizes where
their tiles, remainders and dispatch change. Against the oracle, with the
bounds of the other parity tests: double 1e-10 relative on u, F, Lambda and
<P> after whole iterations and 1e-12 on a projection, float 1e-5 on <P> and
2e-5 on a projection.
"""
import numpy as np
import pytest

import oracle as O
from paper_2010_06697_amd import admm, microstructure as M
from parity_util import gpu_solver, omats, oracle_iterations, random_state, rel

pytestmark = pytest.mark.gpu

MATS = [M.neohooke(10.0, 40.0), M.neohooke(1.0, 4.0)]
LENGTHS = [4, 6, 8, 12, 16, 18, 24, 32, 36, 48, 54, 64, 72, 96, 108, 128, 144, 162, 192, 216, 256]


def say(*a):
    print(*a, flush=True)


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


# every length on every axis, the other edges leaving remainders of the tiles
# (odd numbers of complex lines, columns no multiple of a tile), and the plane
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("n", LENGTHS)
def test_every_length_projects_on_every_axis(precision, n):
    for shape in [(4, 6, n), (6, n, 12), (n, 6, 8), (1, 6, n), (1, n, 18)]:
        say("projection", precision, shape)
        phase = M.random_two_phase(shape, 0.4, seed=1)
        u, F, L = random_state(shape, seed=n)
        s = gpu_solver([phase], MATS, [M.random_fbar(0.03, seed=2)], precision, rho0=2.5)
        s.set_state(0, u=0 * u, F=F, Lambda=L)
        s.project_step()
        got = s.state(0)["u_prev"]
        s.close()
        assert rel(got, O.project(F - L / 2.5)) <= (1e-12 if precision == "fp64" else 2e-5), shape


def check(precision, shape, calls, free=None, graph=1, state=None, **kw):
    phase = M.random_two_phase(shape, 0.4, seed=10)
    Fbar = M.random_fbar(0.04, seed=11)
    if shape[0] == 1:
        Fbar = np.eye(3)
        Fbar[:2, :2] += 0.04 * np.random.default_rng(3).standard_normal((2, 2))
    rho = kw.pop("rho", 8.0)
    s = gpu_solver([phase], MATS, [Fbar], precision, rho0=rho, mu_ref=4.0, use_graph=graph, **kw)
    if state is not None:
        s.set_state(0, u=state[0], F=state[1], Lambda=state[2])
    for n in calls:
        assert s.step(n)[0] == admm.OK
    st = s.state(0)
    P, _ = s.homogenized_stress(0)
    hr = s.history(0)[2]
    s.close()
    u, F, L, r = oracle_iterations(phase, MATS, Fbar, sum(calls), rho, 4.0,
                                   adapt=bool(kw.get("adapt_rho", 0)), state=state)
    Po = O.mean_stress(phase, omats(MATS), F)
    say("  rel u F L P:", rel(st["u"], u), rel(st["F"], F), rel(st["Lambda"], L), rel(P, Po))
    if precision == "fp64":
        assert rel(st["u"], u) <= 1e-10 and rel(st["F"], F) <= 1e-10
        assert rel(st["Lambda"], L) <= 1e-10 and rel(P, Po) <= 1e-10
        if "adapt_rho" in kw:
            assert np.array_equal(hr, r["rho_hist"]) and len(set(hr.tolist())) > 1
    else:
        assert rel(P, Po) <= 1e-5


# the smallest cells; lines of 18 points per thread; a plane; more than 256
# workgroups of voxels (the Newton fallback is a second pass there);
# calls of one iteration (nothing implicit survives a call) and of several
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("shape,calls", [((4, 4, 4), [1, 4]), ((1, 4, 4), [5]),
                                         ((4, 6, 216), [2, 1, 2]), ((6, 162, 12), [4]),
                                         ((1, 54, 162), [3, 2]), ((32, 48, 48), [4])])
def test_implicit_iterations_match_oracle(precision, shape, calls):
    say("implicit iterations", precision, shape, calls)
    check(precision, shape, calls, graph=len(calls) % 2)


# penalty changes inside and between calls: Lambda is recovered, the data formed anew
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("calls", [[25], [3, 1, 12, 9]])
def test_implicit_iterations_through_penalty_changes(precision, calls):
    say("implicit iterations, adaptive penalty", precision, calls)
    check(precision, (16, 12, 24), calls, rho=40.0, adapt_rho=1, rho_min=1.0, rho_max=50.0)


# a third of the voxels outside the closed form's range in the first
# iterations, below and beyond 256 workgroups (in the pass, or a second one)
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("shape", [(12, 16, 24), (36, 48, 48)])
def test_implicit_iterations_with_negative_det_data(precision, shape):
    say("implicit iterations, det A < 0 on a third of the voxels", precision, shape)
    u, F, L = random_state(shape, seed=16)
    rng = np.random.default_rng(17)
    neg = rng.random(shape) < 1.0 / 3.0
    L[8][neg] = -12.0 * rng.uniform(1.2, 1.6, size=int(neg.sum()))
    check(precision, shape, [2, 1], state=(u, F, L), rho=12.0)
