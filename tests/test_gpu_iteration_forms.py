"""The two forms of neo-Hookean iterations with exact local steps: implicit
(F and Lambda held as A, F - A and du between the steps) and explicit
(explicit_fields=1; what a card without room runs), both through admm_step and
admm_solve against the oracle's iterations.

Bounds, those of the other parity tests: double 1e-10 relative on u, F and
Lambda, float 2e-5 (a few hundred units of float rounding over up to 25
iterations). The penalty sequences are the oracle's.
"""
import numpy as np
import pytest

from paper_2010_06697_amd import admm, microstructure as M
from parity_util import gpu_solver, oracle_iterations, random_state, rel

pytestmark = pytest.mark.gpu

MATS = [M.neohooke(10.0, 40.0), M.neohooke(1.0, 4.0)]
TOL = {"fp64": 1e-10, "fp32": 2e-5}


def say(*a):
    print(*a, flush=True)


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def negative(shape, rho, seed):
    """A state whose data A has det A < 0 on a third of the voxels at rho."""
    u, F, L = random_state(shape, seed=seed)
    rng = np.random.default_rng(seed + 1)
    neg = rng.random(shape) < 1.0 / 3.0
    L[8][neg] = -rho * rng.uniform(1.2, 1.6, size=int(neg.sum()))
    return u, F, L


def close(precision, got, want):
    err = {f: rel(got[f], w) for f, w in zip(("u", "F", "Lambda"), want)}
    say("  ", err)
    assert max(err.values()) <= TOL[precision]


# the smallest cell, a plane, remainders, more than 256 workgroups of voxels
@pytest.mark.parametrize("form", [0, 1])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("shape,calls,state", [((4, 4, 4), [1, 4], 0), ((1, 54, 162), [3, 2], 0),
                                               ((12, 16, 24), [2, 1], 1), ((36, 48, 48), [3], 1)])
def test_steps(form, precision, shape, calls, state):
    say("steps", "explicit" if form else "implicit", precision, shape, calls, state)
    phase = M.random_two_phase(shape, 0.4, seed=10)
    Fbar = M.random_fbar(0.04, seed=11)
    if shape[0] == 1:
        Fbar[2, :2] = Fbar[:2, 2] = 0.0
        Fbar[2, 2] = 1.0
    s0 = negative(shape, 12.0, seed=16) if state else None
    s = gpu_solver([phase], MATS, [Fbar], precision, rho0=12.0, mu_ref=4.0, explicit_fields=form,
                   use_graph=len(calls) % 2, check_every=2)
    if s0:
        s.set_state(0, u=s0[0], F=s0[1], Lambda=s0[2])
    for n in calls:
        assert s.step(n)[0] == admm.OK
    got = s.state(0)
    s.close()
    close(precision, got, oracle_iterations(phase, MATS, Fbar, sum(calls), 12.0, 4.0, state=s0)[:3])


@pytest.mark.parametrize("form", [0, 1])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_penalty_changes(form, precision):
    say("penalty changes", "explicit" if form else "implicit", precision)
    phase, Fbar = M.random_two_phase((16, 12, 24), 0.4, seed=10), M.random_fbar(0.04, seed=11)
    s = gpu_solver([phase], MATS, [Fbar], precision, rho0=40.0, mu_ref=4.0, explicit_fields=form,
                   adapt_rho=1, rho_min=1.0, rho_max=50.0)
    for n in (3, 1, 12, 9):
        assert s.step(n)[0] == admm.OK
    got, rho = s.state(0), s.history(0)[2]
    s.close()
    u, F, L, r = oracle_iterations(phase, MATS, Fbar, 25, 40.0, 4.0, adapt=True)
    assert len(set(rho.tolist())) > 1 and np.array_equal(rho, r["rho_hist"])
    close(precision, got, (u, F, L))


# cells that stop at different iterations, whose F and Lambda the end of the
# call writes; the Newton fallback in the pass itself (at most 256 workgroups)
# and in a second one
@pytest.mark.parametrize("form", [0, 1])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("shapes", [[(12, 16, 24), (8, 6, 18)], [(36, 48, 48), (12, 16, 24)]])
def test_solve_leaves_the_last_iterates(form, precision, shapes):
    say("solve", "explicit" if form else "implicit", precision, shapes)
    phases = [M.random_two_phase(sh, 0.4, seed=30 + k) for k, sh in enumerate(shapes)]
    Fbars = [M.random_fbar(a, seed=32) for a in (0.04, 0.002)]
    states = [negative(sh, 12.0, seed=40) if k == 0 else None for k, sh in enumerate(shapes)]
    s = gpu_solver(phases, MATS, Fbars, precision, rho0=12.0, mu_ref=4.0, explicit_fields=form,
                   tol_p=2e-3, tol_d=2e-3, max_iter=24, check_every=4)
    s.set_state(0, u=states[0][0], F=states[0][1], Lambda=states[0][2])
    s.solve()
    its = [s.info(k)[0] for k in range(2)]
    got = [s.state(k) for k in range(2)]
    s.close()
    say("  iterations", its)
    assert its[0] != its[1] and min(its) >= 1
    for k in range(2):
        close(precision, got[k], oracle_iterations(phases[k], MATS, Fbars[k], its[k], 12.0, 4.0,
                                                   state=states[k])[:3])


# a cell has the same bits alone and in any batch, also where the batch is
# beyond 256 workgroups and the voxels without a closed form take the second
# pass, a kernel of its own
@pytest.mark.parametrize("form", [0, 1])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_a_cell_keeps_its_bits_in_a_batch(form, precision):
    say("cell alone and in a batch", "explicit" if form else "implicit", precision)
    shapes = [(12, 16, 24), (36, 48, 48)]
    phases = [M.random_two_phase(sh, 0.4, seed=50 + k) for k, sh in enumerate(shapes)]
    Fbar = M.random_fbar(0.04, seed=52)
    state, out = negative(shapes[0], 12.0, seed=53), []
    for n in (1, 2):
        s = gpu_solver(phases[:n], MATS, [Fbar] * n, precision, rho0=12.0, mu_ref=4.0,
                       explicit_fields=form)
        s.set_state(0, u=state[0], F=state[1], Lambda=state[2])
        assert s.step(3)[0] == admm.OK
        out.append((s.state(0), s.history(0), s.info(0)))
        s.close()
    (a, ha, ia), (b, hb, ib) = out
    same = [np.array_equal(a[f], b[f]) for f in ("u", "F", "Lambda")]
    say("  u F Lambda", same, [rel(a[f], b[f]) for f in ("u", "F", "Lambda")])
    assert all(same) and ia == ib
    assert all(np.array_equal(x, y) for x, y in zip(ha, hb))
