"""admm_solve leaves the displacement of a cell that it does not iterate as the
caller wrote it, in double precision (the float form strips the fluctuation's
mean and checkerboards from every cell of a call).

Two cells are solved, then one gets a new load and the other, converged, a
displacement with a mean and a Nyquist pattern on top: after the next solve that
field is there bit for bit, in both forms of the iterations.
"""
import numpy as np
import pytest

from paper_2010_06697_amd import admm, microstructure as M
from parity_util import gpu_solver

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form", [0, 1])
def test_idle_cell_keeps_its_displacement(form):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    shapes = [(8, 12, 16), (6, 8, 12)]
    print("idle cell", "explicit" if form else "implicit", flush=True)
    phases = [M.random_two_phase(sh, 0.4, seed=k) for k, sh in enumerate(shapes)]
    s = gpu_solver(phases, [M.neohooke(4.0, 8.0), M.neohooke(1.0, 4.0)],
                   [M.random_fbar(0.02, seed=3)] * 2, "fp64", rho0=5.0, mu_ref=2.0, tol_p=1e-4,
                   tol_d=1e-4, explicit_fields=form)
    assert s.solve()[0] == admm.OK
    u = s.state(0)["u"]
    k3, k2, k1 = np.meshgrid(*[np.arange(n) for n in shapes[0]], indexing="ij")
    u = u + 0.25 + 0.5 * (-1.0) ** (k1 + k2 + k3)
    s.set_state(0, u=u)
    s.set_load(1, M.random_fbar(0.03, seed=4))
    assert s.solve()[0] == admm.OK
    got, its = s.state(0)["u"], s.info(1)[0]
    s.close()
    assert its > 1
    same = bool(np.array_equal(got, u))
    assert same
