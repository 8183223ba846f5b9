"""GPU parity of the Bloch wave's secular equation on both sides of its
dispatch: up to 49152 modes one workgroup takes every sum, beyond them several
launches of many workgroups take the first ones. Fixed numbers of iterations
against the oracle (bisection to the last bit), tolerances as for the other
Bloch tests: 1e-9 relative on beta and rho sigma, 1e-7 on the mode.
"""
import numpy as np
import pytest

import oracle as O
from paper_2010_06697_amd import admm, microstructure as M
from parity_util import omats, rel

pytestmark = pytest.mark.gpu

MATS = [M.neohooke(10.0, 20.0), M.neohooke(1.0, 2.0)]


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


# the smallest grid (16 voxels of one workgroup), one workgroup's most modes
# (48 x 32 x 32), the first grid beyond (36 x 48 x 32)
@pytest.mark.parametrize("shape,iters", [((1, 4, 4), 8), ((4, 4, 4), 8), ((32, 32, 48), 6),
                                         ((32, 48, 36), 6)])
def test_secular_dispatch_matches_oracle(shape, iters):
    print("bloch secular", shape, iters, flush=True)
    rng = np.random.default_rng(11)
    n3, n2, n1 = shape
    phase = M.random_two_phase(shape, 0.5, seed=3)
    F = np.zeros((9,) + shape)
    F[[0, 4, 8]] = 1.0
    F += 0.03 * rng.standard_normal(F.shape)
    omega = np.array([0.0, 2 * np.pi / (3 * n2), 0.2])
    p0 = rng.standard_normal((3,) + shape) + 1j * rng.standard_normal((3,) + shape)
    s = admm.Solver([phase], MATS, [np.eye(3)], admm.default_params("fp64"), precision="fp64")
    s.set_state(0, F=F)
    g = s.bloch(0, omega, 30.0, p0, tol=0.0, max_iter=iters)
    s.close()
    o = O.bloch(phase, omats(MATS), F, omega, 30.0, p0, tol=0.0, max_iter=iters)
    assert g["iters"] == iters and g["status"] == admm.NOT_CONVERGED
    scale = max(1.0, abs(o["beta"]))
    print("  beta", g["beta"], o["beta"], "mode", rel(g["p"], o["p"]), flush=True)
    assert abs(g["beta"] - o["beta"]) <= 1e-9 * scale
    assert abs(g["sigma_rho"] - o["sigma_rho"]) <= 1e-9 * scale
    assert rel(g["p"], o["p"]) <= 1e-7
