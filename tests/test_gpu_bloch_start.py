"""Bloch waves from structured start modes: one Fourier mode of a homogeneous cell,
so that the right-hand side of the secular equation holds nothing but rounding at
the smallest |K|^2 and its root lies at that end of the range. The iterations run
on to a fixed point. Which eigenvalue they find from such a start is rounding's
choice, but one it is: the cell's are mu |K|^2 (twice) and (2 mu + lambda) |K|^2
over its modes, K_j = sin(2 pi m_j / n_j + omega_j) (1e-9 relative, as in the other
Bloch tests).
"""
import numpy as np
import pytest

from paper_2010_06697_amd import admm, microstructure as M

pytestmark = pytest.mark.gpu

MATS = [M.neohooke(10.0, 40.0), M.neohooke(1.0, 4.0)]


@pytest.mark.parametrize("shape,omega", [((8, 8, 8), (0.0, 0.0, 0.0)), ((8, 8, 8), (0.1, 0.0, 0.0)),
                                         ((12, 16, 18), (0.3, 0.2, 0.1)),
                                         ((1, 16, 24), (np.pi / 8, 0.0, 0.0))])
def test_bloch_from_one_fourier_mode(shape, omega):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("bloch from one mode", shape, omega, flush=True)
    phase = np.zeros(shape, np.uint8)
    p0 = np.zeros((3,) + shape, complex)
    p0[1] = np.exp(4j * np.pi * np.arange(shape[2]) / shape[2])
    s = admm.Solver([phase], MATS, [np.eye(3)], admm.default_params("fp64"), precision="fp64")
    for n in (1, 5, 400):
        g = s.bloch(0, omega, 80.0, p0, tol=1e-9, max_iter=n)
        print("  ", n, g["beta"], g["sigma_rho"], g["iters"], g["status"], flush=True)
        assert np.isfinite(g["p"]).all() and np.isfinite(g["beta"])
    s.close()
    assert g["status"] == admm.OK
    assert abs(g["beta"] - g["sigma_rho"]) <= 1e-9 * max(1.0, abs(g["beta"]))
    K = [np.sin(2 * np.pi * np.arange(n) / n + w) ** 2 for n, w in zip(shape[::-1], omega)]
    k2 = (K[0][:, None, None] + K[1][None, :, None] + K[2][None, None, :]).ravel()
    eigenvalues = np.concatenate([10.0 * k2, (2 * 10.0 + 40.0) * k2])
    assert np.abs(eigenvalues - g["beta"]).min() <= 1e-9 * max(1.0, abs(g["beta"]))
