"""Every tile width that admm_set_tuning accepts launches Step 2 within 64 KiB of
LDS per workgroup, for every length along x2 and x3, and in plane strain, where
the pass along x2 takes the x3 pass's tile width. On the host, by the launches'
own LDS sizes; on the GPU the projection of the widest plane tile against the
oracle, with the parity tests' bounds."""
import pytest

import host_only

CODE = """
LENGTHS = [4, 6, 8, 12, 16, 18, 24, 32, 36, 48, 54, 64, 72, 96, 108, 128, 144, 162, 192, 216, 256]
worst = 0
for precision, d in ((admm.FP64, 8), (admm.FP32_FP64RED, 16)):
    for n in LENGTHS:
        for shape in ((1, n, 4), (4, n, 4), (n, 4, 4)):
            rc, ctx = init([shape], precision)
            assert rc == admm.OK
            for t in (d // 4, d // 2, d, 2 * d):
                try:
                    admm.admm_set_tuning(ctx, t if shape[1] == n and shape[0] > 1 else d,
                                         t if shape[1] == 4 or shape[0] == 1 else d, 256)
                except admm.AdmmError as e:
                    assert e.code == admm.EINVAL
                    assert 2 * n * t * 128 // d > 65536 and shape[0] != 1, (shape, t)
                    continue
                fake.fake_reset(UNLIMITED)
                admm.admm_project_step(ctx)
                lds = fake.fake_lds_most()
                assert fake.fake_launches() > 0
                if lds > worst:
                    worst = lds
                    print(precision, shape, t, lds, flush=True)
                assert lds <= 65536, (precision, shape, t, lds)
            admm.admm_destroy(ctx)
            keep.clear()
"""


def test_tiles_stay_within_the_lds(tmp_path):
    host_only.run(CODE, tmp_path)


@pytest.mark.gpu
@pytest.mark.parametrize("precision,tile", [("fp64", 16), ("fp32", 32)])
def test_widest_plane_tile_projects(precision, tile):
    import numpy as np

    import oracle as O
    from paper_2010_06697_amd import microstructure as M
    from parity_util import gpu_solver, random_state, rel
    shape = (1, 256, 36)
    print("projection", precision, shape, "tile", tile, flush=True)
    u, F, L = random_state(shape, seed=5)
    s = gpu_solver([np.zeros(shape, np.uint8)], [M.neohooke(1.0, 4.0)], [np.eye(3)], precision,
                   rho0=2.5)
    s.set_tuning(tile // 2, tile, 256)
    s.set_state(0, u=0 * u, F=F, Lambda=L)
    s.project_step()
    got = s.state(0)["u_prev"]
    s.close()
    assert rel(got, O.project(F - L / 2.5)) <= (1e-12 if precision == "fp64" else 2e-5)
