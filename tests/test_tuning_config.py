"""What admm_autotune leaves, on the host: the launches of Step 2 (their grids and
LDS sizes, in order) stand for the configuration, and the event timer is scripted.

- A context's reported configuration, set again or restored from a checkpoint,
  is the one it runs.
- Where no candidate is faster than the default, the default stays.
- Radix sequences are tried for the lengths along x1 alone, whose forward pass is
  the one they drive in Step 2: a length of another axis keeps its default, which
  the Bloch wave's transforms use.
"""
import host_only

CONFIG = """
def launches(ctx):
    fake.fake_reset(UNLIMITED)
    admm.admm_project_step(ctx)
    return fake.fake_launches(), fake.fake_shape_hash()


BATCHES = ([(24, 18, 32), (16, 48, 12)], [(64, 64, 64)], [(6, 4, 8), (96, 128, 128)],
           [(1, 64, 48)], [(1, 256, 256)])
for precision in (admm.FP64, admm.FP32_FP64RED):
    for shapes in BATCHES:
        rc, ctx = init(shapes, precision)
        assert rc == admm.OK
        before = launches(ctx)
        cfg = admm.admm_autotune(ctx, 0)
        blob = admm.admm_get_state(ctx)
        admm.admm_set_tuning(ctx, cfg["tile_y"], cfg["tile_z"], cfg["x_points"], cfg["plans"])
        print(precision, shapes, cfg["x_points"], flush=True)
        assert launches(ctx) == before, "reported configuration"
        admm.admm_set_state(ctx, blob)
        assert launches(ctx) == before, "restored configuration"
        fake.fake_event_ms(1.0, 1.0)  # every candidate as fast as the default
        tuned = admm.admm_autotune(ctx, 1)
        assert launches(ctx) == before, "tuned without a gain"
        assert tuned["plans"] == cfg["plans"]
        admm.admm_destroy(ctx)
        keep.clear()
"""


def test_the_default_is_a_configuration(tmp_path):
    host_only.run(CONFIG, tmp_path)


PLANS = """
for precision in (admm.FP64, admm.FP32_FP64RED):
    for shapes in ([(36, 48, 64), (18, 48, 64)], [(1, 72, 96)]):
        rc, ctx = init(shapes, precision)
        assert rc == admm.OK
        cfg = admm.admm_autotune(ctx, 0)
        fake.fake_event_ms(1000.0, 0.999)  # every candidate faster than the last
        tuned = admm.admm_autotune(ctx, 1)
        x1 = {s[2] for s in shapes}
        print(precision, cfg["plans"], tuned["plans"], flush=True)
        for n, radices in tuned["plans"].items():
            assert (radices != cfg["plans"][n]) == (n in x1), n
        admm.admm_destroy(ctx)
"""


def test_radix_plans_are_timed_where_they_run(tmp_path):
    host_only.run(PLANS, tmp_path)
