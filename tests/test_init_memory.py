"""What implicit iterations take on the card never costs a call its room.

admm_init takes a context whenever its tables and the fields of explicit
iterations fit: the fields of implicit iterations (240 bytes a voxel and more)
are an extra that must not take the room of what the context needs. admm_bloch's
work buffers (about 960 bytes a voxel) may take that room back. On the host,
with device memory budgets in between."""
import host_only

CODE = """
for precision, kept, shapes in ((admm.FP64, 0, [(8, 12, 16), (6, 4, 18)]), (admm.FP64, 0, [(1, 36, 32)]),
                                (admm.FP32_FP64RED, 76, [(8, 12, 16), (6, 4, 18)])):
    V = sum(a * b * c for a, b, c in shapes)
    fake.fake_reset(UNLIMITED)
    rc, ctx = init(shapes, precision)
    assert rc == admm.OK, rc
    whole, extra = fake.fake_used(), fake.fake_largest()
    admm.admm_destroy(ctx)
    assert fake.fake_used() == 0
    # what the context cannot do without: all but the implicit iterations' fields
    # and, in float, the explicit iterations' own in their place
    need = whole - extra + kept * V
    for k in range(41):
        budget = need + (whole - need) * k // 40 + 4096
        fake.fake_reset(budget)
        rc, ctx = init(shapes, precision)
        print(precision, shapes, budget - need, rc, flush=True)
        assert rc == admm.OK, (precision, shapes, budget, need, whole)
        admm.admm_destroy(ctx)
        assert fake.fake_used() == 0  # nothing left behind on either way
    fake.fake_reset(1000)
    rc, ctx = init(shapes, precision)
    assert rc in (admm.EHIP, admm.ENOMEM) and not ctx.value
    assert fake.fake_used() == 0
"""


def test_init_fits_where_explicit_iterations_fit(tmp_path):
    host_only.run(CODE, tmp_path)


BLOCH = """
shape = (8, 12, 16)
V = 8 * 12 * 16
fake.fake_reset(UNLIMITED)
rc, ctx = init([shape], admm.FP64)
assert rc == admm.OK
used, extra = fake.fake_used(), fake.fake_largest()
p = ctypes.create_string_buffer(48 * V)
fake.fake_reset(UNLIMITED)
admm.admm_bloch(ctx, 0, [0.1, 0.2, 0.3], 20.0, 0.0, 2, ctypes.addressof(p))
work = fake.fake_largest()
admm.admm_destroy(ctx)
for budget in (used + work, used + work - 1, used + work - extra):
    fake.fake_reset(budget)
    rc, ctx = init([shape], admm.FP64)
    assert rc == admm.OK
    print("bloch with", budget - used, "of", work, flush=True)
    admm.admm_bloch(ctx, 0, [0.1, 0.2, 0.3], 20.0, 0.0, 2, ctypes.addressof(p))
    assert fake.fake_used() == (used if budget == used + work else used - extra)
    admm.admm_step(ctx, 2, 1)
    admm.admm_destroy(ctx)
    assert fake.fake_used() == 0
"""


def test_bloch_takes_back_the_room(tmp_path):
    host_only.run(BLOCH, tmp_path)
