"""What a step launches, on the host-only runtime of hip_stub.c."""
from hip_stub import run


def test_steps_left_over_by_two_step_tiles_take_the_better_single_step(tmp_path):
    """A lattice whose two-step tiles take more than one round: the calls' single
    steps (those that keep the number of launches nsteps modulo two, or all of a
    call of two or three) run as step(1) runs them -- by the sweep where
    one-step tiles are no faster."""
    run(tmp_path, '''
def steps_of(n, *shape):
    h = ready(lattice(*shape), *shape[:2])
    V.check(L.vanse_step(h, n, None))
    assert L.vanse_time(h) == n
    out = []
    for name, blocks, args in launches:
        if "tile_kernel" in name:
            out.append("T%d" % blocks)
        else:
            assert "step_kernel" in name, name
            out.append("s")
    L.vanse_destroy(h)
    return out

tiled = 0
for nx, ny, precision in ((512, 512, "f32"), (450, 450, "f16s"), (400, 400, "f64"), (350, 700, "f64"), (512, 512, "f64")):
    one, four = steps_of(1, nx, ny, precision), steps_of(4, nx, ny, precision)
    assert len(one) == 1 and len(four) in (2, 4)
    tiled += len(four) == 2
    for n in (2, 3, 5, 6, 7, 8, 10):
        got = steps_of(n, nx, ny, precision)
        assert got == four * (n // 4) + one * (n % 4), (nx, ny, precision, n, got, one, four)
assert tiled                         # some of them take two steps per launch
# small lattices: as many steps per launch as leave one round, in nsteps modulo two launches
for n in range(1, 30):
    got = steps_of(n, 64, 64, "f64")
    assert len(got) % 2 == n % 2 and "s" not in got and len(got) <= n // 4 + 2
''')


def test_a_launch_that_fails_late_is_reported_by_its_call(tmp_path):
    run(tmp_path, '''
for nx, spp in ((64, 1), (64, 2), (2000, 1), (2000, 2)):   # tiles and sweeps
    h = ready(lattice(nx, 64), nx, 64)
    V.check(L.vanse_set_steps_per_pass(h, spp, 0))
    fail_launch = lambda name, k: 0
    V.check(L.vanse_step(h, 40, None))
    n = len(launches)
    assert n > 2
    for k in (1, 2, n):
        del launches[:]
        fail_launch = lambda name, i: i == k
        assert L.vanse_step(h, 40, None) == -3, (nx, spp, k)
    fail_launch = lambda name, k: 0
    del launches[:]
''')


def test_tiles_or_sweep_by_rounds(tmp_path):
    """Which kernel a step takes beyond one round of tiles (and single steps): the
    tile kernel where it measured faster, on either side of the limits."""
    run(tmp_path, '''
def kernel(n, nx, ny, precision, bc_x="periodic", bc_y="periodic", spp=1, hand=0, **has):
    h = lattice(nx, ny, precision, bc_x, bc_y, **has)
    if "mask" in has:
        V.check(L.vanse_set_mask(h, field(nx * ny), None))
    if "drag" in has:
        V.check(L.vanse_set_drag(h, field(nx * ny), 0.0, 0.0, None))
    if "force_field" in has:
        V.check(L.vanse_set_force_field(h, field(nx * ny), field(nx * ny), None))
    ready(h, nx, ny)
    V.check(L.vanse_set_steps_per_pass(h, spp, 0))
    if hand:
        args = [field(nx * ny) for _ in range(hand)]
        if hand == 2:
            V.check(L.vanse_set_void_fraction_next2(h, *args, None, None, None, None))
        else:
            V.check(L.vanse_set_void_fraction_next(h, *args, None))
    launches.clear()
    V.check(L.vanse_step(h, n, None))
    kinds = {"tiles" if "tile_kernel" in name else "sweep" for name, _, _ in launches}
    L.vanse_destroy(h)
    keep.clear()
    assert len(kinds) == 1, kinds
    return kinds.pop()

on = dict(mask=1), dict(drag=1), dict(dynamic_phi=1)
mask, drag, dyn = on
for want, args, has in [
    # two steps per launch: time of tiles over that of the sweep
    ("sweep", (60, 123, 1919, "f64", "periodic", "wall"), drag),               # 1.24
    ("sweep", (60, 500, 504, "f64", "periodic", "wall"), drag),                # 1.13
    ("sweep", (60, 560, 552, "f64"), mask),                                    # 1.10
    ("tiles", (60, 380, 390, "f64"), mask),                                    # 0.80
    ("sweep", (60, 500, 499, "f64"), {}),                                      # 1.1
    ("tiles", (60, 340, 340, "f64"), {}),                                      # 0.75
    ("sweep", (60, 740, 740, "f32", "periodic", "periodic"), {}),              # 1.2
    ("tiles", (60, 540, 540, "f32", "periodic", "wall"), {}),                  # 0.78
    ("tiles", (60, 1003, 777, "f16s", "wall", "wall"), drag),                  # 0.72
    ("sweep", (60, 1500, 1500, "f32", "wall", "wall"), drag),                  # 1.0
    ("sweep", (60, 90, 3000, "f64"), dict(mask=1, dynamic_phi=1)),             # 1.24
    ("tiles", (60, 520, 350, "f64"), dict(force_field=1, drag=1)),             # 0.85
    ("sweep", (60, 520, 350, "f64"), drag),                                    # 1.0
    # pairs
    ("sweep", (60, 740, 743, "f32", "periodic", "periodic", 2), mask),         # 1.10
    ("tiles", (60, 640, 640, "f32", "periodic", "periodic", 2), mask),         # 0.8
    ("sweep", (2, 640, 640, "f64", "periodic", "periodic", 2, 2), dyn),        # 1.15
    ("tiles", (2, 440, 440, "f64", "periodic", "periodic", 2, 2), dyn),        # 0.95
    # one step
    ("sweep", (1, 377, 377, "f16s"), {}),                                      # 1.19
    ("tiles", (1, 377, 377, "f16s", "periodic", "wall"), {}),                  # 0.9
    ("sweep", (1, 440, 440, "f64"), {}),                                       # 1.1
    ("tiles", (1, 340, 340, "f64"), {}),                                       # 0.85
    ("sweep", (1, 440, 440, "f64", "periodic", "periodic", 1, 1), dyn),        # 1.05
    ("tiles", (1, 64, 64, "f64", "periodic", "periodic", 1, 1), dyn),          # 0.9
    ("tiles", (1, 287, 934, "f32", "wall", "periodic"), {}),                   # 0.83
]:
    got = kernel(*args, **has)
    assert got == want, (args, has, got)
''')


def test_batches_that_eight_rows_nearly_fill_keep_them(tmp_path):
    run(tmp_path, '''
def rows(sides, precision, threads, spp=1):
    h = [ready(lattice(s, s, precision), s, s) for s in sides]
    a = (C.c_void_p * len(h))(*[x.value for x in h])
    n, b, t, r = C.c_size_t(), C.c_void_p(), C.c_int(), C.c_int()
    V.check(L.vanse_batch_workspace_bytes_ex(a, len(h), threads, 0, spp, C.byref(n)))
    ws = (C.c_char * (n.value + 256))()
    base = (C.addressof(ws) + 255) // 256 * 256
    V.check(L.vanse_batch_create_ex(a, len(h), threads, 0, spp, C.c_void_p(base), n.value, C.byref(b)))
    V.check(L.vanse_batch_tiles(b, C.byref(t), C.byref(r)))
    L.vanse_batch_destroy(b)
    for x in h:
        L.vanse_destroy(x)
    keep.clear()
    return r.value

six = [117, 233, 350, 467, 583, 700]
assert rows(six, "f32", 64) == rows(six, "f32s", 64) == 8
assert rows(six, "f16s", 64) == 6 and rows(six, "f32", 128) < 8 and rows(six, "f64", 64) == 11
assert rows(six, "f32", 64, 2) == 12
assert rows([100, 150], "f32", 64) == 1
''')
