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
