"""The tile kernel of small lattices against the row sweep (an explicit launch
shape selects it): the same arithmetic and the same storage roundings, so the
populations are equal bit for bit, at tile edges, on lattices smaller than a
tile, and for step counts that leave remainders."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_2409_02964_amd import workloads as W  # noqa: E402

RATES = dict(s_c=1.2, s_e=1.2, s_eps=1.2, s_q=1.2, s_nu=0.8)


def lattice(nx, ny, precision, bc_x, bc_y, options):
    from paper_2409_02964_amd.vanse import Lattice
    phi = W.channel_phi(nx, ny, seed=nx, noise=0.0 if min(nx, ny) < 8 else 0.05)
    lat = Lattice(nx, ny, precision=precision, bc_x=bc_x, bc_y=bc_y, force_field="force" in options,
                  drag="drag" in options, mask="mask" in options)
    lat.set_params(0.5, RATES).set_body_force(2e-5, -1e-5)
    if "mask" in options:
        lat.set_mask(W.solid_mask(nx, ny, seed=ny))
    lat.set_void_fraction(phi)
    if "force" in options:
        rng = np.random.default_rng(1)
        lat.set_force_field(1e-5 * rng.standard_normal((ny, nx)), 1e-5 * rng.standard_normal((ny, nx)))
    if "drag" in options:
        lat.set_drag(1e-3 + 2e-2 * (1 - phi), (1e-4, -2e-4))
    return lat


@pytest.mark.parametrize("precision", ["f64", "f32", "f32s", "f16s"])
@pytest.mark.parametrize("bc_x,bc_y", [("periodic", "periodic"), ("periodic", "wall"), ("wall", "wall"),
                                       ("wall", "periodic")])
@pytest.mark.parametrize("options", ["", "force", "drag", "force drag", "mask", "mask drag"])
def test_tiles_equal_the_sweep(precision, bc_x, bc_y, options):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    # one tile and less, tile_out(32, 2..4) = 22, 16, 10 and one beyond, wide
    # and tall ones, and several rounds of tiles (two steps per launch)
    for nx, ny, steps in [(2, 2, 5), (3, 9, 4), (10, 22, 9), (23, 17, 6), (64, 11, 7), (9, 200, 10), (400, 390, 4)]:
        if "mask" in options and min(nx, ny) < 5:
            continue
        f = torch.from_numpy(W.random_populations(nx, ny, seed=5)).cuda()
        tiles = lattice(nx, ny, precision, bc_x, bc_y, options)
        sweep = lattice(nx, ny, precision, bc_x, bc_y, options).set_tiling(64, 7)
        for n in (steps, 1, 2):
            a = tiles.set_populations(f).step(n).read_populations()
            b = sweep.set_populations(f).step(n).read_populations()
            assert tiles.t == sweep.t == n
            assert torch.isfinite(a).all()
            assert torch.equal(a, b), (nx, ny, n, (a - b).abs().max().item())


def test_captured_steps_can_be_replayed():
    """An even number of steps leaves the state in the buffer that it started
    from, so a captured call advances it at every replay."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    f = torch.from_numpy(W.random_populations(64, 48, seed=5)).cuda()
    lat = lattice(64, 48, "f32s", "periodic", "wall", "drag").set_populations(f)
    ref = lattice(64, 48, "f32s", "periodic", "wall", "drag").set_tiling(64, 7).set_populations(f)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    for n in (2, 6, 10):
        lat.set_populations(f)
        ref.set_populations(f)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=side):
            lat.step(n)
        for k in range(1, 4):
            g.replay()
            ref.step(n)
            torch.cuda.synchronize()
            assert torch.equal(lat.read_populations(), ref.read_populations()), (n, k)


@pytest.mark.parametrize("precision", ["f64", "f32", "f32s", "f16s"])
@pytest.mark.parametrize("bc_y", ["periodic", "wall"])
@pytest.mark.parametrize("options", ["", "force", "drag", "force drag", "mask", "mask drag"])
def test_pairs_equal_the_two_step_sweep(precision, bc_y, options):
    """Two steps per launch: tiles against the two-step sweep (an explicit
    number of rows selects it), pairs, four steps and odd counts."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    for nx, ny, steps in [(2, 2, 5), (11, 9, 4), (22, 23, 8), (64, 45, 6), (400, 390, 4)]:
        if "mask" in options and min(nx, ny) < 5:
            continue
        f = torch.from_numpy(W.random_populations(nx, ny, seed=5)).cuda()
        tiles = lattice(nx, ny, precision, "periodic", bc_y, options).set_steps_per_pass(2)
        sweep = lattice(nx, ny, precision, "periodic", bc_y, options).set_steps_per_pass(2, 5).set_tiling(64, 7)
        for n in (steps, 2, 3):
            a = tiles.set_populations(f).step(n).read_populations()
            b = sweep.set_populations(f).step(n).read_populations()
            assert tiles.t == sweep.t == n
            assert torch.isfinite(a).all()
            assert torch.equal(a, b), (nx, ny, n, (a - b).abs().max().item())


@pytest.mark.parametrize("precision", ["f64", "f32", "f32s", "f16s"])
@pytest.mark.parametrize("bc_y", ["periodic", "wall"])
@pytest.mark.parametrize("options", ["", "drag", "force drag"])
@pytest.mark.parametrize("spp", [1, 2])
def test_moving_void_fraction(precision, bc_y, options, spp):
    """phi, the drag coefficient and the force field handed over step by step
    and in pairs (also stepped singly), tiles against the sweeps."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2409_02964_amd.vanse import Lattice
    nx, ny = 61, 43
    y, x = np.mgrid[0:ny, 0:nx]
    phis = [0.6 + 0.3 * np.sin(2 * np.pi * (x - 0.1 * t) / nx) * np.cos(2 * np.pi * (y + 0.2 * t) / ny)
            for t in range(8)]
    rng = np.random.default_rng(2)
    force = [(1e-5 * rng.standard_normal((ny, nx)), 1e-5 * rng.standard_normal((ny, nx))) for _ in range(8)]
    f = W.random_populations(nx, ny, seed=5)

    def run(swept):
        lat = Lattice(nx, ny, precision=precision, bc_y=bc_y, force_field="force" in options,
                      drag="drag" in options, dynamic_phi=True)
        lat.set_params(0.3, RATES).set_body_force(2e-5, -1e-5).set_steps_per_pass(spp, 5 if swept else 0)
        if swept:
            lat.set_tiling(64, 7)
        lat.set_void_fraction(phis[0])

        def current(t):
            if "drag" in options:
                lat.set_drag(phis[t] * (1 - phis[t]), (1e-2, 0.0))
            if "force" in options:
                lat.set_force_field(*force[t])

        current(0)
        lat.set_populations(f)
        out = []
        for t, how in ((0, "pair"), (2, "singly"), (4, "next"), (5, "held"), (5, "pair")):
            current(t)
            if how == "next":
                lat.set_void_fraction_next(phis[t + 1]).step(1)
            elif how == "held":
                lat.step(5)
            else:
                lat.set_void_fraction_next2(phis[t + 1], phis[t + 2],
                                            phis[t + 1] * (1 - phis[t + 1]) if "drag" in options else None,
                                            force[t + 1] if "force" in options else None)
                if how == "pair":
                    lat.step(2)
                else:
                    lat.step(1).step(1)
            out.append(lat.read_populations())
        return out

    for k, (a, b) in enumerate(zip(run(False), run(True))):
        assert torch.isfinite(a).all()
        assert torch.equal(a, b), (k, (a - b).abs().max().item())


@pytest.mark.parametrize("spp", [1, 2])
@pytest.mark.parametrize("precision", ["f32s", "f16s"])
def test_moving_void_fraction_over_many_nodes(precision, spp):
    """As above over enough nodes and steps to meet values near the middle of
    two FP16 numbers, where rounding twice differs from rounding once."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2409_02964_amd.vanse import Lattice
    nx, ny, steps = 187, 283, 24
    y, x = np.mgrid[0:ny, 0:nx]
    phis = [torch.from_numpy(0.6 + 0.3 * np.sin(2 * np.pi * (x - 0.02 * t) / nx) * np.sin(2 * np.pi * (y - 0.02 * t) / ny)).cuda()
            for t in range(steps + 1)]
    out = []
    for swept in (False, True):
        lat = Lattice(nx, ny, precision=precision, drag=True, dynamic_phi=True).set_params(0.3, RATES)
        lat.set_body_force(1.5e-6, 0.0).set_steps_per_pass(spp, 5 if swept else 0)
        if swept:
            lat.set_tiling(64, 7)
        lat.set_void_fraction(phis[0]).set_drag(phis[0] * (1 - phis[0]), (1e-2, 0.0)).init_equilibrium(1.0, 0.03, 0.015)
        for t in range(0, steps, spp):
            lat.set_drag(phis[t] * (1 - phis[t]), (1e-2, 0.0))
            if spp == 2:
                lat.set_void_fraction_next2(phis[t + 1], phis[t + 2], phis[t + 1] * (1 - phis[t + 1]), None)
            else:
                lat.set_void_fraction_next(phis[t + 1])
            lat.step(spp)
        out.append(lat.read_populations())
    assert torch.isfinite(out[0]).all()
    assert torch.equal(*out)
