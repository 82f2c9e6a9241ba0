"""A void fraction that moves between walls in x, and one that is held on a
lattice built for a moving one (with solid nodes too): tiles of small lattices
and row sweeps (an explicit launch shape selects them) are then other instances
of the kernels, with mirrored lanes beyond the walls only in the sweep.  Equal
bit for bit, and one step of the sweep against the FP64 oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_2409_02964_amd import workloads as W  # noqa: E402

RATES = dict(s_c=1.2, s_e=1.2, s_eps=1.2, s_q=1.2, s_nu=0.8)


def torch_of():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def fields(nx, ny):
    y, x = np.mgrid[0:ny, 0:nx]
    phis = [0.6 + 0.3 * np.sin(2 * np.pi * (x - 0.1 * t) / nx) * np.cos(2 * np.pi * (y + 0.2 * t) / ny)
            for t in range(6)]
    rng = np.random.default_rng(2)
    return phis, [(1e-5 * rng.standard_normal((ny, nx)), 1e-5 * rng.standard_normal((ny, nx))) for _ in range(6)]


def lattice(nx, ny, precision, bc_x, bc_y, options, swept, spp=1):
    from paper_2409_02964_amd.vanse import Lattice
    lat = Lattice(nx, ny, precision=precision, bc_x=bc_x, bc_y=bc_y, force_field="force" in options,
                  drag="drag" in options, mask="mask" in options, dynamic_phi=True)
    lat.set_params(0.3, RATES).set_body_force(2e-5, -1e-5).set_steps_per_pass(spp)
    return lat.set_tiling(64, 7) if swept else lat


# smaller than a tile, with remainders, and several tiles
@pytest.mark.parametrize("nx,ny", [(2, 3), (30, 21), (61, 43)])
@pytest.mark.parametrize("precision", ["f64", "f32", "f32s", "f16s"])
@pytest.mark.parametrize("bc_y", ["periodic", "wall"])
@pytest.mark.parametrize("options", ["", "drag", "force drag"])
@pytest.mark.parametrize("spp", [1, 2])
def test_moving_between_x_walls(nx, ny, precision, bc_y, options, spp):
    torch = torch_of()
    phis, force = fields(nx, ny)
    f = W.random_populations(nx, ny, seed=5)

    def run(swept):
        lat = lattice(nx, ny, precision, "wall", bc_y, options, swept, spp).set_void_fraction(phis[0])

        def current(t):
            if "drag" in options:
                lat.set_drag(phis[t] * (1 - phis[t]), (1e-2, 0.0))
            if "force" in options:
                lat.set_force_field(*force[t])

        current(0)
        lat.set_populations(f)
        out = []
        for t, how in ((0, "next"), (1, "pair"), (3, "singly"), (5, "held")):
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


@pytest.mark.parametrize("precision", ["f64", "f32", "f32s", "f16s"])
@pytest.mark.parametrize("bc_x", ["periodic", "wall"])
@pytest.mark.parametrize("bc_y", ["periodic", "wall"])
@pytest.mark.parametrize("options", ["mask", "mask drag", "mask force drag"])
def test_held_with_solid_nodes(precision, bc_x, bc_y, options):
    torch = torch_of()
    out = []
    for nx, ny, steps in ((22, 10, 5), (61, 43, 9)):
        phis, force = fields(nx, ny)
        f = W.random_populations(nx, ny, seed=5)
        out = []
        for swept in (False, True):
            lat = lattice(nx, ny, precision, bc_x, bc_y, options, swept)
            lat.set_mask(W.solid_mask(nx, ny, seed=ny)).set_void_fraction(phis[0])
            if "drag" in options:
                lat.set_drag(phis[0] * (1 - phis[0]), (1e-2, 0.0))
            if "force" in options:
                lat.set_force_field(*force[0])
            lat.set_populations(f).step(steps)
            a = lat.read_populations()
            # (a hand-over takes the sweep on either)
            lat.set_void_fraction_next(phis[1]).step(1).step(3)
            out.append((a, lat.read_populations()))
        for a, b in zip(*out):
            assert torch.isfinite(a).all()
            assert torch.equal(a, b), (nx, ny, (a - b).abs().max().item())


@pytest.mark.parametrize("bc_y", ["periodic", "wall"])
@pytest.mark.parametrize("options", ["", "force drag"])
@pytest.mark.parametrize("shape", [(64, 7), (256, 3), (128, 64)])
def test_one_swept_step_against_the_oracle(oracle, bc_y, options, shape):
    """The bound is that of the same step by the tile kernel (test_gpu_xwalls)."""
    torch = torch_of()
    nx, ny = 50, 30
    phis, force = fields(nx, ny)
    f = W.random_populations(nx, ny, seed=5)
    beta = phis[0] * (1 - phis[0])
    ora = oracle.Oracle(nx, ny, phis[0], kappa=0.3, rates=RATES, g=(2e-5, -1e-5), bc_x="wall", bc_y=bc_y,
                        force=force[0] if "force" in options else None,
                        drag=(beta, (1e-2, 0.0)) if "drag" in options else None)
    ora.set_populations(f)
    ora.step(1, phi_next=phis[2])
    lat = lattice(nx, ny, "f64", "wall", bc_y, options, False).set_tiling(*shape).set_void_fraction(phis[0])
    if "drag" in options:
        lat.set_drag(beta, (1e-2, 0.0)).set_force_field(*force[0])
    lat.set_populations(torch.from_numpy(f)).set_void_fraction_next(phis[2]).step(1)
    err = np.max(np.abs(lat.read_populations().cpu().numpy() - ora.f)) / np.max(np.abs(ora.f))
    assert err <= 1e-14, err
