"""Default rows per tile of batches: one round of resident workgroups where
tiles of up to 24 rows (31 with two steps per launch) give it.  The rows change
no result, so a batch equals the same lattices in tiles of 20 rows bit for bit."""
import pytest

pytestmark = pytest.mark.gpu

from paper_2409_02964_amd import workloads as W  # noqa: E402

RATES = dict(s_c=1.2, s_e=1.2, s_eps=1.2, s_q=1.2, s_nu=0.8)


# one-row tiles, a few rows, near the last size of one round, beyond it
@pytest.mark.parametrize("sides", [[2, 7], [64, 115, 61], [700, 90, 301], [1400, 1200], [1700, 1500, 5]])
@pytest.mark.parametrize("precision", ["f64", "f32s", "f16s"])
@pytest.mark.parametrize("threads,spp", [(64, 1), (256, 1), (64, 2), (128, 2)])
def test_default_rows(sides, precision, threads, spp):
    import torch
    from paper_2409_02964_amd.vanse import Batch, Lattice
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    out = []
    for rows in (0, 20):
        lats = []
        for L in sides:
            phi = W.periodic_wave(L, L)
            lat = Lattice(L, L, precision=precision, drag=True).set_params(0.5, RATES).set_body_force(2e-6, 1e-6)
            lat.set_steps_per_pass(spp).set_void_fraction(phi).set_drag(1e-2 * phi)
            lats.append(lat.init_equilibrium(1.0, 0.02, 0.01))
        b = Batch(lats, threads=threads, rows=rows, steps_per_pass=spp)
        tiles = b.tiles()
        w = threads - (4 if spp == 1 else 10)
        assert tiles["tiles"] == sum(-(-L // w) * -(-L // tiles["rows"]) for L in sides)
        b.step(3)
        out.append([lat.read_populations() for lat in lats])
        b.close()
    for x, y in zip(*out):
        assert torch.isfinite(x).all()
        assert torch.equal(x, y)
