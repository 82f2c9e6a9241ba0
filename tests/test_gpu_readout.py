"""Read-out and initial state at the edges of the read-out's strips (254
columns) and row blocks, against the FP64 oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_2409_02964_amd import workloads as W  # noqa: E402

RATES = dict(s_c=1.2, s_e=1.2, s_eps=1.2, s_q=1.2, s_nu=0.8)
SHAPES = [(2, 2), (253, 3), (254, 2), (255, 5), (508, 7), (509, 700), (64, 2100)]


@pytest.mark.parametrize("bc_x,bc_y,masked", [("periodic", "periodic", False), ("periodic", "wall", False),
                                              ("wall", "wall", False), ("periodic", "wall", True)])
@pytest.mark.parametrize("nx,ny", SHAPES)
def test_moments_observables_and_populations(oracle, nx, ny, bc_x, bc_y, masked):
    import torch
    from paper_2409_02964_amd.vanse import Lattice
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    if masked and min(nx, ny) < 5:
        pytest.skip("a mask needs room")
    phi = W.channel_phi(nx, ny, seed=nx + ny, noise=0.0 if min(nx, ny) < 8 else 0.05)
    mask = W.solid_mask(nx, ny, seed=nx) if masked else None
    f = W.random_populations(nx, ny, seed=7)
    g, beta = (2e-5, -1e-5), 1e-3 + 2e-2 * (1 - phi)
    lat = Lattice(nx, ny, precision="f64", bc_x=bc_x, bc_y=bc_y, drag=True, mask=masked)
    lat.set_params(0.5, RATES).set_body_force(*g)
    if masked:
        lat.set_mask(mask)
    lat.set_void_fraction(phi).set_drag(beta, (1e-4, 0.0)).set_populations(f)
    o = oracle.Oracle(nx, ny, phi, kappa=0.5, rates=RATES, g=g, bc_x=bc_x, bc_y=bc_y, mask=mask,
                      drag=(beta, (1e-4, 0.0)))
    o.set_populations(f)
    fluid = np.ones((ny, nx), bool) if mask is None else mask == 0
    ref = o.macroscopic()
    got = {k: v.cpu().numpy() for k, v in lat.read_moments().items()}
    # sums of nine values near one and an Eq. (10) gradient of them, each
    # rounded a few times: 64 ulp of the largest value
    tol = 64 * 2.0 ** -52
    for k in ("rho", "ux", "uy"):
        assert np.abs(got[k] - ref[k])[fluid].max() <= tol * max(1.0, np.abs(ref[k][fluid]).max()), k
        assert not got[k][~fluid].any()
    assert np.array_equal(got["p"], got["rho"] / 3.0)
    pops = lat.read_populations().cpu().numpy()
    assert np.abs(pops - f)[:, fluid].max() <= 4 * 2.0 ** -52   # decoded as stored
    assert not pops[:, ~fluid].any()
    obs = lat.observe()
    u2 = (got["ux"] ** 2 + got["uy"] ** 2)[fluid]
    n = int(fluid.sum())
    # FP64 sums of n terms in two orders
    assert abs(obs["mass"] - f[:, fluid].sum()) <= 2.0 ** -52 * n ** 0.5 * 8 * f[:, fluid].sum()
    assert abs(obs["u2"] - u2.sum()) <= 2.0 ** -52 * n ** 0.5 * 8 * u2.sum()
    assert abs(obs["umax"] - np.sqrt(u2.max())) <= 4 * 2.0 ** -52 * obs["umax"]
    assert obs["nonfinite"] == 0 and lat.observe(noalloc=True) == obs
    none, first, bad = lat.residual()
    same, second, _ = lat.residual()
    assert none is None and bad == 0 and same == 0.0 and first == second == obs["u2"]
