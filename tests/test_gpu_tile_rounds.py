"""Lattices of more than one round of tiles: calls whose steps go partly to tiles,
two per launch, and singly (by tiles or the sweep) bit for bit as the row sweep
alone, and captured with the number of launches that leaves the state in place."""
import pytest

pytestmark = pytest.mark.gpu

from test_gpu_tile import lattice  # noqa: E402
from paper_2409_02964_amd import workloads as W  # noqa: E402


@pytest.mark.parametrize("precision,nx,ny", [("f64", 300, 290), ("f32", 400, 390), ("f32s", 430, 365), ("f16s", 381, 390)])
@pytest.mark.parametrize("bc_x,bc_y", [("periodic", "periodic"), ("periodic", "wall"), ("wall", "wall")])
@pytest.mark.parametrize("options", ["", "force drag", "mask drag"])
def test_fours_and_the_rest(precision, nx, ny, bc_x, bc_y, options):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    f = torch.from_numpy(W.random_populations(nx, ny, seed=5)).cuda()
    tiles = lattice(nx, ny, precision, bc_x, bc_y, options)
    sweep = lattice(nx, ny, precision, bc_x, bc_y, options).set_tiling(64, 7)
    for n in (2, 3, 4, 5, 6, 7):
        a = tiles.set_populations(f).step(n).read_populations()
        b = sweep.set_populations(f).step(n).read_populations()
        assert tiles.t == sweep.t == n
        assert torch.isfinite(a).all()
        assert torch.equal(a, b), (n, (a - b).abs().max().item())


@pytest.mark.parametrize("precision,nx,ny", [("f64", 300, 290), ("f16s", 381, 390)])
@pytest.mark.parametrize("n", [2, 6, 8])
def test_replays(precision, nx, ny, n):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    f = torch.from_numpy(W.random_populations(nx, ny, seed=5)).cuda()
    lat = lattice(nx, ny, precision, "periodic", "wall", "drag").set_populations(f)
    ref = lattice(nx, ny, precision, "periodic", "wall", "drag").set_tiling(64, 7).set_populations(f)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=torch.cuda.Stream()):
        lat.step(n)
    for k in range(3):
        g.replay()
        ref.step(n)
        torch.cuda.synchronize()
        assert torch.equal(lat.read_populations(), ref.read_populations()), k
