"""The topology of a step in one workgroup (runs of at most 2048 points of
capacity) against the kernels of larger runs: the same runs at a capacity on
either side of the limit give the same filaments, bit for bit, over steps
with remeshing, reconnection and small-loop removal, down to no points.  (With
wall images both take the same kernels for everything but the topology: the
limit of the fused stages counts the image copies.)"""

import numpy as np
import pytest

import workloads as wl
from tests._cases import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2108_04435_amd as vlb  # noqa: E402


def _steps(cfg, cap, steps):
    run = vlb.Run(cfg["lattice"], cfg["vortex"], cap)
    run.write_fields(cfg["rho"], cfg["u"])
    run.seed(cfg["pos"], cfg["nxt"])
    out = []
    for _ in range(steps):
        run.step(1)
        run.sync()
        out.append(run.read_filaments())
    run.close()
    return out


@pytest.mark.parametrize("remesh", [True, False])
@pytest.mark.parametrize("reconnect", [True, False])
@pytest.mark.parametrize("n_rings", [1, 6, 14])
def test_block_equals_grid(n_rings, reconnect, remesh):
    dims, walls = (48, 40, 44), (False, True, False)
    pos, nxt = wl.random_rings(77 + n_rings, n_rings, 2.0, 9.0, dims, walls, 0.8)
    # a ring about to vanish and one too finely resolved
    a, b = wl.ring((24.0, 20.0, 22.0), 0.55, (0, 0, 1), 5), wl.ring((9.0, 9.0, 9.0), 3.0, (0, 1, 0), 70)
    pos, nxt = wl.concat_loops([(pos, nxt), a, b])
    rho, u = wl.velocity_field(3, dims, (0.0, 0.0, 0.02), 1e-3)
    cfg = dict(lattice=wl.lattice_preset(*dims, walls=walls, precision="f64"),
               vortex=wl.vortex_preset(reconnect=reconnect, remesh=remesh, kappa=0.3,
                                       wall_images=True),
               rho=rho, u=u, pos=pos, nxt=nxt)
    say("topology", n_rings, reconnect, remesh, pos.shape[0], "points")
    for (p0, k0), (p1, k1) in zip(_steps(cfg, 2048, 5), _steps(cfg, 2049, 5)):
        np.testing.assert_array_equal(k0, k1)
        np.testing.assert_array_equal(p0, p1)


@pytest.mark.parametrize("remesh", [True, False])
@pytest.mark.parametrize("cap", [256, 257, 512, 513, 1400])   # 256, 512, 512, 1024, 1024 threads
def test_block_sizes(cap, remesh):
    """Walls on two axes: nine image copies, so that no capacity here takes
    the fused stages.  The sum's chunk count depends on the capacity (3 here, 8
    at 2049), so that the line velocities differ in the order of their parts:
    1e-15 of velocities of order one, and positions of up to 48 by a few ulp
    (7e-15) per step; links are equal, positions to 1e-12 after the first step."""
    dims, walls = (48, 40, 44), (True, True, False)
    ring = wl.ring((24.0, 20.0, 22.0), 7.0, (0.3, 0.2, 1.0), 50)
    a, b = wl.ring((12.0, 30.0, 12.0), 0.55, (0, 0, 1), 5), wl.ring((12.0, 10.0, 9.0), 3.0, (0, 1, 0), 70)
    pos, nxt = wl.concat_loops([ring, a, b])
    rho, u = wl.velocity_field(3, dims, (0.0, 0.0, 0.02), 1e-3)
    cfg = dict(lattice=wl.lattice_preset(*dims, walls=walls, precision="f64"),
               vortex=wl.vortex_preset(remesh=remesh, kappa=0.3, wall_images=True),
               rho=rho, u=u, pos=pos, nxt=nxt)
    say("topology sizes", cap, remesh, pos.shape[0], "points")
    a, b = _steps(cfg, cap, 5), _steps(cfg, 2049, 5)
    np.testing.assert_allclose(a[0][0], b[0][0], rtol=0, atol=1e-12)
    for (_, k0), (_, k1) in zip(a, b):
        np.testing.assert_array_equal(k0, k1)


def test_block_to_no_points():
    dims = (24, 24, 24)
    pos, nxt = wl.ring((12.0, 12.0, 12.0), 0.5, (0, 0, 1), 4)   # shorter than a loop may be
    rho, u = wl.velocity_field(3, dims, (0.0, 0.0, 0.0), 0.0)
    cfg = dict(lattice=wl.lattice_preset(*dims, precision="f64"),
               vortex=wl.vortex_preset(reconnect=True), rho=rho, u=u, pos=pos, nxt=nxt)
    for cap in (64, 512, 1024, 2048, 2049):
        out = _steps(cfg, cap, 3)
        assert [p.shape[0] for p, _ in out] == [0, 0, 0]
