"""Every phase of the topology in one workgroup with work to do: deletions,
midpoints, reconnections and vanishing loops in the same steps, with up to as
many points as one round of the block takes and with more, against the kernels
of larger runs (bit for bit, as a capacity on either side of the limit selects
them) and the stand-alone topology; and steps whose midpoints or reconnection
candidates do not fit.

The filaments are all but at rest, so that the first step's decisions are those
of the topology applied to the seeded points."""

import numpy as np
import pytest

import workloads as wl
from tests._cases import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2108_04435_amd as vlb  # noqa: E402

DIMS, WALLS = (48, 40, 44), (False, True, False)


def uneven_rings(n_rings, seed):
    """Rings whose segments are 0.35 to 1.4 long and, every third, 0.2 to 0.75
    (remeshing keeps 0.7 to 0.95), two rings of opposite sense 0.5 apart, and a
    loop too short to stay."""
    rng = np.random.default_rng(seed)
    loops = [wl.ring((24.0, 20.0, 30.0), 5.0, (0.0, 0.0, 1.0), 36),
             wl.ring((24.1, 20.0, 30.5), 5.0, (0.0, 0.0, -1.0), 36)]
    for k in range(n_rings):
        R = rng.uniform(4.0, 8.0)
        m = int(round(2 * np.pi * R / (0.47 if k % 3 == 0 else 0.85)))
        c = [rng.uniform(0.0, DIMS[0]), rng.uniform(R + 1.0, DIMS[1] - 2.0 - R),
             rng.uniform(0.0, DIMS[2])]
        n = wl.random_unit(rng)
        th = 2 * np.pi * (np.arange(m) + rng.uniform(-0.3, 0.3, m)) / m
        e1 = np.cross(n, np.eye(3)[int(np.argmin(np.abs(n)))])
        e1 /= np.linalg.norm(e1)
        e2 = np.cross(n, e1)
        p = np.array(c) + R * (np.cos(th)[:, None] * e1 + np.sin(th)[:, None] * e2)
        loops.append((p, (np.arange(m) + 1) % m))
    loops.append(wl.ring((24.0, 20.0, 22.0), 0.55, (0, 0, 1), 4))
    pos, nxt = wl.concat_loops(loops)
    for a in (0, 2):
        pos[:, a] = np.mod(pos[:, a], DIMS[a])
    return pos, nxt


def _run(pos, nxt, cap, recon_cap=1 << 16, dims=DIMS, walls=WALLS, **vor):
    """A run all but at rest (velocities of 1e-8).  With wall images no capacity
    in question takes the fused stages."""
    vor = dict(dict(kappa=1e-8, wall_images=True), **vor)
    run = vlb.Run(wl.lattice_preset(*dims, walls=walls, precision="f64"), wl.vortex_preset(**vor),
                  cap, recon_cap=recon_cap)
    rho, u = wl.velocity_field(3, dims, (0.0, 0.0, 0.0), 0.0)
    run.write_fields(rho, u)
    run.seed(pos, nxt)
    return run


@pytest.mark.parametrize("reconnect", [True, False])
@pytest.mark.parametrize("n_rings", [8, 23])   # within one round of the block, two rounds
def test_phases_equal_grid(n_rings, reconnect):
    pos, nxt = uneven_rings(n_rings, 900 + n_rings)
    n = pos.shape[0]
    say("topology phases", n_rings, reconnect, n, "points")
    assert n < 900 if n_rings == 8 else 1100 < n < 1900
    ref = _run(pos, nxt, 2049, reconnect=reconnect)
    stats = ref.apply_topology()
    say(stats)
    assert stats["deleted"] >= 20 and stats["inserted"] > 20 and stats["loops_removed_pts"] >= 4
    assert not reconnect or stats["reconnections"] > 2
    p_ref, k_ref = ref.read_filaments()
    ref.close()
    runs = [_run(pos, nxt, cap, reconnect=reconnect) for cap in (2048, 2049)]
    for step in range(4):
        out = []
        for run in runs:
            run.step(1)
            run.sync()
            out.append(run.read_filaments())
        np.testing.assert_array_equal(out[0][1], out[1][1])
        np.testing.assert_array_equal(out[0][0], out[1][0])
        if step == 0:
            np.testing.assert_array_equal(out[0][1], k_ref)
            np.testing.assert_allclose(out[0][0], p_ref, rtol=0, atol=1e-6)
    for run in runs:
        run.close()


@pytest.mark.parametrize("reconnect", [True, False])
@pytest.mark.parametrize("rings,cap,images", [(1, 60, False), (1, 60, True), (25, 1400, True),
                                              (40, 2048, True), (40, 2049, True)])
def test_midpoints_do_not_fit(rings, cap, images, reconnect):
    """Segments of 1.2: a midpoint each, for which the capacity has no room."""
    # (rings above one another, further apart than reconnection reaches)
    loops = [wl.ring((24.0, 20.0, 1.1 * k), 7.64, (0.0, 0.0, 1.0), 40) for k in range(rings)]
    pos, nxt = wl.concat_loops(loops)
    n = pos.shape[0]
    assert n <= cap < 2 * n
    say("midpoints", n, "points, capacity", cap, images, reconnect)
    run = _run(pos, nxt, cap, reconnect=reconnect, wall_images=images)
    for _ in range(2):   # and again, from the state that is kept
        with pytest.raises(vlb.VlbError) as ei:
            run.step(1)
            run.sync()
        assert ei.value.code == vlb.VLB_ECAPACITY
        p, k = run.read_filaments()
        np.testing.assert_array_equal(k, nxt)
        np.testing.assert_allclose(p, pos, rtol=0, atol=1e-5)
    run.close()


def _bundle(n_b, nz=20, L=16.0):
    """A line along +z and n_b lines along -z at 0.4 around it: every point of
    the first has an exchange candidate on each of the others."""
    z = (np.arange(nz) + 0.5) * L / nz
    pos, nxt = [np.stack([np.full(nz, 8.0), np.full(nz, 8.0), z], 1)], [(np.arange(nz) + 1) % nz]
    for m in range(n_b):
        a = 2 * np.pi * m / n_b
        pos.append(np.stack([np.full(nz, 8.0 + 0.4 * np.cos(a)), np.full(nz, 8.0 + 0.4 * np.sin(a)),
                             z], 1))
        nxt.append((m + 1) * nz + (np.arange(nz) - 1) % nz)
    return np.concatenate(pos), np.concatenate(nxt)


@pytest.mark.parametrize("cap", [400, 2048, 2049])
@pytest.mark.parametrize("lines,recon_cap", [(9, 1 << 14), (2, 4)])   # slots, the step's list
def test_candidates_do_not_fit(lines, recon_cap, cap):
    pos, nxt = _bundle(lines)
    say("candidates", lines, recon_cap, cap)
    run = _run(pos, nxt, cap, recon_cap, dims=(16, 16, 16), walls=(False,) * 3, wall_images=False,
               reconnect=True, remesh=False)
    for _ in range(2):
        with pytest.raises(vlb.VlbError) as ei:
            run.step(1)
            run.sync()
        assert ei.value.code == vlb.VLB_ECAPACITY
        _, k = run.read_filaments()
        np.testing.assert_array_equal(k, nxt)
    run.close()
    # with room for all of them the same step reconnects
    pos, nxt = _bundle(2)
    run = _run(pos, nxt, cap, 1 << 14, dims=(16, 16, 16), walls=(False,) * 3, wall_images=False,
               reconnect=True, remesh=False)
    run.step(1)
    run.sync()
    assert not np.array_equal(run.read_filaments()[1], nxt)
    run.close()
