"""Small runs on one stream, whose later stages carry the spreading, the
lattice update and the moments in blocks of their own, against the same run
with one launch for each (a timed run): the same bits over several steps, for
every number of stages, flow axis, precision and parity."""

import numpy as np
import pytest

import workloads as wl
from tests._cases import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2108_04435_amd as vlb  # noqa: E402


def _end(dims, walls, precision, vortex, timed, calls, cap):
    lattice = wl.lattice_preset(*dims, walls=walls, precision=precision)
    pos, nxt = wl.random_rings(5, 3, 2.0, 6.0, dims, walls, 0.8)
    rho, u = wl.velocity_field(3, dims, (0.0, 0.005, 0.02), 1e-3)
    run = vlb.Run(lattice, wl.vortex_preset(**vortex), n_cap=cap)
    run.write_fields(rho, u)
    run.seed(pos, nxt)
    if timed:
        run.set_timing(True, 64)
    for k in calls:
        run.step(k)
    run.sync()
    out = run.read_filaments() + (run.read_state()[0].cpu().numpy(), run.read_force())
    run.close()
    return out


@pytest.mark.parametrize("precision", ["f64", "f32", "f16"])
@pytest.mark.parametrize("dims,walls", [((32, 32, 32), (False, False, False)),
                                        ((26, 40, 31), (True, True, False)),
                                        ((24, 24, 41), (False, False, True)),
                                        ((300, 24, 20), (False, False, False))])
@pytest.mark.parametrize("vortex", [
    dict(), dict(mass_balance=True), dict(mass_balance=True, mass_balance_axis=0),
    dict(rk_stages=2, mass_balance=True), dict(rk_stages=1), dict(rk_stages=2, vfm_substeps=3),
    dict(coupling=False)])
@pytest.mark.parametrize("cap", [300, 1500])
def test_carried_equals_launched(dims, walls, precision, vortex, cap):
    axis = vortex.get("mass_balance_axis", 2)
    if vortex.get("mass_balance") and walls[axis]:
        pytest.skip("the flow axis is periodic")
    say("carry", dims, walls, precision, vortex, cap)
    calls = (1, 2, 4)
    for a, b in zip(_end(dims, walls, precision, vortex, False, calls, cap),
                    _end(dims, walls, precision, vortex, True, calls, cap)):
        np.testing.assert_array_equal(a, b)
