"""Force spreading of forces that overflowed: a node's sum is infinite where its
contributions are infinite of one sign, NaN where of both, finite elsewhere, with
few and with many points to a cell."""

import numpy as np
import pytest

import workloads as wl
from oracle import vfm
from oracle.lbm import Lattice
from tests._cases import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2108_04435_amd as vlb  # noqa: E402


@pytest.mark.parametrize("cap", [600, 17000])
@pytest.mark.parametrize("per_cell", [3, 8, 9, 40])
def test_overflowed_forces(per_cell, cap):
    dims = (16, 18, 20)
    lat = Lattice(*dims)
    a = wl.ring((6.5, 7.5, 8.5), 0.45, (0.2, 0.3, 1.0), 4 * per_cell)
    b = wl.ring((8.0, 9.0, 14.0), 4.0, (0.1, 0.2, 1.0), 30)
    pos, nxt = wl.concat_loops([a, b])
    say("overflowed forces", per_cell, cap)
    # velocities of 1e159, finite, times rho_s kappa = 1e320: beyond FP64
    run = vlb.Run(wl.lattice_preset(*dims, precision="f64"),
                  wl.vortex_preset(remesh=False, kappa=1e160, rho_s_over_rho_n=1e160), n_cap=cap)
    rho, u = wl.velocity_field(5, dims, (0.0, 0.0, 0.0), 0.0)
    run.write_fields(rho, u)
    run.seed(pos, nxt)
    out = run.eval_line_velocity()
    assert np.isfinite(out["sdot"]).all() and np.isinf(out["force"]).any()
    F = run.read_force()
    with np.errstate(invalid="ignore"):
        ref = vfm.spread(out["force"], pos, lat)
    assert np.isinf(ref).any()
    np.testing.assert_array_equal(np.isnan(F), np.isnan(ref))
    np.testing.assert_array_equal(F[np.isinf(ref)], ref[np.isinf(ref)])
    ok = np.isfinite(ref)
    np.testing.assert_array_equal(np.isfinite(F), ok)
    run.close()
