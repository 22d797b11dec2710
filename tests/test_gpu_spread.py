"""Force spreading with crowded cells: bins of more points than the gather
takes in order (it then adds exactly, in integers), beside ordinary ones,
against the oracle's spreading; repeated evaluations give the same bits, and
a second, sparser state leaves no force behind at the nodes of the first."""

import numpy as np
import pytest

import workloads as wl
from oracle import vfm
from oracle.lbm import Lattice
from tests._cases import rel_l2, say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2108_04435_amd as vlb  # noqa: E402

# FP64: a node adds up to some hundred products of four factors; FP32: the
# same forces rounded once to single precision
TOL = {"f64": 1e-12, "f32": 2e-6}


def _crowded(per_cell):
    """A small ring of 4 x per_cell points spanning about four cells, and two
    ordinary rings."""
    a = wl.ring((9.5, 10.5, 11.5), 0.45, (0.2, 0.3, 1.0), 4 * per_cell)
    b = wl.ring((20.0, 18.0, 12.0), 6.0, (0.0, 1.0, 0.4), 44)
    c = wl.ring((1.0, 2.0, 22.0), 5.0, (1.0, 0.1, 0.0), 37)
    return wl.concat_loops([a, b, c])


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("walls", [(False, False, False), (True, False, True)])
@pytest.mark.parametrize("per_cell", [2, 8, 9, 40, 220])
@pytest.mark.parametrize("cap", [1000, 17000])   # a wave per point, a thread per node
def test_crowded_cells(per_cell, walls, precision, cap):
    dims = (30, 26, 28)
    lat = Lattice(*dims, walls=walls)
    pos, nxt = _crowded(per_cell)
    pos = vfm.wrap_positions(pos, lat)
    n = pos.shape[0]
    say("spread", per_cell, walls, precision, n, "points")
    run = vlb.Run(wl.lattice_preset(*dims, walls=walls, precision=precision),
                  wl.vortex_preset(remesh=False), n_cap=cap)
    rho, u = wl.velocity_field(5, dims, (0.01, 0.0, 0.02), 1e-3)
    run.write_fields(rho, u)
    run.seed(pos, nxt)
    out = run.eval_line_velocity()
    F = run.read_force()
    ref = vfm.spread(out["force"], pos, lat)
    err = rel_l2(F, ref)
    say("rel l2", err)
    assert err <= TOL[precision]
    assert not F[ref == 0.0].any()
    run.eval_line_velocity()
    np.testing.assert_array_equal(run.read_force(), F)
    # another state: the first one's nodes are zero again
    pos2, nxt2 = wl.ring((15.0, 13.0, 14.0), 5.0, (0.3, 0.2, 1.0), 36)
    run.seed(pos2, nxt2)
    out = run.eval_line_velocity()
    F = run.read_force()
    ref = vfm.spread(out["force"], vfm.wrap_positions(pos2, lat), lat)
    assert rel_l2(F, ref) <= TOL[precision]
    assert not F[ref == 0.0].any()
    run.close()
