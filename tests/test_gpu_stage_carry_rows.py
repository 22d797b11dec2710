"""Small runs on FP16 lattices of 256-node rows: the update that a stage carries
goes node by node, the one launched by itself four nodes to a lane; the same
bits over both parities, with and without walls beyond z, up to the
largest lattice of a run on one stream."""

import numpy as np
import pytest

from tests._cases import say
from tests.test_gpu_stage_carry import _end

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,walls", [((256, 24, 20), (False, False, False)),
                                        ((256, 17, 22), (False, False, True)),
                                        ((256, 84, 83), (False, False, False))])
@pytest.mark.parametrize("vortex", [dict(mass_balance=True, mass_balance_axis=0),
                                    dict(rk_stages=2), dict(coupling=False)])
def test_carried_rows_equal_launched(dims, walls, vortex):
    say("carry rows", dims, walls, vortex)
    calls = (1, 2, 4)
    for a, b in zip(_end(dims, walls, "f16", vortex, False, calls, 300),
                    _end(dims, walls, "f16", vortex, True, calls, 300)):
        np.testing.assert_array_equal(a, b)
