"""A checkpoint written from memory that is not the GPU's (pinned host memory
here, which any route can read): the same populations as from the GPU's."""

import ctypes

import numpy as np
import pytest

import workloads as wl
from tests._cases import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2108_04435_amd as vlb  # noqa: E402


@pytest.mark.parametrize("precision", ["f64", "f32", "f16"])
def test_state_from_pinned_memory(precision):
    dims = (12, 10, 14)
    say("state from host memory", precision)
    run = vlb.Run(wl.lattice_preset(*dims, precision=precision), wl.vortex_preset(), 16)
    host = torch.empty(run.state_bytes(), dtype=torch.uint8, pin_memory=True).random_(0, 256)
    run._check(run.lib.vlb_write_state(run.h, ctypes.c_void_p(host.data_ptr()), 5))
    got, step = run.read_state()
    assert step == 5
    np.testing.assert_array_equal(got.cpu().numpy(), host.numpy())
    run.write_state(host.cuda(), 7)
    np.testing.assert_array_equal(run.read_state()[0].cpu().numpy(), host.numpy())
    run.close()
