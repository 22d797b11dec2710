"""Reading and writing the populations in the natural layout: any pattern of
bytes comes back, from buffers that start on 16 bytes and ones that start on
one value only, with sizes that 16 does not divide, and below and above the
size from which accesses are non-temporal."""

import ctypes

import pytest

import workloads as wl
from tests._cases import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2108_04435_amd as vlb  # noqa: E402


@pytest.mark.parametrize("dims,precision", [
    ((5, 7, 9), "f16"), ((5, 7, 9), "f32"), ((5, 7, 9), "f64"), ((33, 31, 17), "f16"),
    ((64, 64, 64), "f32"), ((256, 256, 96), "f16")])
@pytest.mark.parametrize("read_off", [0, 1])
@pytest.mark.parametrize("write_off", [0, 1])
def test_state_round_trip(dims, precision, read_off, write_off):
    say("state copy", dims, precision, read_off, write_off)
    size = {"f16": 2, "f32": 4, "f64": 8}[precision]
    run = vlb.Run(wl.lattice_preset(*dims, precision=precision), wl.vortex_preset(), 16)
    n = run.state_bytes()
    src = torch.randint(0, 256, (n + size,), dtype=torch.uint8, device="cuda")
    dst = torch.full((n + 3 * size,), 77, dtype=torch.uint8, device="cuda")
    a, b = src[write_off * size:][:n], dst[read_off * size:][:n]
    torch.cuda.synchronize()
    run._check(run.lib.vlb_write_state(run.h, ctypes.c_void_p(a.data_ptr()), 0))
    run._check(run.lib.vlb_read_state(run.h, ctypes.c_void_p(b.data_ptr())))
    assert torch.equal(a, b)
    assert bool((dst[:read_off * size] == 77).all()) and bool((dst[read_off * size + n:] == 77).all())
    run.close()
