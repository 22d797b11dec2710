"""Points between a run and the host where no pinned memory is to be had: the
same results, by copies.  A child process in which every allocation of pinned
memory fails (a stand-in for the runtime's function, loaded before the library)
against this one."""

import os
import shutil
import subprocess
import sys

import numpy as np
import pytest

from tests._cases import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

STANDIN = """
#include <stddef.h>
int vlb_test_refused;
int hipHostMalloc(void** p, size_t n, unsigned flags) {
  (void)n; (void)flags;
  *p = 0;
  ++vlb_test_refused;
  return 2;  /* out of memory */
}
"""


def work():
    """Results of every call that moves points, as a flat dict of arrays."""
    import ctypes

    import paper_2108_04435_amd as vlb
    import workloads as wl

    out = {}
    dims = (24, 20, 28)
    for precision in ("f64", "f32"):
        rho, u = wl.velocity_field(3, dims, (0.0, 0.005, 0.02), 1e-3)
        run = vlb.Run(wl.lattice_preset(*dims, precision=precision), wl.vortex_preset(), 200)
        run.write_fields(rho, u)
        run.seed(np.zeros((0, 3)), np.zeros(0, np.int32))
        out[precision + "none"] = run.read_filaments()[0]
        pos, nxt = wl.ring((12.0, 10.0, 14.0), 5.0, (0.3, 0.2, 1.0), 36)
        run.seed(pos, nxt)
        for k, v in run.eval_line_velocity().items():
            out[precision + k] = v
        m = ctypes.c_int64(0)
        buf = np.full((36, 3), -1.0)
        code = run.lib.vlb_read_filaments(run.h, 35, buf.ctypes.data_as(ctypes.c_void_p), None,
                                          ctypes.byref(m))
        assert code == vlb.VLB_ENOSPACE and m.value == 36 and (buf == -1.0).all()
        run.step(3)
        run.sync()
        out[precision + "pos"], out[precision + "nxt"] = run.read_filaments()
        # latched errors are reported with the points
        run.write_fields(np.full(dims[::-1], np.nan), np.full((3,) + dims[::-1], np.nan))
        run.seed(pos, nxt)
        try:
            run.eval_line_velocity()
            raise AssertionError("no error for a non-finite velocity")
        except vlb.VlbError as e:
            assert e.code == vlb.VLB_ENUMERIC
        run.close()
    return out


CHILD = """
import ctypes, sys
sys.path.insert(0, sys.argv[1])
stand_in = ctypes.CDLL(sys.argv[2], mode=ctypes.RTLD_GLOBAL)
import numpy as np
from tests.test_gpu_no_pinned_memory import work
out = work()
assert ctypes.c_int.in_dll(stand_in, "vlb_test_refused").value > 0
np.savez(sys.argv[3], **out)
"""


def test_points_by_copies(tmp_path):
    gcc = shutil.which("gcc")
    if gcc is None:
        pytest.skip("no C compiler for the stand-in")
    src, lib, res = tmp_path / "s.c", tmp_path / "s.so", tmp_path / "out.npz"
    src.write_text(STANDIN)
    subprocess.run([gcc, "-shared", "-fPIC", "-o", str(lib), str(src)], check=True)
    say("no pinned memory")
    r = subprocess.run([sys.executable, "-c", CHILD, ROOT, str(lib), str(res)],
                       capture_output=True, text=True, timeout=100, cwd=ROOT)
    assert r.returncode == 0, r.stderr[-2000:]
    got, want = np.load(res), work()
    assert sorted(got.files) == sorted(want)
    for k in want:
        np.testing.assert_array_equal(got[k], want[k])
