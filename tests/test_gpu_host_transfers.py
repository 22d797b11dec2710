"""Point data between a run and the host on either side of the largest size
that goes through the run's pinned memory (1 MiB with a 64-byte header): what
was seeded comes back bit for bit, and a line velocity read with its four
arrays at once equals the one read array by array."""

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

ROOM = (1 << 20) - 64


def _run(n, cap, precision="f64"):
    dims = (16, 16, 16)
    rng = np.random.default_rng(n)
    # one closed chain of short steps inside the box
    t = 2.0 * np.pi * np.arange(n) / max(n, 1)
    pos = 8.0 + np.stack([5.0 * np.cos(t), 5.0 * np.sin(t), 3.0 * np.sin(7.0 * t)], 1)
    pos = pos.reshape(n, 3) + rng.uniform(-0.5, 0.5, (n, 3))
    run = vlb.Run(wl.lattice_preset(*dims, precision=precision), wl.vortex_preset(kappa=0.1), cap)
    rho, u = wl.velocity_field(3, dims, (0.0, 0.0, 0.02), 1e-3)
    run.write_fields(rho, u)
    run.seed(pos, (np.arange(n) + 1) % max(n, 1))
    return run, pos


@pytest.mark.parametrize("n", [0, 3, 257, ROOM // 32, ROOM // 32 + 1, ROOM // 28, ROOM // 28 + 1])
@pytest.mark.parametrize("precision", ["f64", "f32"])
def test_seed_and_read_back(n, precision):
    say("transfers", n, "points", precision)
    run, pos = _run(n, n + 5, precision)
    assert run.n_points() == n
    got, nxt = run.read_filaments()
    np.testing.assert_array_equal(got, pos)
    np.testing.assert_array_equal(nxt, (np.arange(n) + 1) % max(n, 1))
    m = ctypes.c_int64(0)
    if n:  # no room: the count, and nothing written
        buf = np.full((n, 3), -1.0)
        code = run.lib.vlb_read_filaments(run.h, n - 1, buf.ctypes.data_as(ctypes.c_void_p), None,
                                          ctypes.byref(m))
        assert code == vlb.VLB_ENOSPACE and m.value == n and (buf == -1.0).all()
    run.close()


@pytest.mark.parametrize("n", [5, ROOM // 96, ROOM // 96 + 1])
def test_line_velocity_arrays(n):
    say("line velocity", n, "points")
    run, _ = _run(n, n + 5)
    out = run.eval_line_velocity()
    for i, k in enumerate(("vs", "vn", "sdot", "force")):
        one = np.zeros((n, 3))
        ptrs = [None] * 4
        ptrs[i] = one.ctypes.data_as(ctypes.c_void_p)
        run._check(run.lib.vlb_eval_line_velocity(run.h, *ptrs))
        assert np.abs(one).max() > 0.0
        np.testing.assert_array_equal(out[k], one)
    run.close()


def test_more_runs_than_flag_slots():
    """Seventy runs at once (the process keeps 64 pinned slots for flags), a
    non-finite velocity latched by the last of them, and slots given back."""
    dims = (8, 8, 8)
    for _ in range(2):
        runs = [vlb.Run(wl.lattice_preset(*dims, precision="f32"), wl.vortex_preset(), 16)
                for _ in range(70)]
        for run in runs:
            run.step(1)
            run.sync()
        pos = np.array([[2.0, 2.0, 2.0], [3.0, 2.0, 2.0], [3.0, 3.0, 2.0], [2.0, 3.0, 2.0]])
        run = runs[-1]
        run.write_fields(np.full(dims, np.nan), np.full((3,) + dims, np.nan))
        run.seed(pos, np.array([1, 2, 3, 0]))
        with pytest.raises(RuntimeError, match="non-finite"):
            run.step(1)
            run.sync()
        run.seed(pos, np.array([1, 2, 3, 0]))
        assert run.n_points() == 4
        for run in runs:
            run.close()
