"""The end of a run beside others: it waits for its own work only, its pinned
memory goes to later runs, and more runs at once than the process keeps pinned
memory for move their points all the same."""

import numpy as np
import pytest

import workloads as wl
from tests._cases import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2108_04435_amd as vlb  # noqa: E402


def _small(cap, stream=None):
    run = vlb.Run(wl.lattice_preset(16, 16, 16, precision="f32"), wl.vortex_preset(), cap,
                  stream=stream)
    pos, nxt = wl.ring((8.0, 8.0, 8.0), 4.0, (0.0, 0.0, 1.0), 30)
    run.seed(pos, nxt)
    np.testing.assert_array_equal(run.read_filaments()[0], pos)
    return run


def test_destroy_does_not_wait_for_other_runs():
    dims = (128, 128, 128)
    big = vlb.Run(wl.lattice_preset(*dims, precision="f32"), wl.vortex_preset(), 16,
                  stream=torch.cuda.Stream())
    big.step(2)
    big.sync()
    small = [_small(4096, torch.cuda.Stream()) for _ in range(3)]
    torch.cuda.synchronize()
    say("destroy beside queued work")
    big.step(5000)   # far longer than the calls below
    done = torch.cuda.Event()
    done.record(big.stream)
    for run in small:
        run.close()
    assert not done.query()
    big.sync()
    big.close()


@pytest.mark.parametrize("cap,count", [(16000, 20), (40, 80)])   # beyond the bytes, the blocks
def test_more_runs_than_pinned_memory(cap, count):
    say("pinned memory", cap, count)
    for _ in range(2):
        runs = [_small(cap) for _ in range(count)]
        pos, nxt = wl.ring((7.0, 8.0, 9.0), 3.0, (0.0, 1.0, 0.3), 25)
        want = None
        for run in runs:
            run.seed(pos, nxt)
            out = run.eval_line_velocity()
            want = want or out
            for k in out:
                np.testing.assert_array_equal(out[k], want[k])
            np.testing.assert_array_equal(run.read_filaments()[0], pos)
        for run in runs[::-1]:
            run.close()


def test_points_beyond_a_smaller_block():
    """A run whose block is smaller than its capacity asks for: blocks of all
    sizes go round."""
    caps = [30, 16000, 300, 60, 9000, 2000]
    for shift in range(len(caps)):
        runs = [_small(max(30, c)) for c in caps[shift:] + caps[:shift]]
        for run in runs[::2] + runs[1::2]:
            run.close()
