"""The stand-alone sum over every route it can take: each set of closed axes
(the FP64 kernel is specialised on it), point counts on both sides of the
count from which it takes two targets per lane, of the one up to which the
FP32 sum reads positions and of the one up to which it is one launch, ragged
last blocks and tiles.  Against the oracle's sum at sampled targets, in FP64."""

import numpy as np
import pytest

import workloads as wl
from oracle import coupled, vfm
from oracle.lbm import Lattice
from tests._cases import rel_l2, say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2108_04435_amd as vlb  # noqa: E402

# FP64: about 30 roundings of 1.1e-16 per pair and a sum of up to 1.7e4 terms
# whose magnitudes exceed the result's a few times over.  FP32: the same
# count of 6e-8.
TOL = {"f64": 1e-12, "f32": 1e-5}


def _points(seed, n, dims, walls):
    """n points: rings, the last one cut to a closed loop of what is left."""
    pos, nxt = [], []
    rng = np.random.default_rng(seed)
    left = n
    while left > 0:
        m = min(left, int(rng.integers(20, 60)))
        if left - m < 3:
            m = left
        R = 0.9 * m / (2 * np.pi)
        R = min(R, 0.3 * min(dims))
        c = [rng.uniform(R, d - 1 - R) for d in dims]
        p, k = wl.ring(c, R, wl.random_unit(rng), m, phase=rng.uniform())
        nxt.append(k + (n - left))
        pos.append(p)
        left -= m
    lat = Lattice(*dims, walls=walls)
    return vfm.wrap_positions(np.concatenate(pos), lat), np.concatenate(nxt), lat


def _check(n, dims, walls, precision):
    pos, nxt, lat = _points(n, n, dims, walls)
    assert pos.shape[0] == n
    say("sum", n, dims, walls, precision)
    v = vlb.biot_savart(pos, nxt, dims, walls, kappa=0.1, precision=precision)
    t = np.unique(np.r_[0:min(n, 70), max(0, n - 70):n])
    ref = vfm.biot_savart_nonlocal(pos, nxt, coupled.prev_from_next(nxt), lat, 0.1, targets=t)
    err = rel_l2(v[t], ref)
    say("rel l2", err)
    assert err <= TOL[precision]


@pytest.mark.parametrize("n", [700, 1300])   # one launch, chunks
@pytest.mark.parametrize("mask", range(8))
def test_every_set_of_closed_axes(mask, n):
    walls = tuple(bool((mask >> a) & 1) for a in range(3))
    _check(n, (40, 36, 48), walls, "f64")


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("n", [3, 63, 65, 257, 1023, 1025, 1280, 1281, 4096, 4097, 16383,
                               16385])
def test_point_counts(n, precision):
    _check(n, (64, 64, 64), (False, True, False), precision)
