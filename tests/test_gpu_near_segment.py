"""The pair sum close to a segment, beside its start, where |R2| is nearly the
segment's length: targets 2^-12 from the start of segments of about 0.8, in
every kernel that adds pairs, against the same sum in extended precision.

Every coordinate is a multiple of 2^-20 in a box of powers of two, so that the
32-bit position grid holds it exactly and only the arithmetic of the sum is
compared; the near pair is above 1e3 times everything else at its target."""

import numpy as np
import pytest

from tests._cases import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2108_04435_amd as vlb  # noqa: E402

NEAR = 2.0 ** -12
# FP32: the separations and the segment vector round once on conversion, the
# dot products, roots, reciprocal and products add up to 32 roundings of 2^-24
# at the most, where no step cancels; up to 80 pairs are added behind the near
# one by the same wave, half a rounding each.
# FP64: the same count of 2^-53, up to 256 pairs by the same wave, and the two
# inverse roots' Newton steps, 1.5 (6e-8)^2 each.
TOL = {"f32": 72 * 2.0 ** -24, "f64": (32 + 128) * 2.0 ** -53 + 3 * 6e-8 ** 2}


def _layout(pairs, dims, seed):
    """pairs segments a -> b (b links to itself: an open line of two points)
    and a target beside each a that links to itself, in cells of their own."""
    rng = np.random.default_rng(seed)
    side = int(np.ceil(pairs ** (1 / 3)))
    cell = np.array(dims, float) / side
    pos, nxt = [], []
    for k in range(pairs):
        i = np.array([k % side, (k // side) % side, k // side ** 2])
        d = rng.normal(size=3)
        d *= rng.uniform(0.7, 0.95) / np.linalg.norm(d)
        a = (i + rng.uniform(0.45, 0.55, 3)) * cell
        o = np.cross(d, rng.normal(size=3))
        o *= NEAR / np.linalg.norm(o)
        n = len(pos)
        pos += [a, a + d, a + o]
        nxt += [n + 1, n + 1, n + 2]
    grid = 2.0 ** 20
    pos = np.round(np.array(pos) * grid) / grid
    return np.mod(pos, np.array(dims, float)), np.array(nxt)


def _reference(pos, nxt, dims, targets):
    ld = np.longdouble
    L = np.array(dims, ld)
    p = pos.astype(ld)
    src = np.flatnonzero(nxt != np.arange(len(nxt)))
    image = lambda x: x - L * np.round(x / L)  # noqa: E731
    d = image(p[nxt[src]] - p[src])
    out = np.zeros((len(targets), 3), ld)
    for m, j in enumerate(targets):
        r1 = image(p[src] - p[j])
        r2 = r1 + d
        n1, n2 = np.sqrt((r1 * r1).sum(1)), np.sqrt((r2 * r2).sum(1))
        q = n1 * n2
        f = (n1 + n2) / (q * (q + (r1 * r2).sum(1)))
        out[m] = (f[:, None] * np.cross(r1, d)).sum(0)
    return out


def _check(v, ref, precision):
    err = np.abs((v.astype(np.longdouble) - ref)).max(1) / np.sqrt((ref * ref).sum(1))
    say("largest relative error", float(err.max()))
    assert err.max() <= TOL[precision]


# 180 points: one launch; 1800: chunks from positions; 6000: from grid
# coordinates (FP32); 18000: two targets per lane (FP64)
@pytest.mark.parametrize("pairs", [60, 600, 2000, 6000])
@pytest.mark.parametrize("dims", [(64, 64, 64), (64, 32, 128)])   # one grid step, one per axis
@pytest.mark.parametrize("precision", sorted(TOL))
def test_beside_a_start(precision, dims, pairs):
    pos, nxt = _layout(pairs, dims, pairs)
    say("near a start", precision, dims, len(pos), "points")
    v = vlb.biot_savart(pos, nxt, dims, kappa=4.0 * np.pi, precision=precision)
    t = np.arange(2, len(pos), 3)[:60]
    _check(v[t], _reference(pos, nxt, dims, t), precision)


@pytest.mark.parametrize("levels", [1, 2])
@pytest.mark.parametrize("dims", [(64, 64, 64), (64, 32, 128)])
def test_beside_a_start_farfield(dims, levels):
    pos, nxt = _layout(600, dims, 7)
    say("near a start, far field", dims, levels)
    v = vlb.biot_savart_farfield(pos, nxt, dims, 8, 0.25, 4.0 * np.pi, levels=levels)
    t = np.arange(2, len(pos), 3)[:60]
    _check(v[t], _reference(pos, nxt, dims, t), "f32")
