"""The far-field sum where its kernels' splits have their edges, against the
oracle of the same approximation: cells of more points than the ordering
block has threads (256) and of one wave's, counts of points around the 64
and 256 targets of a wave and a block, waves whose targets lie on both sides
of the box boundary, and fewer cells than chunks."""

import numpy as np
import pytest

from oracle import coupled, farfield, vfm
from oracle.lbm import Lattice
from tests._cases import rel_l2, say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2108_04435_amd as vlb  # noqa: E402


def _image(d, L):
    return d - L * np.round(d / L)


@pytest.mark.parametrize("levels", [1, 2])
@pytest.mark.parametrize("dims,cell,points", [
    ((32, 32, 32), 8, 2600),   # 325 points per cell of 16: two rounds of ranks
    ((32, 32, 32), 16, 2600),  # one level: the same; two: one cell of 32
    ((64, 64, 32), 8, 64), ((64, 64, 32), 8, 65), ((64, 64, 32), 8, 257),
    ((48, 96, 48), 8, 1000)])
def test_farfield_edges(dims, cell, points, levels):
    """Rings of 26 points (the last one of the rest) centred anywhere in the
    box, so that some lie across its boundary.  FP32 arithmetic on 32-bit
    positions: 1e-5 of the FP64 oracle in the L2 norm, as for the other
    tangles, over the targets that keep 0.05 from the segments of other
    points: at a distance e from a segment of length l the pair's denominator
    (|r1| + |r2|)^2 - l^2 is of order e^2, so that FP32 leaves the velocity
    2^-24 (l/e)^2 of itself, 2e-5 of one pair there, and anything below (the
    first case has one such target, at 0.003)."""
    rng = np.random.default_rng(points + cell)
    L = np.array(dims, float)
    pos, nxt = [], []
    while len(pos) < points:
        m = min(26, points - len(pos))
        m = m if points - len(pos) - m >= 3 or m == points - len(pos) else m - 3
        th = 2.0 * np.pi * np.arange(m) / m
        e = np.linalg.qr(rng.normal(size=(3, 2)))[0]
        ring = rng.uniform(0.0, 1.0, 3) * L + 3.4 * (np.outer(np.cos(th), e[:, 0]) +
                                                     np.outer(np.sin(th), e[:, 1]))
        nxt += [len(pos) + (i + 1) % m for i in range(m)]
        pos += list(ring)
    lat = Lattice(*dims)
    pos = vfm.wrap_positions(np.array(pos), lat)
    nxt = np.array(nxt)
    say(f"farfield edges {dims} cell {cell} levels {levels}: {len(pos)} points")
    got = vlb.biot_savart_farfield(pos, nxt, dims, cell, 0.5, 0.1, levels=levels)
    ref, st = farfield.biot_savart_farfield(pos, nxt, coupled.prev_from_next(nxt), lat, 0.1, cell,
                                            0.5, levels=levels)
    say(f"  far {st['far']:.1f}, split {st['split']:.1f}, direct {st['direct']:.0f}")
    d = _image(pos[nxt] - pos, L)
    keep = np.ones(len(pos), bool)
    for j in range(len(pos)):
        r = _image(pos[j] - pos, L)
        t = np.clip((r * d).sum(1) / (d * d).sum(1), 0.0, 1.0)
        off = ((r - t[:, None] * d) ** 2).sum(1)
        off[[j, np.flatnonzero(nxt == j)[0]]] = 1.0
        keep[j] = off.min() > 0.05 ** 2
    assert keep.mean() > 0.95
    assert rel_l2(got[keep], ref[keep]) <= 1e-5
