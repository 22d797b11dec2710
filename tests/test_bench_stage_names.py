"""Which runs the benchmark reports as stepping by fused stages: the rule of the
library by the capacity, the wall images, the lattice's time and the far field."""

import bench
import workloads as wl


def _case(dims, walls=(False, False, False), precision="f64", **vor):
    return wl.lattice_preset(*dims, walls=walls, precision=precision), wl.vortex_preset(**vor)


def test_fused_stages_rule():
    cfg = wl.config_ring32()
    assert bench.fused_stages(cfg["lattice"], cfg["vortex"], bench.point_capacity(64))
    small = (32, 32, 32)
    lat, vor = _case(small)
    assert bench.fused_stages(lat, vor, 1536) and not bench.fused_stages(lat, vor, 1537)
    # a longer lattice: 504 bytes per node, 5e-5 s at 5 TB/s from 496032 nodes on
    lat, vor = _case((64, 64, 128))
    assert bench.fused_stages(lat, vor, 1024) and not bench.fused_stages(lat, vor, 1025)
    # wall images on two axes: nine copies
    lat, vor = _case(small, (True, True, False), wall_images=True)
    assert bench.fused_stages(lat, vor, 170) and not bench.fused_stages(lat, vor, 171)
    lat, vor = _case(small, precision="f32")
    vor["ff_cell"] = 8
    assert not bench.fused_stages(lat, vor, 64)
