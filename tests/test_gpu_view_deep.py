"""View rays over terrain far below the datum of a small body.

The walk's height series is cut short, and what it leaves out grows with the fourth power of the
depth, so over a floor at a tenth of the radius below the datum it must still not put a ray above
a cell that it enters.  One texel near the datum keeps the tile's top there.  Walk and dense march
give the same hits bit for bit, with step counts and without."""
import math

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ss():
    import paper_2005_06671_amd as m
    m.lib()
    return m


# (radius, depth of the floor, texel): 2 to 20% of the radius, and the Moon's deepest floor
BODIES = [(262.7e3, 20e3, 10.0), (11e3, 1e3, 1.0), (1e3, 100.0, 0.25), (5e3, 1e3, 0.5),
          (6e4, 1.2e3, 5.0), (1737400.0, 9e3, 20.0)]


@pytest.mark.parametrize("radius,depth,texel", BODIES)
@pytest.mark.parametrize("down", [4.0, 15.0, 60.0])
def test_deep_floor_walk_equals_dense(ss, radius, depth, texel, down):
    rows, width = 250, 320
    rng = np.random.default_rng(rows)
    y, x = np.mgrid[0:rows, 0:width]
    h = sum(2.0 * texel / (k + 1) * np.sin(0.05 * 1.9 ** k * (x * math.cos(k) + y * math.sin(k)) + k)
            for k in range(5)) + rng.uniform(0, 0.3 * texel, (rows, width)) - depth
    h[3, 5] = -0.01 * depth
    h = torch.from_numpy(h.astype(np.float32)).cuda()
    bound = ss.bound_build(h)
    # an eye over one side of the floor, looking across it `down` degrees below the horizon
    s = width * texel
    d = math.radians(down)
    look = (math.cos(d), 0.2 * math.cos(d), -math.sin(d))
    up = (math.sin(d), 0.0, math.cos(d))
    eye = (-0.3 * s, -0.1 * s, 0.12 * s * math.tan(d) + 6.0 * texel - depth)
    cam = dict(width=160, height=90, eye=eye, fwd=look, right=(0.0, -0.5, 0.0),
               up=tuple(0.1 * v for v in up), step_m=0.25 * texel)
    print("deep", radius, depth, texel, down, flush=True)
    t, xy = ss.view_cast(h, texel, ss.Camera(**cam), radius, bound)
    tc, xyc, _ = ss.view_cast(h, texel, ss.Camera(**cam), radius, bound, steps=True)
    td, xyd = ss.view_cast(h, texel, ss.Camera(mode=ss.SS_VIEW_DENSE, **cam), radius, bound)
    assert int(torch.isfinite(td).sum()) > 2000
    assert torch.equal(tc, td)
    assert torch.equal(xyc.nan_to_num(-9.0), xyd.nan_to_num(-9.0))
    assert torch.equal(t, td), int((t != td).sum())
    assert torch.equal(xy.nan_to_num(-9.0), xyd.nan_to_num(-9.0))
