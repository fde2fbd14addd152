"""The view walk's approximate cell geometry never changes a hit: pyramid walk and dense march
give the same lengths and positions bit for bit, on bodies whose terrain is shallow against the
radius (series form of the height) and not (root form), on the plane, and beside missing heights."""
import math

import numpy as np
import pytest
import torch

from synth import view_scene

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ss():
    import paper_2005_06671_amd as m
    m.lib()
    return m


@pytest.mark.parametrize("radius", [1737400.0, 2.0e5, 6.0e4, math.inf])
@pytest.mark.parametrize("kind", ["oblique", "grazing", "nadir", "outside", "flyover"])
def test_walk_equals_dense(ss, kind, radius):
    for rows, width, texel in ((131, 190, 20.0), (256, 256, 10.0)):
        print(kind, radius, rows, width, flush=True)
        rng = np.random.default_rng(rows)
        y, x = np.mgrid[0:rows, 0:width]
        h = sum(200.0 / (k + 1) * np.sin(0.03 * 1.8 ** k * (x * math.cos(k) + y * math.sin(k)) + k)
                for k in range(7)) + rng.uniform(0, 2.0, (rows, width))
        h = torch.from_numpy(h.astype(np.float32)).cuda()
        h[20:35, 40:70] = math.nan
        bound = ss.bound_build(h)
        c = view_scene(kind, 150, 101, width, rows, texel, 0.4 * texel)
        t, xy = ss.view_cast(h, texel, ss.Camera(**c), radius, bound)
        td, xyd = ss.view_cast(h, texel, ss.Camera(mode=ss.SS_VIEW_DENSE, **c), radius, bound)
        assert torch.equal(t, td)
        assert torch.equal(xy.nan_to_num(-9.0), xyd.nan_to_num(-9.0))


@pytest.mark.parametrize("radius", [1737400.0, 6.0e4, math.inf])
def test_counting_walk_hits_the_same(ss, radius):
    """The walk that counts its samples and cells keeps rounded cell geometry: same hits."""
    rng = np.random.default_rng(4)
    h = torch.from_numpy(rng.normal(0, 30, (256, 200)).astype(np.float32)).cuda()
    bound = ss.bound_build(h)
    for kind in ("oblique", "grazing", "flyover"):
        print("counting", kind, radius, flush=True)
        cam = ss.Camera(**view_scene(kind, 150, 101, 200, 256, 10.0, None))
        t, xy = ss.view_cast(h, 10.0, cam, radius, bound)
        tc, xyc, steps = ss.view_cast(h, 10.0, cam, radius, bound, steps=True)
        assert torch.equal(t, tc)
        assert torch.equal(xy.nan_to_num(-9.0), xyc.nan_to_num(-9.0))
        assert bool((steps >= 0).all()) and bool((steps[torch.isfinite(t)][:, 0] > 0).all())
