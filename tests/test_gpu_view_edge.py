"""View rays that hit at the tile's very edge: the walk tests the last samples before the ray leaves
the tile, however its own crossings of the edge round.

Only the last half texel along an edge has a height (a wall; the rest is missing), and steps are
longer than that, so a ray hits there or nowhere, and of a million rays some have their one sample
within rounding of the edge."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ss():
    import paper_2005_06671_amd as m
    m.lib()
    return m


@pytest.mark.parametrize("side", ["+x", "-x", "+y", "-y"])
@pytest.mark.parametrize("radius", [1737400.0, 4.0e4, math.inf])
def test_hits_in_the_last_half_texel(ss, side, radius):
    n, texel = 400, 20.0
    h = torch.full((n, n), math.nan)
    {"+x": h[:, -1], "-x": h[:, 0], "+y": h[-1], "-y": h[0]}[side][:] = 2000.0
    h = h.cuda()
    bound = ss.bound_build(h)
    s, sign = n * texel, 1.0 if side[0] == "+" else -1.0
    ax = 0 if side[1] == "x" else 1
    fwd, right, eye = [0.0] * 3, [0.0] * 3, [0.0] * 3
    fwd[ax], right[1 - ax], eye[ax] = sign, 0.8, -0.45 * sign * s
    eye[2] = 300.0
    hits = 0
    for step in (0.61, 0.73, 0.97):
        cam = dict(width=1024, height=700, eye=tuple(eye), fwd=tuple(fwd), right=tuple(right),
                   up=(0.0, 0.0, 0.03), step_m=step * texel)
        print("edge", side, radius, step, flush=True)
        t, xy = ss.view_cast(h, texel, ss.Camera(**cam), radius, bound)
        td, xyd = ss.view_cast(h, texel, ss.Camera(mode=ss.SS_VIEW_DENSE, **cam), radius, bound)
        hits += int(torch.isfinite(td).sum())
        assert torch.equal(t, td), int((t != td).sum())
        assert torch.equal(xy.nan_to_num(-9.0), xyd.nan_to_num(-9.0))
    assert hits > 100000
