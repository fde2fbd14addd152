"""The exact mode under steep suns takes the same route in every call, whatever the tile's bend: the
batched forms give the per-tile call's values bit for bit also where a small body's rays run far out
and samples of almost vertical rays are lost to rounding."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ss():
    import paper_2005_06671_amd as m
    m.lib()
    return m


def tile(rows, width, amp):
    g = torch.Generator().manual_seed(61)
    h, n, a = torch.zeros(rows, width), 3, 1.0
    while n < 2 * max(rows, width) and a > 1e-4:
        r = torch.randn(1, 1, min(n, 4 * rows) + 1, n + 1, generator=g)
        h += a * torch.nn.functional.interpolate(r, size=(rows, width), mode="bicubic", align_corners=True)[0, 0]
        n, a = 2 * n, 0.48 * a
    return (0.5 * amp * h).cuda()


@pytest.mark.parametrize("deg", [29.0, 31.0, 60.0, 89.9544])
@pytest.mark.parametrize("rows,width,texel,radius", [(3, 40000, 0.21, 8403.0), (300, 257, 20.0, 1737400.0),
                                                     (200, 300, 10.0, math.inf)])
def test_batched_equals_per_tile(ss, form, deg, rows, width, texel, radius):
    h = tile(rows, width, 56.0 * texel)
    p = ss.Params(radius_m=radius, mode=ss.SS_MODE_EXACT)
    e = math.radians(deg)
    for rl in (math.radians(0.267), 0.4):
        print(form, deg, rows, width, rl, flush=True)
        one = ss.shadow_cast(h, texel, e, 1e-8, rl, p)
        both = ss.shadow_cast_batched([h], [texel], [(e, 1e-8, rl), (0.9 * e, 0.3, rl)], p)[0]
        assert torch.equal(one, both[0])
        assert torch.equal(ss.shadow_cast(h, texel, 0.9 * e, 0.3, rl, p), both[1])
