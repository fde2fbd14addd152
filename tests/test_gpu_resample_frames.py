"""Frames whose axes are off by as much as is accepted (each product within 1e-9): on a large body
that is many texels of a fine tile, and which texels a source covers still follows from the
forward positions alone, as in the oracle."""
import math

import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ss():
    import paper_2005_06671_amd as m
    m.lib()
    return m


@pytest.mark.parametrize("radius,texel", [(1737400.0, 1e-4), (1737400.0, 3e-5), (6.4e6, 2e-3), (1e9, 0.05),
                                          (1737400.0, 20.0)])
@pytest.mark.parametrize("tilt", ["dst", "src", "both", "scale"])
def test_axes_at_the_tolerance(ss, radius, texel, tilt):
    off = 0.9e-9
    c, ex, ey = np.array([0.6, 0.0, 0.8]), np.array([0.8, 0.0, -0.6]), np.array([0.0, 1.0, 0.0])
    for sx, sy in ((1, 1), (-1, 1), (1, -1), (-1, -1)):
        bent = dict(ex=tuple(ex + sx * off * c), ey=tuple(ey + sy * off * c))
        if tilt == "scale":
            bent = dict(ex=tuple(ex * (1 + sx * 0.45e-9)), ey=tuple(ey * (1 + sy * 0.45e-9)))
        plain = dict(ex=tuple(ex), ey=tuple(ey))
        fs = dict(width=70, rows=90, texel_m=texel, centre=tuple(c), origin=(20 * texel, -15 * texel),
                  **(bent if tilt in ("src", "both", "scale") else plain))
        fd = dict(width=110, rows=130, texel_m=0.9 * texel, centre=tuple(c), origin=(0.0, 0.0),
                  **(bent if tilt in ("dst", "both") else plain))
        h = np.random.default_rng(3).normal(0, 5.0, (90, 70)).astype(np.float32)
        ref = np.full((130, 110), np.nan, dtype=np.float32)
        ref = oracle.resample(h, oracle.Frame(**fs), oracle.Frame(**fd), radius, dst=ref)[0]
        out = torch.full((130, 110), math.nan, dtype=torch.float32, device="cuda")
        ss.resample(torch.from_numpy(h).cuda(), ss.Frame(**fs), out, ss.Frame(**fd), radius)
        print(radius, texel, tilt, sx, sy, int(np.isfinite(ref).sum()), flush=True)
        assert np.array_equal(out.cpu().numpy(), ref, equal_nan=True)
