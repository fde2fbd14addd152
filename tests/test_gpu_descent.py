"""A ray's shadow factor does not depend on the wavefront it runs in.

Wavefronts whose rays head the same way descend together (fitted tip heights with
exact bounds where two are close, runs ended once nothing below can matter); others
take the general descent.  Shading the same texel centres in a shuffled order puts
rays of different headings, runs and terrain into one wavefront, so the two launches
choose differently among those paths; every value has to be the same, bit for bit,
as has every value with the early exits off, and with another ray tile (small tiles
in the default one share a ray tile's runs among the wavefronts of a workgroup)."""
import math

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

RL = math.radians(0.267)
MOON = 1737400.0


@pytest.fixture(scope="module")
def ss():
    import paper_2005_06671_amd as m
    m.lib()
    return m


def rough(rows, width, seed, amp=300.0):
    rng = np.random.default_rng(seed)
    y, x = np.mgrid[0:rows, 0:width].astype(np.float64)
    h = np.zeros((rows, width))
    for k in range(9):
        f = 0.02 * 1.9 ** k
        th = rng.uniform(0, 2 * math.pi)
        h += amp / 1.7 ** k * np.sin(f * (x * math.cos(th) + y * math.sin(th)) + rng.uniform(0, 6))
    return h.astype(np.float32)


def shuffled(ss, h, texel, e, a, p, seed):
    """shadow_points at every texel centre in a random order, put back in place."""
    rows, width = h.shape
    g = torch.Generator().manual_seed(seed)
    order = torch.randperm(rows * width, generator=g).to(h.device)
    xy = torch.stack([(order % width).float() + 0.5,
                      torch.div(order, width, rounding_mode="floor").float() + 0.5], dim=1)
    out = torch.empty(rows * width, device=h.device)
    out[order] = ss.shadow_points(h, texel, e, a, xy.contiguous(), RL, p)
    return out.view(rows, width)


SHAPES = [(1, 9), (7, 5), (16, 16), (33, 97), (64, 64), (130, 257), (257, 130), (512, 512)]
# (elevation deg, azimuth, radius, texel): azimuth pi/2 splits the tile into columns heading
# left and right; 0.2 deg puts part of the tile's rays below their horizon; a radius of 30 km
# is too small for the fit; 70 deg shortens the path over the texels
SUNS = [(1.5, 0.7, MOON, 20.0), (20.0, 0.5 * math.pi, MOON, 20.0), (0.2, 3.3, MOON, 200.0),
        (3.0, 5.9, math.inf, 10.0), (8.0, 2.2, 3.0e4, 10.0), (70.0, 4.0, 3.0e5, 50.0),
        (-0.3, 1.1, MOON, 30.0)]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: f"{s[0]}x{s[1]}")
def test_any_wavefront_same_value(ss, shape):
    for k, (deg, az, radius, texel) in enumerate(SUNS):
        print(shape, deg, az, radius, texel, flush=True)
        h = torch.from_numpy(rough(*shape, seed=k, amp=15.0 * texel)).cuda()
        e = math.radians(deg)
        for mode in (ss.SS_MODE_DP, ss.SS_MODE_POINT, ss.SS_MODE_EXACT):
            p = ss.Params(radius_m=radius, max_len_m=0.0 if k % 2 else 300.0 * texel, mode=mode)
            grid = ss.shadow_cast(h, texel, e, az, RL, p)
            p.prune = 0
            full = ss.shadow_cast(h, texel, e, az, RL, p)
            p.prune = 1
            p.ray_tile = ss.RAY_TILES["16x4"]
            other = ss.shadow_cast(h, texel, e, az, RL, p)
            p.ray_tile = 0
            mixed = shuffled(ss, h, texel, e, az, p, 7 + k)
            assert torch.equal(grid, full), (deg, mode)
            assert torch.equal(grid, mixed), (deg, mode)
            assert torch.equal(grid, other), (deg, mode)


def test_holes_and_infinities(ss):
    """Heights that are missing (NaN) or infinite: the same values on every path.  (A point at
    a texel centre takes its height from the bilinear terrain, which reads the next column and
    row with weight 0: beside a missing or infinite height it has none, so those points are
    left out.)"""
    h = torch.from_numpy(rough(200, 170, 3)).cuda()
    h[40:75, 30:90] = math.nan
    h[120:123, 100:140] = math.nan
    h[10, 10] = math.inf
    h[150:160, 20:40] = -math.inf
    bad = ~torch.isfinite(h)
    bad[:, :-1] |= ~torch.isfinite(h)[:, 1:]
    bad[:-1] |= bad[1:].clone()
    for deg, az in ((1.5, 0.7), (20.0, 0.5 * math.pi), (4.0, 3.9)):
        p = ss.Params(radius_m=MOON)
        grid = ss.shadow_cast(h, 20.0, math.radians(deg), az, RL, p)
        mixed = shuffled(ss, h, 20.0, math.radians(deg), az, p, 5)
        assert torch.equal(grid[~bad], mixed[~bad]), (deg, az)
        p.prune = 0
        assert torch.equal(grid, ss.shadow_cast(h, 20.0, math.radians(deg), az, RL, p)), (deg, az)


@pytest.mark.parametrize("rows,width,share", [(257, 300, 0.05), (700, 900, 0.003)])
def test_scattered_missing_heights(ss, rows, width, share):
    """Single missing heights show at the lowest level only, where a run whose first texel
    has none ends: grid launches (wavefronts that descend together) agree with shuffled
    points, on the sphere and on the plane."""
    g = torch.Generator().manual_seed(1)
    h = torch.from_numpy(rough(rows, width, 1))
    h[torch.rand(rows, width, generator=g) < share] = math.nan
    h = h.cuda()
    bad = torch.isnan(h)
    bad[:, :-1] |= torch.isnan(h)[:, 1:]
    bad[:-1] |= bad[1:].clone()
    for deg, az in ((1.5, 0.7), (4.0, 3.9), (0.2, 2.0)):
        for radius in (MOON, math.inf):
            print("scattered", rows, width, deg, radius, flush=True)
            p = ss.Params(radius_m=radius)
            grid = ss.shadow_cast(h, 20.0, math.radians(deg), az, RL, p)
            mixed = shuffled(ss, h, 20.0, math.radians(deg), az, p, 5)
            assert torch.equal(grid[~bad], mixed[~bad]), (deg, az, radius)


@pytest.mark.parametrize("mode", ["DP", "UNIFORM", "EXACT", "POINT"])
def test_recorded_sample_is_the_smallest(ss, mode):
    """The deciding sample a forward records, with the early exits and without: the same on
    every penumbra ray, and on a lit one the same or one before the exit over the tile's
    top, never one that a run ended early would have hidden."""
    h = torch.from_numpy(rough(257, 300, 1)).cuda()
    for deg, az, radius in ((1.5, 0.7, MOON), (4.0, 3.9, math.inf), (12.0, 0.5 * math.pi, MOON)):
        kw = dict(mode=getattr(ss, "SS_MODE_" + mode), radius_m=radius)
        e = math.radians(deg)
        s0, every = ss.shadow_cast_save(h, 20.0, e, az, RL, ss.Params(prune=0, **kw))
        s1, quick = ss.shadow_cast_save(h, 20.0, e, az, RL, ss.Params(**kw))
        assert torch.equal(s0, s1)
        part = (s0 > 0) & (s0 < 1)
        assert torch.equal(every[part], quick[part])
        if mode != "EXACT":  # its walk passes over more on lit rays
            lit = s0 >= 1
            # a sample recorded with the exits lies before one found only without them
            changed = lit & (every != quick)
            assert bool((quick[changed] < every[changed]).all())
