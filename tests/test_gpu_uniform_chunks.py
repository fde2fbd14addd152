"""Uniform stepping in chunks, and the mipmap's word on missing heights.

Stepping with prune passes over chunks of steps that cannot matter; without it every
step is taken.  The values have to be the same bit for bit on finite tiles, and also
on tiles with missing or infinite heights, where a sample that touches one may count
as in shadow and nothing may be passed over.  The points path groups other rays into
a wavefront and has to agree with the grid."""
import math

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

MOON = 1737400.0
RL = math.radians(0.267)


@pytest.fixture(scope="module")
def ss():
    import paper_2005_06671_amd as ss
    return ss


def rough(rows, width, seed, amp=300.0):
    rng = np.random.default_rng(seed)
    y, x = np.mgrid[0:rows, 0:width].astype(np.float64)
    h = np.zeros((rows, width))
    for k in range(9):
        f = 0.02 * 1.9 ** k
        th = rng.uniform(0, 2 * math.pi)
        h += amp / 1.7 ** k * np.sin(f * (x * math.cos(th) + y * math.sin(th)) + rng.uniform(0, 6))
    return torch.from_numpy(h.astype(np.float32))


SHAPES = [(1, 1), (2, 1), (1, 40), (7, 9), (64, 64), (65, 63), (130, 257), (300, 512)]


@pytest.mark.parametrize("rows,width", SHAPES)
@pytest.mark.parametrize("step,cap", [(0.3, 0.0), (0.5, 777.0), (1.0, 0.0), (4.0, 2000.0), (37.0, 0.0)])
def test_chunks_equal_every_step(ss, rows, width, step, cap):
    h = rough(rows, width, rows).cuda()
    for deg, az, radius in ((1.5, 0.7, MOON), (12.0, 0.5 * math.pi, math.inf), (4.0, 3.9, MOON),
                            (0.2, 2.0, math.inf), (-0.2, 4.0, 3e4)):
        print("chunks", rows, width, step, cap, deg, radius, flush=True)
        kw = dict(mode=ss.SS_MODE_UNIFORM, uniform_step=step, radius_m=radius)
        if cap:
            kw["max_len_m"] = cap
        e = math.radians(deg)
        if cap / 20.0 > 48 * max(rows, width):  # more runs than a plan holds: refused, as ever
            with pytest.raises(ss.SoftShadowError):
                ss.shadow_cast(h, 20.0, e, az, RL, ss.Params(**kw))
            continue
        quick = ss.shadow_cast(h, 20.0, e, az, RL, ss.Params(**kw))
        every = ss.shadow_cast(h, 20.0, e, az, RL, ss.Params(prune=0, **kw))
        assert torch.equal(quick, every), (deg, az, radius)


def shuffled(ss, h, texel, e, a, p):
    """shadow_points at every texel centre in a shuffled order, put back in place."""
    rows, width = h.shape
    order = torch.randperm(rows * width, generator=torch.Generator().manual_seed(3)).to(h.device)
    xy = torch.stack([(order % width).float() + 0.5,
                      torch.div(order, width, rounding_mode="floor").float() + 0.5], dim=1)
    out = torch.empty(rows * width, device=h.device)
    out[order] = ss.shadow_points(h, texel, e, a, xy.contiguous(), RL, p)
    return out.view(rows, width)


@pytest.mark.parametrize("value", [math.nan, -math.inf, math.inf])
def test_missing_heights(ss, value):
    """Not a chunk is passed over: the grid agrees with shuffled points, where a wavefront's
    rays lie far apart.  (Points beside a hole have no height of their own.)"""
    h = rough(130, 257, 5)
    h[torch.rand(130, 257, generator=torch.Generator().manual_seed(2)) < 0.002] = value
    h = h.cuda()
    bad = ~torch.isfinite(h)
    bad[:, :-1] |= bad[:, 1:].clone()
    bad[:-1] |= bad[1:].clone()
    for deg, az in ((1.5, 0.7), (4.0, 3.9)):
        p = ss.Params(mode=ss.SS_MODE_UNIFORM, uniform_step=0.5, radius_m=MOON)
        grid = ss.shadow_cast(h, 20.0, math.radians(deg), az, RL, p)
        mixed = shuffled(ss, h, 20.0, math.radians(deg), az, p)
        assert torch.equal(grid[~bad], mixed[~bad]), (deg, az)


def word_of(ss, h, fuse):
    rows, width = h.shape
    mm = ss.maxmip(h, fuse_depth=fuse)
    top = ss.maxmip_level_offset(width, rows, ss.maxmip_levels(width, rows) - 1)
    got = mm[top:top + 2].cpu().numpy().view(np.uint32)
    key = (0x5F3C9A17 ^ (width * 0x9E3779B1) ^ (rows * 0x85EBCA6B)) & 0xFFFFFFFF
    return mm, (int(got[0]) ^ key) == int(got[1])


@pytest.mark.parametrize("rows,width", [(2, 1), (1, 3), (64, 64), (65, 63), (130, 257), (1000, 777),
                                        (4100, 130)])
@pytest.mark.parametrize("fuse", [1, 2, 3, 4, 5, 6])
def test_word_on_finite_heights(ss, rows, width, fuse):
    """The word says finite for finite tiles only, wherever the other height lies, and the
    levels are those of the maxima that pass over it (as fmax does)."""
    h = rough(rows, width, 3)
    assert word_of(ss, h.cuda(), fuse)[1]
    g = torch.Generator().manual_seed(rows)
    spots = [(0, 0), (rows - 1, width - 1), (rows - 1, 0), (0, width - 1)]
    spots += [(int(torch.randint(rows, (1,), generator=g)), int(torch.randint(width, (1,), generator=g)))
              for _ in range(3)]
    for n, (y, x) in enumerate(spots):
        bad = h.clone()
        bad[y, x] = (math.nan, math.inf, -math.inf)[n % 3]
        if n == 0:
            bad[:2, :2] = math.nan
        mm, finite = word_of(ss, bad.cuda(), fuse)
        assert not finite, (y, x)
        want = bad
        for got in ss.maxmip_unpack(mm, width, rows):
            want = torch.nn.functional.pad(want, (0, want.shape[1] % 2, 0, want.shape[0] % 2),
                                           value=-math.inf)  # absent
            want = torch.fmax(torch.fmax(want[::2, ::2], want[1::2, ::2]),
                              torch.fmax(want[::2, 1::2], want[1::2, 1::2]))
            assert torch.equal(torch.nan_to_num(got.cpu(), nan=1e30), torch.nan_to_num(want, nan=1e30)), (y, x)


@pytest.mark.parametrize("step", [1e4, 1e9, 1e30, 1e300])
def test_steps_longer_than_any_tile(ss, step):
    """A step of any finite length is accepted: one sample, or none once it overflows."""
    h = rough(65, 130, 9).cuda()
    print("step", step, flush=True)
    kw = dict(mode=ss.SS_MODE_UNIFORM, uniform_step=step, radius_m=MOON)
    quick = ss.shadow_cast(h, 20.0, math.radians(1.5), 0.7, RL, ss.Params(**kw))
    every = ss.shadow_cast(h, 20.0, math.radians(1.5), 0.7, RL, ss.Params(prune=0, **kw))
    assert torch.equal(quick, every)
