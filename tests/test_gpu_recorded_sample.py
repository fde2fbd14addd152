"""The deciding sample a forward records on lit rays.

With the early exits a ray stops looking once the terrain's top clears the sun's disc from there
on; a sample found only without them has to lie past that exit, which is worked out here in
float64.  So a sample that a run ended early, or a chunk passed over, would have hidden shows."""
import math

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

RL = math.radians(0.267)
MOON = 1737400.0
TEXEL = 20.0


@pytest.fixture(scope="module")
def ss():
    import paper_2005_06671_amd as m
    m.lib()
    return m


def rough(rows, width, seed, amp):
    rng = np.random.default_rng(seed)
    y, x = np.mgrid[0:rows, 0:width].astype(np.float64)
    h = np.zeros((rows, width))
    for k in range(9):
        f = 0.02 * 1.9 ** k
        th = rng.uniform(0, 2 * math.pi)
        h += amp / 1.7 ** k * np.sin(f * (x * math.cos(th) + y * math.sin(th)) + rng.uniform(0, 6))
    return h.astype(np.float32)


def cleared(h, radius, e, a, t):
    """[len(t), rows, width]: the tile's top clears r_L from ray length t on (a shade loosely)."""
    rows, width = h.shape
    L = np.array([math.cos(e) * math.cos(a), math.cos(e) * math.sin(a), math.sin(e)])
    hp = h.astype(np.float64)
    rise_top = np.maximum(hp.max() - hp, 0.0)
    need = math.tan(RL + 1e-5) * (1 - 1e-4)
    t = np.asarray(t, np.float64).reshape(-1, 1, 1)
    if math.isinf(radius):
        d = t * L[2] - rise_top
        num, den = d * math.hypot(L[0], L[1]), t - d * L[2]
    else:
        X = (np.arange(width) + 0.5 - width / 2) * TEXEL / radius
        Y = ((np.arange(rows) + 0.5 - rows / 2) * TEXEL / radius)[:, None]
        g = np.sqrt(1 + X * X + Y * Y)
        s = (X * L[0] + Y * L[1] + L[2]) / g
        x = t / (radius + hp)
        w = np.sqrt(1 + x * (2 * s + x))
        d = (radius + hp) * (w - 1) - rise_top
        num, den = d * np.sqrt(1 - s * s), t * w - d * (s + x)
    return (d > -1e-2) & ((den <= 0) | (num >= need * den - 1e-2))


@pytest.mark.parametrize("mode,step", [("DP", 0), ("POINT", 0), ("UNIFORM", 1.0), ("UNIFORM", 0.5)])
@pytest.mark.parametrize("deg,az,radius", [(1.5, 0.7, MOON), (4.0, 3.9, math.inf), (12.0, 0.5 * math.pi, MOON),
                                           (30.0, 2.2, MOON)])
def test_lit_rays_record_every_sample_before_the_exit(ss, mode, step, deg, az, radius):
    rows, width = 257, 300
    hn = rough(rows, width, 1, 300.0)
    h, e = torch.from_numpy(hn).cuda(), math.radians(deg)
    kw = dict(mode=getattr(ss, "SS_MODE_" + mode), radius_m=radius, uniform_step=step or 1.0)
    s0, every = ss.shadow_cast_save(h, TEXEL, e, az, RL, ss.Params(prune=0, **kw))
    s1, quick = ss.shadow_cast_save(h, TEXEL, e, az, RL, ss.Params(**kw))
    print(mode, step, deg, radius, flush=True)
    assert torch.equal(s0, s1)
    every, quick = every.cpu().numpy(), quick.cpu().numpy()
    hd = 0.5 * TEXEL / math.cos(e)
    inc = hd if mode != "UNIFORM" else step * 2 * hd
    if mode == "UNIFORM":  # the exit is looked at every 16 steps
        at = hd + inc * np.arange(0, 4096, 16)
    else:                  # and at each run's start: runs of 5, 6, 7, ... levels, the tile's at most
        levels, a0, at = ss.maxmip_levels(width, rows), 0, []
        for j in range(40):
            at.append(max(hd, (a0 + 1) * hd - 1.5 * hd))
            a0 += 2 << (min(5 + j, levels) - 1)
        at = np.array(at)
    at = at[at < 1.5 * TEXEL * math.hypot(rows, width) / math.cos(e)]
    out = cleared(hn, radius, e, az, at)
    first = np.where(out.any(0), at[out.argmax(0)], np.inf)
    lit = (s0 >= 1).cpu().numpy()
    changed = lit & (every != quick)
    t_every = hd + inc * every
    assert lit.sum() > 10000
    assert (every[changed] >= 0).all()
    late = t_every[changed] >= first[changed] - 1e-3 * inc
    assert late.all(), (int((~late).sum()), int(changed.sum()))
    # a ray that looked at anything found something: the first step or run lies inside the tile
    looked = lit & (first > at[0]) & (every >= 0) & (t_every < first - 1e-3 * inc)
    assert (quick[looked] == every[looked]).all() and (quick[looked] >= 0).all()
    if deg < 5.0:
        assert looked.sum() > 1000
