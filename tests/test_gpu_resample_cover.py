"""Resampling visits only the destination texels its source can cover, and takes short forms of
the divisions: the result equals the oracle's bit for bit, coverage included, wherever the source
lies -- inside, beside and around the destination, beyond it, turned, on wide frames whose
planes bend away from each other, and behind the destination plane."""
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


def frame(rng, w, rows, texel, away, turn, origin):
    c = np.array([math.sin(away), 0.3 * math.sin(away), math.cos(away)])
    c /= np.linalg.norm(c)
    a = np.cross(c, (0.0, 1.0, 0.0))
    a /= np.linalg.norm(a)
    ex = math.cos(turn) * a + math.sin(turn) * np.cross(c, a)
    return dict(width=w, rows=rows, texel_m=texel, centre=tuple(c), ex=tuple(ex),
                ey=tuple(np.cross(c, ex)), origin=origin)


# (body radius, source side, spacing, angle between the frames, source offset in its sides)
CASES = [(1737400.0, 60, 30.0, 0.0, 0.0), (1737400.0, 200, 3.0, 2e-3, 0.3),
         (1737400.0, 33, 10.0, 1.5e-3, 0.0), (1737400.0, 64, 10.0, 0.2, 0.0),
         (5000.0, 130, 40.0, 0.5, 0.1), (5000.0, 130, 40.0, 1.2, 0.0), (3000.0, 257, 60.0, 2.8, 0.0),
         (1.0e-3, 50, 1e-7, 0.0, 0.2), (1737400.0, 1, 900.0, 0.0, 0.4)]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_covered_texels_bitwise(ss, case):
    radius, side, texel, away, off = CASES[case]
    for trial in range(4):
        rng = np.random.default_rng(100 * case + trial)
        fs = frame(rng, side, side + trial, texel, away, rng.uniform(0, 6.3),
                   (off * side * texel, -off * side * texel * trial))
        w, rows = int(rng.integers(1, 150)), int(rng.integers(1, 150))
        fd = frame(rng, w, rows, texel * rng.uniform(0.3, 1.6), 0.0, rng.uniform(0, 6.3), (0.0, 0.0))
        h = rng.normal(0, 500.0, (fs["rows"], fs["width"])).astype(np.float32)
        ref = np.full((rows, w), np.nan, dtype=np.float32)
        ref = oracle.resample(h, oracle.Frame(**fs), oracle.Frame(**fd), radius, dst=ref)[0]
        out = torch.full((rows, w), math.nan, dtype=torch.float32, device="cuda")
        ss.resample(torch.from_numpy(h).cuda(), ss.Frame(**fs), out, ss.Frame(**fd), radius)
        print(case, trial, int(np.isfinite(ref).sum()), "of", ref.size, flush=True)
        assert np.array_equal(out.cpu().numpy(), ref, equal_nan=True)
