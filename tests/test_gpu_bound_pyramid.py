"""The tap-bound pyramid's first levels, built in one pass: every level against maxima taken
by torch, at sizes around the 64-texel blocks, with rows that are and are not a multiple of
16 bytes, with a source off its alignment, and with missing heights."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ss():
    import paper_2005_06671_amd as ss
    return ss


def reference(h):
    """Level 0 and up; fmax passes over NaN, -0 becomes +0, texels beyond an edge are absent."""
    inf = math.inf
    pad = torch.nn.functional.pad(h[None, None], (1, 1, 1, 1), mode="replicate")[0, 0]
    rows, width = h.shape
    level = torch.full_like(h, math.nan)
    for dy in range(3):
        for dx in range(3):
            level = torch.fmax(level, pad[dy:dy + rows, dx:dx + width])
    level = level + 0.0
    levels = [level]
    while max(level.shape) > 1:
        level = torch.nn.functional.pad(level, (0, level.shape[1] % 2, 0, level.shape[0] % 2), value=-inf)
        level = torch.fmax(torch.fmax(level[::2, ::2], level[1::2, ::2]),
                           torch.fmax(level[::2, 1::2], level[1::2, 1::2]))
        levels.append(level)
    return levels


@pytest.mark.parametrize("rows,width", [(1, 1), (2, 1), (1, 5), (4, 4), (3, 33), (63, 64), (64, 64),
                                        (65, 68), (64, 65), (130, 260), (257, 131), (500, 1028)])
@pytest.mark.parametrize("kind", ["plain", "shifted", "holes"])
def test_levels(ss, rows, width, kind):
    print("bound", rows, width, kind, flush=True)
    g = torch.Generator().manual_seed(rows * 1000 + width)
    h = torch.randn(rows, width, generator=g) * 100
    h[torch.rand(rows, width, generator=g) < 0.1] = -0.0
    if kind == "holes":
        h[torch.rand(rows, width, generator=g) < 0.2] = math.nan
        h[rows // 3:rows // 2, :] = math.nan
        h[:, :width // 3] = -math.inf
    want = reference(h)
    if kind == "shifted":
        d = torch.empty(rows * width + 1, device="cuda")[1:].view(rows, width)
        d.copy_(h)
    else:
        d = h.cuda()
    b = ss.bound_build(d).cpu()
    for m, ref in enumerate(want):
        off = ss.bound_level_offset(width, rows, m) if m else 0
        got = b[off:off + ref.numel()].view(ref.shape)
        same = (got.view(torch.int32) == ref.view(torch.int32)) | (torch.isnan(got) & torch.isnan(ref))
        assert bool(same.all()), (m, int((~same).sum()))
