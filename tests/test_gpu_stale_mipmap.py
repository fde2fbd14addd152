"""Heights that go missing after the mipmap was built.

Maxima pass over missing heights, so a mipmap stays what a build would write when holes appear
beside the maxima; only the word after its top texel still says that every height is finite.
Uniform and exact stepping must not take its word for it: the values are those of a mipmap built
from the heights as they are, in every call that steps, also where the ray window or the list of
points is small against the tile."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu

RL = math.radians(0.267)
TEXEL = 20.0


@pytest.fixture(scope="module")
def ss():
    import paper_2005_06671_amd as m
    m.lib()
    return m


def tile(rows, width, seed):
    g = torch.Generator().manual_seed(seed)
    x = torch.nn.functional.interpolate(torch.randn(1, 1, 9, 9, generator=g), size=(rows, width),
                                        mode="bicubic", align_corners=True)[0, 0]
    return (300.0 * x + 3.0 * torch.rand(rows, width, generator=g)).cuda()


def punch(h, value, how):
    """h with missing heights that leave every 2 x 2 maximum as it is."""
    low = torch.zeros_like(h, dtype=torch.bool)
    low[:-1, :-1] = (h[:-1, :-1] < h[1:, :-1]) & (h[:-1, :-1] < h[:-1, 1:])
    low[1::2] = False
    low[:, 1::2] = False
    if how != "some":
        k = low.reshape(-1).nonzero()
        low[:] = False
        low.view(-1)[k[k.numel() // 2 if how == "one" else -1]] = True
    else:
        low &= (torch.rand(h.shape, generator=torch.Generator().manual_seed(1)) < 0.05).cuda()
    out = h.clone()
    out[low] = value
    return out


@pytest.mark.parametrize("mode", ["UNIFORM", "EXACT"])
@pytest.mark.parametrize("value,how", [(math.nan, "some"), (math.nan, "one"), (-math.inf, "some"),
                                       (math.nan, "last")])
@pytest.mark.parametrize("rows,width", [(64, 96), (300, 257), (517, 640)])
def test_word_left_by_an_earlier_build(ss, mode, value, how, rows, width):
    p = ss.Params(mode=getattr(ss, "SS_MODE_" + mode))
    whole = tile(rows, width, rows)
    h = punch(whole, value, how)
    fresh, bound = ss.maxmip(h), ss.bound_build(h)
    xy = torch.rand(20, 30, 2, generator=torch.Generator().manual_seed(2)).cuda()
    xy *= torch.tensor([float(width), float(rows)], device="cuda")
    g = torch.ones(rows, width, device="cuda")

    def calls(mm):
        e, a, kw = math.radians(3.0), 0.7, dict(params=p, bound=bound)
        mms = (mm(), mm(), mm(), mm(), mm(), mm(), mm(), mm())
        s = ss.shadow_cast(h, TEXEL, e, a, RL, mm=mms[0], **kw)
        yield "cast", s
        yield "again", ss.shadow_cast(h, TEXEL, e, a, RL, mm=mms[0], **kw)
        yield "window", ss.shadow_cast(h, TEXEL, e, a, RL, mm=mms[1], window=(9, 5, 8, 3), **kw)
        yield "counted", ss.shadow_cast_counted(h, TEXEL, e, a, RL, mm=mms[2], **kw)[0]
        yield "points", ss.shadow_points(h, TEXEL, e, a, xy.view(-1, 2), RL, mm=mms[3], **kw)
        yield "few", ss.shadow_points(h, TEXEL, e, a, xy[0, :3], RL, mm=mms[4], **kw)
        yield "image", ss.shadow_points_image(h, TEXEL, e, a, xy, RL, mm=mms[5], **kw)
        yield "back", ss.shadow_cast_backward(h, TEXEL, e, a, g, RL, mm=mms[6], **kw)[0]
        yield "backpen", ss.shadow_cast_backward_penumbra(h, TEXEL, e, a, s, g, RL, mm=mms[7], **kw)[0]

    def earlier():  # built before the heights went missing
        return ss.maxmip(whole)

    def filled():  # another build's buffer, the levels filled in by hand
        mm = ss.maxmip(whole)
        for to, frm in zip(ss.maxmip_unpack(mm, width, rows), ss.maxmip_unpack(fresh, width, rows)):
            to.copy_(frm)
        return mm

    want = list(calls(lambda: fresh))
    for kind in (earlier, filled):
        print(mode, value, how, rows, width, kind.__name__, flush=True)
        for (name, w), (_, got) in zip(want, calls(kind)):
            if "back" in name:  # sums in any order
                assert torch.equal(torch.isnan(w), torch.isnan(got)), name
                assert torch.allclose(w, got, rtol=1e-3, atol=1e-4 * float(w.nan_to_num().abs().max()),
                                      equal_nan=True), name
            else:
                assert torch.equal(w.nan_to_num(-1.0), got.nan_to_num(-1.0)), (kind.__name__, name)
