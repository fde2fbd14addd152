"""The look at the heights ahead of stepping, recorded into a graph: each replay sees the heights as
they are, with holes made and closed again between replays, on the capture's stream and another."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu

RL = math.radians(0.267)


@pytest.fixture(scope="module")
def ss():
    import paper_2005_06671_amd as m
    m.lib()
    return m


@pytest.mark.parametrize("mode", ["UNIFORM", "EXACT"])
def test_replays_see_the_heights(ss, mode):
    g = torch.Generator().manual_seed(5)
    x = torch.nn.functional.interpolate(torch.randn(1, 1, 9, 9, generator=g), size=(260, 300),
                                        mode="bicubic", align_corners=True)[0, 0]
    whole = (300.0 * x + 3.0 * torch.rand(260, 300, generator=g)).cuda()
    low = (whole[::2, ::2] < whole[1::2, ::2]) & (whole[::2, ::2] < whole[::2, 1::2])
    low &= (torch.rand(low.shape, generator=g) < 0.05).cuda()
    holed = whole.clone()
    holed[::2, ::2][low] = math.nan
    p, e, a = ss.Params(mode=getattr(ss, "SS_MODE_" + mode)), math.radians(3.0), 0.7

    def eager(h):
        return ss.shadow_cast(h, 20.0, e, a, RL, p, bound=bound).nan_to_num(-1.0)

    h, out = whole.clone(), torch.empty_like(whole)
    bound = ss.bound_build(holed)
    mm = ss.maxmip(h)
    want = {0: eager(whole), 1: eager(holed)}
    assert not torch.equal(want[0], want[1])
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        ss.shadow_cast(h, 20.0, e, a, RL, p, mm=mm, bound=bound, out=out)
    for k, hole in enumerate((0, 0, 1, 1, 0, 1, 0)):
        print("replay", mode, k, hole, flush=True)
        h.copy_(holed if hole else whole)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out.nan_to_num(-1.0), want[hole]), k
        # and eagerly, on another stream, with the same mipmap
        with torch.cuda.stream(side):
            side.wait_stream(torch.cuda.current_stream())
            s = ss.shadow_cast(h, 20.0, e, a, RL, p, mm=mm, bound=bound)
        torch.cuda.current_stream().wait_stream(side)
        assert torch.equal(s.nan_to_num(-1.0), want[hole]), k
        torch.cuda.synchronize()


@pytest.mark.parametrize("rows,width", [(1, 2), (1, 3), (5, 7), (64, 64), (33, 129), (1023, 1021), (2100, 2048)])
@pytest.mark.parametrize("offset", [0, 1, 2, 3])
def test_every_height_is_looked_at(ss, rows, width, offset):
    """One missing height anywhere takes the word back, whatever the heights' address and number; a
    finite tile keeps it."""
    n = rows * width
    h = torch.rand(n + offset, generator=torch.Generator().manual_seed(n)).cuda()[offset:].view(rows, width)
    assert h.data_ptr() % 16 == 4 * offset
    top = ss.maxmip_level_offset(width, rows, ss.maxmip_levels(width, rows) - 1)
    p = ss.Params(mode=ss.SS_MODE_UNIFORM, radius_m=math.inf, max_len_m=50.0)
    mm = ss.maxmip(h)
    word = mm[top + 1].view(torch.int32).item()
    spots = sorted({0, 1, n // 2, n // 3, n - 1, max(n - 2, 0), max(n - 5, 0), min(n - 1, 4 * 256 * 4 + 3)})
    for k, value in zip(spots + [None], (math.nan, math.inf, -math.inf, math.nan) * 4):
        print("look", rows, width, offset, k, flush=True)
        was = None
        if k is not None:
            was = h.view(-1)[k].item()
            h.view(-1)[k] = value
        mm[top + 1] = torch.tensor(word, dtype=torch.int32).view(torch.float32)
        ss.shadow_cast(h, 10.0, 0.05, 0.7, RL, p, mm=mm)
        kept = mm[top + 1].view(torch.int32).item() == word
        assert kept == (k is None), k
        if k is not None:
            h.view(-1)[k] = was
