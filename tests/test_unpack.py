"""Levels cut out of a packed pyramid (no GPU: layout and views only)."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2005_06671_amd as ss

SIZES = [(1, 1), (2, 1), (3, 5), (64, 64), (65, 63), (257, 130), (512, 512), (1019, 1531)]


def top_end(width, rows):
    """Floats up to and including the top texel, without the padding after it."""
    return ss.maxmip_level_offset(width, rows, ss.maxmip_levels(width, rows) - 1) + 1


@pytest.mark.parametrize("width,rows", SIZES)
def test_levels_are_views_at_their_offsets(width, rows):
    n = max(1, ss.maxmip_floats(width, rows))
    mm = torch.arange(n, dtype=torch.float32)
    levels = ss.maxmip_unpack(mm, width, rows)
    assert len(levels) == ss.maxmip_levels(width, rows) - 1
    w, r = width, rows
    for m, lv in enumerate(levels, 1):
        w, r = (w + 1) // 2, (r + 1) // 2
        off = ss.maxmip_level_offset(width, rows, m)
        assert lv.shape == (r, w) and lv.data_ptr() == mm[off:].data_ptr()
        assert torch.equal(lv, mm[off:off + w * r].view(r, w))


@pytest.mark.parametrize("width,rows", SIZES[1:])
def test_buffers_that_end_after_the_top_texel(width, rows):
    """The padding after the top texel need not be there, in either pyramid."""
    end = top_end(width, rows)
    whole = torch.rand(ss.maxmip_floats(width, rows))
    for a, b in zip(ss.maxmip_unpack(whole[:end].clone(), width, rows),
                    ss.maxmip_unpack(whole, width, rows)):
        assert torch.equal(a, b)
    base = ss.bound_level_offset(width, rows, 1)
    whole = torch.rand(ss.bound_floats(width, rows))
    cut = ss.bound_unpack(whole[:base + end].clone(), width, rows)
    assert len(cut) == ss.maxmip_levels(width, rows)
    for a, b in zip(cut, ss.bound_unpack(whole, width, rows)):
        assert torch.equal(a, b)
    with pytest.raises(RuntimeError):
        ss.maxmip_unpack(whole[:end - 1].clone(), width, rows)


def test_levels_can_be_written_in_place():
    """Each level is a view of its own: written in place under autograd, strided buffers."""
    width, rows = 130, 70
    mm = torch.zeros(ss.maxmip_floats(width, rows))
    src = torch.ones(35, 65, requires_grad=True)
    ss.maxmip_unpack(mm, width, rows)[0].copy_(src)
    mm.sum().backward()
    assert torch.equal(src.grad, torch.ones_like(src))
    b = torch.zeros(ss.bound_floats(width, rows))
    src = torch.ones(35, 65, requires_grad=True)
    ss.bound_unpack(b, width, rows)[1].mul_(2.0).add_(src)
    b.sum().backward()
    assert torch.equal(src.grad, torch.ones_like(src))
    wide = torch.rand(2 * ss.maxmip_floats(width, rows))[::2]
    for a, c in zip(ss.maxmip_unpack(wide, width, rows), ss.maxmip_unpack(wide.clone(), width, rows)):
        assert torch.equal(a, c)


@pytest.mark.parametrize("call", [ss.maxmip_levels, ss.maxmip_floats, ss.bound_floats,
                                  lambda w, r: ss.maxmip_level_offset(w, r, 1),
                                  lambda w, r: ss.bound_level_offset(w, r, 1)])
def test_layout_of_any_integer(call):
    """Sizes of every integer type, as they are at the call, and no floats, whatever was asked
    before."""
    want, other = call(300, 200), call(600, 200)
    assert call(np.int64(300), 200) == call(np.array(300), 200) == want
    w = torch.tensor(300)
    assert call(w, 200) == want
    w.fill_(600)
    assert call(w, 200) == other
    for bad in (300.0, "300", None, [300]):
        with pytest.raises(ctypes.ArgumentError):
            call(bad, 200)


def test_unpack_of_any_integer():
    mm = torch.rand(ss.maxmip_floats(300, 200))
    want = ss.maxmip_unpack(mm, 300, 200)
    for w in (np.int64(300), np.array(300), torch.tensor(300)):
        got = ss.maxmip_unpack(mm, w, 200)
        assert len(got) == len(want) and all(torch.equal(a, b) for a, b in zip(got, want))
    with pytest.raises(ctypes.ArgumentError):
        ss.maxmip_unpack(mm, 300.0, 200)
