"""The tuner's built-in candidates (no GPU): the shape of an untuned call comes
first, the kernels that the default chooses from are among them, and a stored
shape is not used across the size at which the default changes kernels."""

import pytest

import paper_1001_1718_amd as xr
from route_util import SRC, route, shape

U8, F16, F32 = xr.XR_U8, xr.XR_F16, xr.XR_F32

# (mode, dtype, channels, (in_h, in_w), (out_h, out_w))
CASES = [
    ("bilinear", U8, 1, (512, 512), (1024, 1024)), ("bicubic", U8, 4, (4096, 4096), (8192, 8192)),
    ("bicubic", F16, 4, (4096, 4096), (2048, 2048)), ("bicubic", U8, 1, (3507, 2479), (4559, 3223)),
    ("bicubic", F32, 4, (3000, 4000), (1080, 1440)), ("bilinear", F32, 4, (3000, 4000), (1080, 1440)),
    ("nearest", F32, 4, (1000, 1200), (600, 720)), ("bilinear", U8, 1, (200, 200), (260, 260)),
    ("bicubic", F16, 4, (200, 300), (300, 450)), ("bicubic", F32, 4, (3000, 32000), (4000, 3200)),
]


@pytest.mark.parametrize("mode, dtype, channels, in_hw, out_hw", CASES)
def test_untuned_shape_and_its_kernels_are_candidates(mode, dtype, channels, in_hw, out_hw):
    key = (mode, dtype, channels, in_hw[1], in_hw[0], out_hw[1], out_hw[0])
    cands = xr.tune_candidates(*key)
    assert cands[0].as_tuple() == xr.get_tile(*key).as_tuple()
    routes = {route(mode, dtype, in_hw, out_hw, channels, tile=t) for t in cands}
    assert not any(r.startswith("error") for r in routes)
    assert route(mode, dtype, in_hw, out_hw, channels) in routes and "gather" in routes
    small = min(out_hw) < 500
    if small:
        # the per-tap strips, the default there, and the walk where it is built
        assert "strip" in routes and "walk" in {
            route(mode, dtype, in_hw, out_hw, channels, planes=99, tile=t) for t in cands}
    elif "walk" in routes:  # the walk's own columns per thread in many shapes
        own = xr.get_tile(*key).ppt_x
        assert sum(c.kernel == xr.XR_KERNEL_STRIP and c.ppt_x == own for c in cands) >= 50


def test_antialiased_candidates():
    walk = xr.tune_candidates("bilinear_aa", U8, 4, 1024, 1024, 512, 512)  # one launch whatever the block
    assert sum(c.kernel == xr.XR_KERNEL_STRIP_LDS for c in walk) == 1
    tiles = xr.tune_candidates("bilinear_aa", U8, 4, 512, 512, 200, 200)
    assert {(16, 8), (64, 4), (64, 2)} <= {(c.block_w, c.block_h) for c in tiles if c.kernel == xr.XR_KERNEL_STRIP_LDS}
    for t in walk + tiles:
        assert not route("bilinear_aa", U8, (512, 512), (200, 200), 4, tile=t).startswith("error")


def test_stored_shapes_stop_at_the_walks_least_output():
    large, small = ("bilinear", U8, 1, 700, 700, 1000, 1000), ("bilinear", U8, 1, 200, 200, 300, 300)  # up to 2^20 pixels
    before = {k: xr.get_tile(*k).as_tuple() for k in (large, small)}
    shape = xr.tile(xr.XR_KERNEL_STRIP, 128, 2, 8, 16)
    for one, other in ((large, small), (small, large)):
        xr.set_tile(*one, shape)
        try:
            assert xr.get_tile(*one).as_tuple() == shape.as_tuple()
            assert xr.get_tile(*other).as_tuple() == before[other]
        finally:
            xr.set_tile(*one, xr.tile(xr.XR_KERNEL_AUTO))


def test_a_set_shape_holds_for_either_map():
    key = ("bilinear", U8, 1, 1000, 1000, 2000, 2000)
    call = ("bilinear", U8, (1000, 1000), (2000, 2000), 1)
    kinds = (dict(), dict(mapping="paper"), dict(src_data=SRC + 1))
    before = [shape(*call, **k) for k in kinds]
    t = xr.tile(xr.XR_KERNEL_STRIP, 128, 2, 16, 8)
    xr.set_tile(*key, t)
    try:
        assert [shape(*call, **k) for k in kinds] == [t.as_tuple()] * 3
    finally:
        xr.set_tile(*key, xr.tile(xr.XR_KERNEL_AUTO))
    assert [shape(*call, **k) for k in kinds] == before
