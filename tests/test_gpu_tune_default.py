"""GPU test of the tuner's built-in list: whatever it keeps (the untuned shape or
a stored one), later calls give the same bits, and the shape that it reports is
the one they resolve to; a shape tuned on one size of batch is not another's."""

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1001_1718_amd as xr  # noqa: E402
from route_util import SRC, shape  # noqa: E402

DEV = "cuda:0"
CODES = {torch.uint8: xr.XR_U8, torch.float16: xr.XR_F16, torch.float32: xr.XR_F32}


@pytest.mark.parametrize("mode, dtype, channels, in_hw, out_hw", [
    ("bicubic", torch.float32, 4, (500, 900), (300, 540)), ("bilinear", torch.uint8, 1, (200, 200), (260, 261)),
    ("bicubic", torch.uint8, 1, (700, 900), (910, 1170)), ("bicubic_aa", torch.uint8, 4, (1024, 1024), (512, 512)),
    ("bilinear_aa", torch.float16, 1, (301, 500), (60, 97)), ("bilinear", torch.uint8, 1, (301, 77), (602, 154))])
def test_autotune_keeps_results(mode, dtype, channels, in_hw, out_hw):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(1)
    x = (torch.rand((*in_hw, channels), generator=gen, device=DEV) * 255).to(dtype)
    key = (mode, CODES[dtype], channels, in_hw[1], in_hw[0], out_hw[1], out_hw[0])
    untuned = shape(mode, CODES[dtype], in_hw, out_hw, channels)
    before = xr.resize(x, out_hw, mode)
    out = torch.empty_like(before)
    try:
        best, ms = xr.autotune(x, out, mode, reps=2, groups=3)
        assert ms > 0 and torch.equal(out, before)
        now = shape(mode, CODES[dtype], in_hw, out_hw, channels)  # (77 columns of bytes: not aligned)
        if mode.endswith("_aa"):  # (an untuned antialiased call is a strip shape by name)
            assert now in (untuned, best.as_tuple())
        else:
            assert now == best.as_tuple()
        assert torch.equal(xr.resize(x, out_hw, mode), before)
        assert torch.equal(xr.resize(x, out_hw, mode, tile=best), before)
    finally:
        xr.set_tile(*key, xr.tile(xr.XR_KERNEL_AUTO))


def _shape(batch):
    """block_w, block_h and strip rows that a batch was prepared with."""
    at = batch.ws_ptr - batch.workspace.data_ptr()
    return batch.workspace[at:at + 24].cpu().view(torch.int32)[2:5].tolist()


def test_batch_shapes_are_kept_per_size_of_batch():
    def pairs(side):  # float32 RGBA: a wavefront covers 64 columns
        x = torch.rand((64, 64, 4), device=DEV)
        return [(x, torch.empty((side, side, 4), device=DEV), "bilinear")]

    small, large = pairs(300), pairs(8192)  # 65 and 43,776 wavefronts at 24 rows
    untuned = _shape(xr.Batch(large))
    b = xr.Batch(small)
    ref = xr.resize(small[0][0], (300, 300))
    b.autotune(candidates=[xr.tile(xr.XR_KERNEL_STRIP, 64, 3, 0, 5)], reps=1, groups=1)
    assert _shape(xr.Batch(small)) == [64, 3, 5] and _shape(xr.Batch(large)) == untuned == [128, 2, 24]
    best, _ = b.autotune(reps=2, groups=3)
    again = xr.Batch(small)
    assert _shape(again) == [best.block_w, best.block_h, best.ppt_y]
    small[0][1].zero_()
    again.run()
    assert torch.equal(small[0][1], ref)


def test_shapes_of_the_exact_kernels_stay_with_them():
    """A shape tuned at x2 is neither the printed map's nor an unaligned image's."""
    x = torch.zeros((300, 400), dtype=torch.uint8, device=DEV)
    out = torch.empty((600, 800), dtype=torch.uint8, device=DEV)
    call = ("bilinear", xr.XR_U8, (300, 400), (600, 800))
    others = (dict(mapping="paper"), dict(src_data=SRC + 1))
    untuned = [shape(*call, **k) for k in others]
    best = xr.tile(xr.XR_KERNEL_STRIP, 128, 2, 8, 16)
    xr.autotune(x, out, "bilinear", candidates=[best], reps=1, groups=1)
    try:
        assert shape(*call) == best.as_tuple()
        assert [shape(*call, **k) for k in others] == untuned
    finally:
        xr.set_tile("bilinear", xr.XR_U8, 1, 400, 300, 800, 600, xr.tile(xr.XR_KERNEL_AUTO))
