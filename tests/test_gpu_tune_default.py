"""GPU test of the tuner's built-in list: whatever it keeps (the untuned shape or
a stored one), later calls give the same bits, and the shape that it reports is
the one they resolve to."""

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1001_1718_amd as xr  # noqa: E402

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
    untuned = xr.get_tile(*key)
    before = xr.resize(x, out_hw, mode)
    out = torch.empty_like(before)
    try:
        best, ms = xr.autotune(x, out, mode, reps=2, groups=3)
        assert ms > 0 and torch.equal(out, before)
        now = xr.get_tile(*key).as_tuple()
        if mode.endswith("_aa"):  # (an untuned antialiased call is a strip shape by name)
            assert now in (untuned.as_tuple(), best.as_tuple())
        else:
            assert now == best.as_tuple()
        assert torch.equal(xr.resize(x, out_hw, mode), before)
        assert torch.equal(xr.resize(x, out_hw, mode, tile=best), before)
    finally:
        xr.set_tile(*key, xr.tile(xr.XR_KERNEL_AUTO))
