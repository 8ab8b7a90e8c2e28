"""GPU test of the antialiased gather walk (the default where enough strips fill
the GPU): every value must equal, bit for bit, the one-pixel-per-thread
gather's, whose results tests/test_gpu_forward.py holds to the oracle (both
evaluate the same float32 sequence). The shapes sit at the walk's edges: one
column tile or one column more, strips that end early, one tap and the most
taps held in registers and more, rows at every byte alignment, infinities."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1001_1718_amd as xr  # noqa: E402

DEV = "cuda:0"
GATHER = xr.tile(xr.XR_KERNEL_GATHER, 32, 4)
# (in_h, in_w, out_h, out_w): unchanged rows, x0.5, 5 taps, the register limit,
# past it, wide windows, a column tile and its neighbours, growing columns
SHAPES = [(9, 13, 9, 13), (16, 24, 8, 12), (11, 29, 6, 13), (23, 41, 9, 16), (30, 61, 7, 9), (20, 300, 5, 21),
          (9, 129, 9, 64), (9, 131, 5, 65), (70, 5, 67, 11), (5, 1, 3, 1), (8, 127, 8, 127), (6, 257, 5, 129),
          (12, 390, 3, 64), (14, 500, 4, 41)]


def _data(shape, dtype, seed):
    rng = np.random.default_rng(seed)
    if dtype == torch.uint8:
        return torch.from_numpy(rng.integers(0, 256, shape, dtype=np.uint8)).to(DEV)
    x = torch.from_numpy(rng.standard_normal(shape).astype(np.float32)).to(dtype)
    x.view(-1)[:: 4099] = float("inf")
    return x.to(DEV)


@pytest.mark.parametrize("mode", ["bilinear_aa", "bicubic_aa"])
@pytest.mark.parametrize("channels", [1, 4])
@pytest.mark.parametrize("dtype", [torch.uint8, torch.float16, torch.float32])
def test_walk_equals_gather(mode, channels, dtype):
    for k, (ih, iw, oh, ow) in enumerate(SHAPES):
        planes = min(max(1100, 300000 // (oh * ow)), 60000)  # past 2^18 results
        # rows of an odd pitch that start anywhere (whole pixels)
        whole = _data((planes, ih, iw + 3, channels), dtype, 100 + k)
        x = whole[:, :, 1:1 + iw]
        got = torch.empty((planes, oh, ow, channels), dtype=dtype, device=DEV)
        ref = torch.empty_like(got)
        xr.resize_into(x, got, mode)
        xr.resize_into(x, ref, mode, tile=GATHER)
        eq = (got == ref) | ((got != got) & (ref != ref))
        assert bool(eq.all()), (ih, iw, oh, ow, int((~eq).sum()))


def test_walk_band_of_an_image():
    """Output rows 300 .. 899 of a 4096 x 2000 image from the rows they need."""
    x = _data((4096, 2000, 4), torch.uint8, 7)
    first, last = xr.needed_rows(4096, 1500, 300, 600, "bicubic_aa")
    got = torch.empty((600, 700, 4), dtype=torch.uint8, device=DEV)
    whole = torch.empty((1500, 700, 4), dtype=torch.uint8, device=DEV)
    xr.resize_into(x[first:last + 1], got, "bicubic_aa", src_row0=first, src_height=4096, dst_row0=300,
                   dst_height=1500)
    xr.resize_into(x, whole, "bicubic_aa", tile=GATHER)
    assert torch.equal(got, whole[300:900])


@pytest.mark.parametrize("mode, ih, iw, oh, ow, planes, channels", [
    ("bilinear_aa", 135, 384, 16, 46, 96, 1), ("bicubic_aa", 300, 500, 40, 67, 1, 4), ("bicubic_aa", 301, 499, 23, 17, 3, 1)])
def test_small_outputs_with_large_windows(mode, ih, iw, oh, ow, planes, channels):
    x = _data((planes, ih, iw, channels), torch.float32, ow)
    got, ref = (torch.empty((planes, oh, ow, channels), dtype=torch.float32, device=DEV) for _ in range(2))
    xr.resize_into(x, got, mode)
    xr.resize_into(x, ref, mode, tile=GATHER)
    assert bool(((got == ref) | ((got != got) & (ref != ref))).all())
