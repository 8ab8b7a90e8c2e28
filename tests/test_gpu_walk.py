"""GPU test of the staged walk (general ratios, its default launch, and batches):
every value must equal, bit for bit, the one-pixel-per-thread gather's, whose
results tests/test_gpu_forward.py holds to the oracle (both evaluate the same
float32 sequence). The shapes sit at the walk's edges: images narrower than the
taps, outputs of one run, one tile of columns and its neighbours, rows at every
byte alignment, row ratios whose output rows share no tap rows, strips of one
row and longer than the image, staged rows near and past the LDS limit;
infinities in the sources."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1001_1718_amd as xr  # noqa: E402

DEV = "cuda:0"
GATHER = xr.tile(xr.XR_KERNEL_GATHER, 64, 4)
SHAPES = [(1, 1, 5, 4), (3, 2, 7, 9), (7, 5, 9, 16), (19, 40, 25, 51), (64, 300, 50, 257), (5, 515, 7, 513),
          (90, 33, 13, 31), (240, 100, 17, 90), (33, 700, 40, 180), (33, 2600, 40, 181), (12, 70, 75, 420)]


def _data(shape, dtype, seed):
    rng = np.random.default_rng(seed)
    if dtype == torch.uint8:
        return torch.from_numpy(rng.integers(0, 256, shape, dtype=np.uint8)).to(DEV)
    x = torch.from_numpy(rng.standard_normal(shape).astype(np.float32)).to(dtype)
    x.view(-1)[::4099] = float("inf")
    return x.to(DEV)


def _same(a, b):
    return bool(((a == b) | ((a != a) & (b != b))).all())


@pytest.mark.parametrize("mode", ["bilinear", "bicubic", "nearest"])
@pytest.mark.parametrize("channels", [1, 4])
@pytest.mark.parametrize("dtype", [torch.uint8, torch.float16, torch.float32])
def test_walk_equals_gather(mode, channels, dtype):
    for k, (ih, iw, oh, ow) in enumerate(SHAPES):
        # two planes whose rows have an odd pitch and start anywhere (whole
        # pixels), written into rows that do too
        x = _data((2, ih, iw + 3, channels), dtype, 300 + k)[:, :, 1:1 + iw]
        out = torch.zeros((2, oh, ow + 5, channels), dtype=dtype, device=DEV)
        ref = torch.empty((2, oh, ow, channels), dtype=dtype, device=DEV)
        for mapping in ("half_pixel", "paper"):
            xr.resize_into(x, ref, mode, tile=GATHER, mapping=mapping)
            ppx = (1, 2, 4) if channels == 4 else (4, 8, 16)
            for t in [None] + [xr.tile(xr.XR_KERNEL_STRIP, 64, 2, p, h, o) for p in ppx for h, o in ((1, 0), (37, 1))]:
                out.zero_()
                xr.resize_into(x, out[:, :, 2:2 + ow], mode, tile=t, mapping=mapping)
                assert _same(out[:, :, 2:2 + ow], ref), (ih, iw, oh, ow, mapping, t)
                assert not bool(out[:, :, :2].any()) and not bool(out[:, :, 2 + ow:].any())


@pytest.mark.parametrize("dtype", [torch.uint8, torch.float16, torch.float32])
def test_batch_equals_gather(dtype):
    pairs = []
    for k, (ih, iw, oh, ow) in enumerate(SHAPES + [(40, 60, 41, 1)]):
        for channels in (1, 4):
            x = _data((ih, iw, channels), dtype, 500 + k)
            for mode in ("bilinear", "bicubic"):
                pairs.append((x, torch.empty((oh, ow, channels), dtype=dtype, device=DEV), mode))
    for t in (None, xr.tile(xr.XR_KERNEL_STRIP, 64, 4, 0, 3), xr.tile(xr.XR_KERNEL_STRIP, 128, 1, 0, 256)):
        for _, d, _ in pairs:
            d.zero_()
        xr.Batch(pairs, tile=t).run()
        for x, d, mode in pairs:
            ref = torch.empty_like(d)
            xr.resize_into(x, ref, mode, tile=GATHER)
            assert _same(d, ref), (tuple(x.shape), tuple(d.shape), mode, t)


def test_walk_near_the_lds_limit():
    # float32 RGBA rows of just under and over 4 KiB per wavefront: workgroups
    # of the default tile then hold fewer wavefronts, or the walk does not apply
    for iw, ow in [(720, 184), (735, 184), (1500, 380), (1600, 400), (1700, 400)]:
        x = _data((41, iw, 4), torch.float32, iw)
        ref, out = (torch.empty((300, ow, 4), dtype=torch.float32, device=DEV) for _ in range(2))
        for mode in ("bilinear", "bicubic"):
            xr.resize_into(x, ref, mode, tile=GATHER)
            for t in (None, xr.tile(xr.XR_KERNEL_STRIP, 64, 4, 1, 256), xr.tile(xr.XR_KERNEL_STRIP, 256, 1, 1, 9)):
                out.zero_()
                xr.resize_into(x, out, mode, tile=t)
                assert _same(out, ref), (iw, ow, mode, t)
            for t in (None, xr.tile(xr.XR_KERNEL_STRIP, 64, 4, 0, 256)):
                out.zero_()
                xr.Batch([(x, out, mode)], tile=t).run()
                assert _same(out, ref), (iw, ow, mode, t)


@pytest.mark.parametrize("dtype", [torch.uint8, torch.float16, torch.float32])
@pytest.mark.parametrize("kinds", [(("bilinear", 1), ("bicubic", 4)), (("bilinear", 4), ("bicubic", 4)),
                                   (("bicubic", 1),), (("bilinear", 1), ("bilinear", 4), ("bicubic", 1))])
def test_batch_of_some_kinds(kinds, dtype):
    """Uneven counts of tiles per kind; jobs of long staged rows among short ones."""
    pairs = []
    for n, (mode, channels) in enumerate(kinds):
        for k in range(1 + 5 * n):
            ih, iw, oh, ow = (20 + 7 * k, 900 + 31 * k, 33, 270 - k) if k % 4 == 0 else (9 + k, 40 + 9 * k, 31 + k, 77)
            x = _data((ih, iw, channels), dtype, 900 + 10 * n + k)
            pairs.append((x, torch.zeros((oh, ow, channels), dtype=dtype, device=DEV), mode))
    for t in (None, xr.tile(xr.XR_KERNEL_STRIP, 192, 1, 0, 5), xr.tile(xr.XR_KERNEL_STRIP, 64, 3, 0, 256)):
        for _, d, _ in pairs:
            d.zero_()
        xr.Batch(pairs, tile=t).run()
        for x, d, mode in pairs:
            ref = torch.empty_like(d)
            xr.resize_into(x, ref, mode, tile=GATHER)
            assert _same(d, ref), (tuple(x.shape), tuple(d.shape), mode, t)
