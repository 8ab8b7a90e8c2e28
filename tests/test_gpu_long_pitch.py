"""GPU test of row pitches whose strips reach past 2 GiB: every value equals the
one-pixel-per-thread gather's, and nothing outside the view is written."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1001_1718_amd as xr  # noqa: E402
from oracle import ref_resize as R  # noqa: E402

DEV = "cuda:0"
MODES = {"bilinear": 0, "bicubic": 1}
GATHER = xr.tile(xr.XR_KERNEL_GATHER, 64, 4)


def _bytes(shape, seed):
    return torch.from_numpy(np.random.default_rng(seed).integers(1, 256, shape, dtype=np.uint8)).to(DEV)


@pytest.mark.parametrize("mode", ["bilinear", "bicubic"])
@pytest.mark.parametrize("rows, pitch", [(40, 96 << 20), (5, 1 << 30), (2, 1 << 31)])
def test_batch_into_rows_of_a_long_pitch(mode, rows, pitch):
    """An output whose last run of columns ends past the image's edge, so that
    lanes of the last wavefront have no columns."""
    x = _bytes((23, 50, 1), 3)
    wide = torch.zeros((rows, pitch, 1), dtype=torch.uint8, device=DEV)
    out = wide[:, 256:256 + 70]
    ref = torch.empty((rows, 70, 1), dtype=torch.uint8, device=DEV)
    xr.resize_into(x, ref, mode, tile=GATHER)
    for t in (None, xr.tile(xr.XR_KERNEL_STRIP, 64, 1, 0, 256)):
        out.zero_()
        xr.Batch([(x, out, mode)], tile=t).run()
        assert torch.equal(out, ref)
        assert int(torch.count_nonzero(wide)) == int(torch.count_nonzero(ref))


@pytest.mark.parametrize("mode", ["bilinear", "bicubic"])
@pytest.mark.parametrize("in_hw, out_hw, pitch", [((7, 33), (14, 66), 120 << 20), ((7, 33), (14, 66), 160 << 20),
                                                  ((10, 66), (5, 33), 180 << 20), ((6, 66), (3, 33), 1 << 30)])
def test_exact_ratios_into_rows_of_a_long_pitch(mode, in_hw, out_hw, pitch):
    x = _bytes((*in_hw, 4), 5)
    wide = torch.zeros((out_hw[0], pitch // 4, 4), dtype=torch.uint8, device=DEV)
    out = wide[:, 64:64 + out_hw[1]]
    ref = torch.empty((*out_hw, 4), dtype=torch.uint8, device=DEV)
    xr.resize_into(x, ref, mode, tile=GATHER)
    xr.resize_into(x, out, mode)
    assert torch.equal(out, ref)
    assert int(torch.count_nonzero(wide)) == int(torch.count_nonzero(ref))


@pytest.mark.parametrize("mode", ["bilinear", "bicubic"])
def test_adjoint_at_x2_into_rows_of_a_long_pitch(mode):
    """Gradient rows 160 MiB apart; each value is a float32 sum of at most 64
    products (the suite's bound, 1e-5 of their magnitudes)."""
    g = np.random.default_rng(7).standard_normal((12, 40)).astype(np.float32)
    wide = torch.zeros((6, 40 << 20), dtype=torch.float32, device=DEV)
    got = xr.resize_backward(torch.from_numpy(g).to(DEV), (6, 20), mode, layout="hwc", out=wide[:, 8:28]).cpu().numpy()
    ref = R.adjoint(g[None, :, :, None], 6, 20, MODES[mode])[0, :, :, 0]
    bound = 1e-5 * R.adjoint(g[None, :, :, None], 6, 20, MODES[mode], absolute=True)[0, :, :, 0]
    assert np.all(np.abs(got - ref) <= bound)
    assert int(torch.count_nonzero(wide)) == np.count_nonzero(got)
