"""GPU test of row pitches whose strips reach past 2 GiB: every value equals the
one-pixel-per-thread gather's, and nothing outside the view is written."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1001_1718_amd as xr  # noqa: E402

DEV = "cuda:0"
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
