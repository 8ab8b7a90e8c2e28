"""GPU test of the adjoint's gather walk (taken where enough strips fill the
GPU): planes of a large stack must equal, bit for bit, the same planes passed
alone (too few strips, so the owner-computes kernel; both sum in one fixed
order), and the float64 oracle within the suite's float32 bound. The shapes sit
at the walk's edges: source rows and columns that no output touches, at the
borders and inside, one source row or column, one tap and more taps than
registers hold, one column tile and its neighbours."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1001_1718_amd as xr  # noqa: E402
from gpu_util import check_f16_sum, check_f32  # noqa: E402
from oracle import ref_resize as R  # noqa: E402
from synth import fields  # noqa: E402

DEV = "cuda:0"
MODES = {"bilinear": 0, "bicubic": 1}
SHAPES = [(9, 13, 9, 13), (8, 12, 12, 18), (6, 64, 4, 48), (5, 65, 7, 97), (70, 40, 9, 5), (1, 6, 9, 31), (7, 1, 3, 4),
          (9, 11, 1, 1), (67, 9, 100, 40), (3, 130, 4, 131),
          (4, 128, 5, 77), (5, 129, 3, 260), (3, 40, 4, 390)]


@pytest.mark.parametrize("mode", ["bilinear", "bicubic"])
@pytest.mark.parametrize("channels", [1, 4])
@pytest.mark.parametrize("dtype", [torch.float16, torch.float32])
def test_walk_equals_single_planes(mode, channels, dtype):
    for k, (ih, iw, oh, ow) in enumerate(SHAPES):
        planes = max(1100, 300000 // (ih * iw))  # past 2^18 results
        g = torch.from_numpy(fields.normal_f32((planes, oh, ow, channels), seed=50 + k)).to(dtype).to(DEV)
        got = xr.resize_backward(g, (ih, iw), mode, layout="hwc")
        for p in (0, 517, planes - 1):
            one = xr.resize_backward(g[p:p + 1], (ih, iw), mode, layout="hwc")
            assert torch.equal(got[p:p + 1], one), (ih, iw, oh, ow, p)
        gp = g[517:518].float().cpu().numpy()
        ref = R.adjoint(gp, ih, iw, MODES[mode])
        scale = R.adjoint(gp, ih, iw, MODES[mode], absolute=True)
        check = check_f32 if dtype == torch.float32 else check_f16_sum
        check(got[517:518].cpu().numpy(), ref, scale, what=f"adjoint walk {ih}x{iw}-{oh}x{ow}")
