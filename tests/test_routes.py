"""Which kernel a call runs, on both sides of every rule of the dispatch (no GPU)."""

import pytest

import paper_1001_1718_amd as xr
from route_util import SRC, route, route_backward

U8, F16, F32 = xr.XR_U8, xr.XR_F16, xr.XR_F32
MIB = 1 << 20

FORWARD = [
    # the exact-ratio kernels; on unaligned rows, under the printed map and for
    # nearest neighbour the general ones; at very long pitches too
    ("x2", dict(mode="bicubic", dtype=U8, in_hw=(4096, 4096), out_hw=(8192, 8192), channels=4)),
    ("walk", dict(mode="bicubic", dtype=U8, in_hw=(4096, 4096), out_hw=(8192, 8192), src_data=SRC + 1)),
    ("walk", dict(mode="bicubic", dtype=U8, in_hw=(4096, 4096), out_hw=(8192, 8192), channels=4, mapping="paper")),
    ("walk", dict(mode="nearest", dtype=F16, in_hw=(4096, 4096), out_hw=(8192, 8192), channels=4)),
    ("x05", dict(mode="bicubic", dtype=F16, in_hw=(4096, 4096), out_hw=(2048, 2048), channels=4)),
    ("x2", dict(mode="bicubic", dtype=F32, in_hw=(64, 64), out_hw=(128, 128), dst_pitch=120 * MIB)),
    ("strip", dict(mode="bicubic", dtype=F32, in_hw=(64, 64), out_hw=(128, 128), dst_pitch=128 * MIB)),
    # small one-channel uint8 images at x2 (the x2 kernel moves dwords of source)
    ("walk", dict(mode="bilinear", dtype=U8, in_hw=(512, 512), out_hw=(1024, 1024))),
    # general ratios: the staged walk from 1700 runs of 256 columns (2100 of 128 RGBA pixels) on
    ("walk", dict(mode="bicubic", dtype=U8, in_hw=(1500, 200), out_hw=(1700, 256))),
    ("strip", dict(mode="bicubic", dtype=U8, in_hw=(1500, 200), out_hw=(1699, 256))),
    ("walk", dict(mode="bicubic", dtype=F32, in_hw=(1500, 100), out_hw=(2100, 128), channels=4)),
    ("strip", dict(mode="bicubic", dtype=F32, in_hw=(1500, 100), out_hw=(2099, 128), channels=4)),
    ("walk", dict(mode="bicubic", dtype=F32, in_hw=(512, 512), out_hw=(768, 768), planes=48)),
    ("walk", dict(mode="bicubic", dtype=F32, in_hw=(3000, 4000), out_hw=(1080, 1440), channels=4)),
    # (later where the per-tap strips are the faster ones)
    ("walk", dict(mode="nearest", dtype=U8, in_hw=(1500, 200), out_hw=(2600, 256))),
    ("strip", dict(mode="nearest", dtype=F16, in_hw=(1500, 200), out_hw=(2599, 256))),
    ("walk", dict(mode="nearest", dtype=F32, in_hw=(1500, 200), out_hw=(1700, 256))),
    ("walk", dict(mode="nearest", dtype=U8, in_hw=(1500, 100), out_hw=(3400, 128), channels=4)),
    ("strip", dict(mode="nearest", dtype=F16, in_hw=(1500, 100), out_hw=(3399, 128), channels=4)),
    ("walk", dict(mode="bilinear", dtype=F16, in_hw=(1500, 100), out_hw=(2600, 128), channels=4)),
    ("strip", dict(mode="bilinear", dtype=F16, in_hw=(1500, 100), out_hw=(2599, 128), channels=4)),
    ("walk", dict(mode="bicubic", dtype=F16, in_hw=(1500, 65), out_hw=(3500, 128), channels=4)),
    ("strip", dict(mode="bicubic", dtype=F16, in_hw=(1500, 65), out_hw=(3499, 128), channels=4)),
    ("walk", dict(mode="bicubic", dtype=F16, in_hw=(1500, 64), out_hw=(2100, 128), channels=4)),
    ("strip", dict(mode="bilinear", dtype=F32, in_hw=(1500, 128), out_hw=(3499, 128), channels=4)),
    ("walk", dict(mode="bilinear", dtype=F32, in_hw=(1500, 129), out_hw=(2100, 128), channels=4)),
    # copies of RGBA bytes into outputs of 2^23 pixels and more
    ("strip", dict(mode="nearest", dtype=U8, in_hw=(2000, 2000), out_hw=(2048, 4096), channels=4)),
    ("walk", dict(mode="nearest", dtype=U8, in_hw=(2000, 2000), out_hw=(2047, 4096), channels=4)),
    ("walk", dict(mode="nearest", dtype=U8, in_hw=(2000, 4097), out_hw=(2048, 4096), channels=4)),
    # row pitches past 4 MiB, rows too long for LDS, outputs narrower than a run
    ("walk", dict(mode="bicubic", dtype=U8, in_hw=(3000, 2000), out_hw=(4000, 2600), dst_pitch=4 * MIB)),
    ("strip", dict(mode="bicubic", dtype=U8, in_hw=(3000, 2000), out_hw=(4000, 2600), dst_pitch=5 * MIB)),
    ("strip", dict(mode="bicubic", dtype=F32, in_hw=(3000, 32000), out_hw=(4000, 3200), channels=4)),
    ("strip", dict(mode="bicubic", dtype=U8, in_hw=(3000, 3), out_hw=(4000, 2))),
    # named kernels
    ("gather", dict(mode="bicubic", dtype=U8, in_hw=(512, 512), out_hw=(1024, 1024),
                    tile=xr.tile(xr.XR_KERNEL_GATHER, 64, 4))),
    ("strip", dict(mode="bicubic", dtype=U8, in_hw=(512, 512), out_hw=(1024, 1024),
                   tile=xr.tile(xr.XR_KERNEL_STRIP_ANY, 64, 4, 8, 8))),
    ("walk", dict(mode="bicubic", dtype=U8, in_hw=(700, 900), out_hw=(1000, 1300),
                  tile=xr.tile(xr.XR_KERNEL_STRIP, 64, 4, 4, 8))),
    # (on small outputs only where the walk is the faster one)
    ("strip", dict(mode="bicubic", dtype=F16, in_hw=(600, 800), out_hw=(200, 270), channels=4,
                   tile=xr.tile(xr.XR_KERNEL_STRIP, 64, 4, 2, 2))),
    ("walk", dict(mode="bicubic", dtype=F16, in_hw=(600, 800), out_hw=(200, 270), channels=4, planes=6,
                  tile=xr.tile(xr.XR_KERNEL_STRIP, 64, 4, 2, 2))),
    ("strip", dict(mode="bicubic", dtype=F32, in_hw=(600, 800), out_hw=(200, 270),
                   tile=xr.tile(xr.XR_KERNEL_STRIP, 64, 4, 4, 6))),
    ("walk", dict(mode="bicubic", dtype=F32, in_hw=(600, 800), out_hw=(200, 270),
                  tile=xr.tile(xr.XR_KERNEL_STRIP, 64, 4, 4, 2))),
    ("walk", dict(mode="bicubic", dtype=U8, in_hw=(600, 800), out_hw=(200, 270),
                  tile=xr.tile(xr.XR_KERNEL_STRIP, 64, 4, 4, 6))),
    ("walk", dict(mode="bicubic", dtype=F32, in_hw=(200, 300), out_hw=(300, 450),
                  tile=xr.tile(xr.XR_KERNEL_STRIP, 64, 4, 4, 6))),
    ("error 11", dict(mode="bicubic", dtype=F32, in_hw=(4, 32768), out_hw=(4, 64),
                      tile=xr.tile(xr.XR_KERNEL_STRIP_LDS, 512, 1, 8, 4))),
    # antialiased: the walk from 2^18 results on, where rows shrink or stay; not
    # for a few columns of many samples
    ("aa walk", dict(mode="bilinear_aa", dtype=U8, in_hw=(700, 1024), out_hw=(512, 512))),
    ("aa tile", dict(mode="bilinear_aa", dtype=U8, in_hw=(700, 1024), out_hw=(511, 512))),
    ("aa walk", dict(mode="bicubic_aa", dtype=U8, in_hw=(512, 300), out_hw=(512, 600))),
    ("aa tile", dict(mode="bicubic_aa", dtype=U8, in_hw=(511, 300), out_hw=(512, 600))),
    ("aa walk", dict(mode="bilinear_aa", dtype=U8, in_hw=(60, 200), out_hw=(30, 24), planes=512)),
    ("aa tile", dict(mode="bilinear_aa", dtype=U8, in_hw=(60, 200), out_hw=(30, 23), planes=512)),
    # (from more results on for one-channel bicubic columns, by samples and type)
    ("aa walk", dict(mode="bicubic_aa", dtype=F32, in_hw=(1820, 1820), out_hw=(640, 1024))),
    ("aa tile", dict(mode="bicubic_aa", dtype=F32, in_hw=(1820, 2926), out_hw=(639, 1024))),
    ("aa walk", dict(mode="bicubic_aa", dtype=F16, in_hw=(1380, 2926), out_hw=(480, 1024))),
    ("aa tile", dict(mode="bicubic_aa", dtype=F16, in_hw=(1380, 2926), out_hw=(479, 1024))),
    ("aa walk", dict(mode="bicubic_aa", dtype=F32, in_hw=(1800, 4096), out_hw=(448, 1024))),
    ("aa tile", dict(mode="bicubic_aa", dtype=F32, in_hw=(1800, 4096), out_hw=(447, 1024))),
    ("aa walk", dict(mode="bicubic_aa", dtype=U8, in_hw=(1800, 4096), out_hw=(384, 1024))),
    ("aa tile", dict(mode="bicubic_aa", dtype=U8, in_hw=(1800, 4096), out_hw=(383, 1024))),
    ("aa walk", dict(mode="bicubic_aa", dtype=F16, in_hw=(768, 2048), out_hw=(384, 1024))),
    ("aa tile", dict(mode="bicubic_aa", dtype=F16, in_hw=(768, 2048), out_hw=(383, 1024))),
    ("aa walk", dict(mode="bilinear_aa", dtype=F32, in_hw=(1280, 4096), out_hw=(320, 1024))),
    ("aa tile", dict(mode="bilinear_aa", dtype=F32, in_hw=(1280, 4096), out_hw=(319, 1024))),
    ("aa walk", dict(mode="bicubic_aa", dtype=F16, in_hw=(400, 1300), out_hw=(308, 1024), channels=4)),
    ("aa tile", dict(mode="bicubic_aa", dtype=F16, in_hw=(400, 1300), out_hw=(307, 1024), channels=4)),
    ("aa gather", dict(mode="bicubic_aa", dtype=F32, in_hw=(8000, 500), out_hw=(20, 20), channels=4)),
]


@pytest.mark.parametrize("want, call", FORWARD)
def test_forward_route(want, call):
    assert route(**call) == want


@pytest.mark.parametrize("want, call", [
    ("adjoint x2", dict(mode="bilinear", dtype=F32, in_hw=(64, 64), out_hw=(128, 128))),
    ("adjoint walk", dict(mode="bilinear", dtype=F32, in_hw=(512, 512), out_hw=(768, 768))),
    ("adjoint owner", dict(mode="bilinear", dtype=F32, in_hw=(511, 512), out_hw=(768, 768))),
    ("adjoint walk", dict(mode="bicubic", dtype=F16, in_hw=(480, 640), out_hw=(360, 480), channels=4)),
    ("adjoint walk", dict(mode="bicubic", dtype=F32, in_hw=(352, 1024), out_hw=(1100, 3000))),
    ("adjoint owner", dict(mode="bicubic", dtype=F32, in_hw=(351, 1024), out_hw=(1100, 3000))),
    ("adjoint walk", dict(mode="bicubic", dtype=F32, in_hw=(80, 1024), out_hw=(250, 3000), planes=8)),
    ("adjoint owner", dict(mode="bicubic", dtype=F32, in_hw=(79, 1024), out_hw=(250, 3000), planes=8)),
])
def test_adjoint_route(want, call):
    assert route_backward(**call) == want


def test_lds_tiles_are_taken_as_documented():
    """XR_KERNEL_STRIP_LDS: the row segment of a workgroup's bw ppt_x columns, in
    chunks of 4 bytes or a pixel, needs at most 64 bytes a lane and 64 KiB for
    three rows; pixels under 4 bytes lie in rows of whole words."""
    taken = refused = 0
    for mode, taps in (("nearest", 1), ("bilinear", 2), ("bicubic", 4)):
        for dtype, size in ((U8, 1), (F16, 2), (F32, 4)):
            for channels, ppx in ((1, 8), (4, 4)):
                for bw in (64, 192, 512):
                    for in_w, out_w in ((37, 74), (36, 75), (300, 40), (4096, 300), (32768, 64), (640, 5600), (8192, 1100)):
                        px = size * channels
                        chunk = max(px, 4)
                        seg = (min(bw * ppx, out_w) - 1) * in_w // out_w + taps + 1
                        chunks = -(-(seg * px + chunk - px) // chunk)
                        fits = (-(-chunks // bw) <= 64 // chunk and 3 * (-(-chunks * chunk // 16) * 16) <= 65536 and
                                (px >= 4 or in_w * px % 4 == 0))
                        got = route(mode, dtype, (50, in_w), (70, out_w), channels,
                                    tile=xr.tile(xr.XR_KERNEL_STRIP_LDS, bw, 1, ppx, 6))
                        assert fits == (got != "error 11")
                        taken, refused = taken + fits, refused + (not fits)
    assert taken > 100 and refused > 100


@pytest.mark.parametrize("mode, dtype, channels, in_hw, out_hw, ppt_x, rows", [
    ("bicubic", U8, 1, (3507, 2479), (4559, 3223), 4, 16), ("bilinear", U8, 4, (800, 800), (4700, 4700), 2, 16),
    ("nearest", F16, 4, (2600, 2860), (3380, 3716), 2, 8), ("bilinear", F16, 4, (2600, 2860), (3380, 3716), 2, 8),
    ("bicubic", F16, 4, (2600, 2860), (3380, 3716), 2, 16), ("bilinear", F32, 4, (2600, 2860), (3380, 3716), 1, 16),
    ("bicubic", F16, 4, (2600, 2860), (780, 856), 1, 2), ("bilinear", F16, 4, (4000, 6000), (1818, 2727), 1, 4),
    ("bicubic", F16, 4, (2600, 2860), (1300, 1431), 2, 4)])
def test_default_strips_of_the_walk(mode, dtype, channels, in_hw, out_hw, ppt_x, rows):
    t = xr.get_tile(mode, dtype, channels, in_hw[1], in_hw[0], out_hw[1], out_hw[0])
    assert t.as_tuple() == (xr.XR_KERNEL_STRIP, 64, 4, ppt_x, rows, 0)
