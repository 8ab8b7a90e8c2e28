"""Names the kernel a call runs (xr_internal_route in the library; no HIP call)."""

import ctypes

import paper_1001_1718_amd as xr
from paper_1001_1718_amd import _lib

ROUTES = ["", "gather", "strip", "walk", "x2", "x05", "aa gather", "aa tile", "aa walk", "adjoint x2", "adjoint owner",
          "adjoint walk"]
SRC, DST = 0x7F0000000000, 0x7E0000000000  # never dereferenced

_img, _tile, _i32 = ctypes.POINTER(_lib.XrImage), ctypes.POINTER(_lib.XrTile), ctypes.c_int32
_lib.lib.xr_internal_route.argtypes = [_img, _img, _i32, _i32, _tile, _tile]
_lib.lib.xr_internal_route_backward.argtypes = [_img, _img, _i32]


def picture(data, h, w, channels, dtype, planes=1, pitch=None):
    size = {xr.XR_U8: 1, xr.XR_F16: 2, xr.XR_F32: 4}[dtype]
    pitch = pitch or w * channels * size
    return _lib.XrImage(data, w, h, channels, dtype, pitch, planes, pitch * h if planes > 1 else 0, 0, h)


def _name(code):
    return ROUTES[code] if code > 0 else f"error {-code}"


def route(mode, dtype, in_hw, out_hw, channels=1, planes=1, tile=None, mapping="half_pixel", src_pitch=None,
          dst_pitch=None, src_data=SRC):
    s, d = picture(src_data, *in_hw, channels, dtype, planes, src_pitch), picture(DST, *out_hw, channels, dtype, planes,
                                                                                  dst_pitch)
    return _name(_lib.lib.xr_internal_route(s, d, xr.filter_code(mode), xr.mapping_code(mapping), tile, None))


def route_backward(mode, dtype, in_hw, out_hw, channels=1, planes=1):
    g, s = picture(SRC, *out_hw, channels, dtype, planes), picture(DST, *in_hw, channels, dtype, planes)
    return _name(_lib.lib.xr_internal_route_backward(g, s, xr.filter_code(mode)))


def shape(mode, dtype, in_hw, out_hw, channels=1, mapping="half_pixel", src_data=SRC):
    """The shape that an AUTO call resolves to."""
    s, d, t = picture(src_data, *in_hw, channels, dtype), picture(DST, *out_hw, channels, dtype), _lib.XrTile()
    assert _lib.lib.xr_internal_route(s, d, xr.filter_code(mode), xr.mapping_code(mapping), None, t) > 0
    return t.as_tuple()
