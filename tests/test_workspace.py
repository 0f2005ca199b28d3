"""The least workspace of flr_denoise (flr_denoise_min_workspace_bytes) and the
calls between it and the preferred one, on the host (nothing is launched)."""
import ctypes

import pytest

from paper_2410_11625_amd import _lib
from paper_2410_11625_amd._lib import FlrParams

FUSED, TWO_PASS = 1, 2


def _p(H, W, Q, C, r, path=FUSED, average=1):
    return FlrParams(height=H, width=W, num_guides=Q, num_channels=C, radius=r, eps=1e-3,
                     eps_mul=0.0, reg_mode=0, average_coeffs=average, fused=path, flags=0,
                     tile_rows=0)


@pytest.fixture(scope="module")
def L():
    return _lib.lib()


def _sizes(L, p):
    return (L.flr_denoise_workspace_bytes(ctypes.byref(p)),
            L.flr_denoise_min_workspace_bytes(ctypes.byref(p)))


def test_ring_of_large_frames(L):
    # per workgroup 2r + 1 rows of (Q+1) C 256 floats; the image grows with the
    # frame, the ring with the workgroups
    for H, W, Q, C in ((1080, 1920, 8, 3), (1080, 1920, 12, 3), (4096, 4096, 3, 1)):
        need, least = _sizes(L, _p(H, W, Q, C, 8))
        assert 0 < least < need and least % (17 * (Q + 1) * C * 1024) == 0, (need, least)
    need, least = _sizes(L, _p(8192, 8192, 8, 3, 8))
    assert least < need // 20


@pytest.mark.parametrize("p", [
    _p(64, 96, 4, 1, 8),                        # a ring larger than the image
    _p(1080, 1920, 5, 3, 8),                    # channels the one-kernel form cannot hold
    _p(1080, 1920, 8, 3, 8, path=TWO_PASS), _p(1080, 1920, 8, 3, 8, path=0),
    _p(1080, 1920, 8, 3, 8, average=0), _p(0, 5, 3, 1, 2)])
def test_no_less_elsewhere(L, p):
    need, least = _sizes(L, p)
    assert least == need


def test_too_small_is_refused(L):
    g, y, o, ws = 0x10000000000, 0x20000000000, 0x30000000000, 0x40000000000
    for p in (_p(1080, 1920, 8, 3, 8), _p(1080, 1920, 5, 3, 8), _p(64, 96, 4, 1, 8)):
        need, least = _sizes(L, p)
        st = L.flr_denoise(ctypes.byref(p), g, y, o, ws, least - 1, None)
        assert st == 8, (need, least, st)       # FLR_ERR_WORKSPACE, before any launch


def test_flnr_takes_the_smaller_form(L):
    g, y, k, o, ws = (i << 40 for i in range(1, 6))
    p = _p(1080, 1920, 12, 3, 8)
    need, least = _sizes(L, p)
    net = L.flr_net_workspace_bytes(1080, 1920)
    assert L.flr_flnr_workspace_bytes(ctypes.byref(p)) == (need + 255) // 256 * 256 + net
    small = (least + 255) // 256 * 256 + net
    assert L.flr_flnr_denoise(ctypes.byref(p), g, y, k, o, ws, small - 1, None) == 8
    # enough: past the size check, on to the next one (here: a misaligned input)
    assert L.flr_flnr_denoise(ctypes.byref(p), g + 4, y, k, o, ws, small, None) == 7


def test_small_windows_on_small_frames_ask_for_the_ring(L):
    """One kernel: 2r + 1 rows of (Q+1) C 256 floats for each of the frame's
    rows; the coefficient image, where it is smaller, is still enough."""
    for H, W, Q, C, r in ((64, 96, 3, 1, 1), (64, 96, 6, 3, 0), (200, 160, 1, 3, 1)):
        need, least = _sizes(L, _p(H, W, Q, C, r))
        assert need == H * (2 * r + 1) * (Q + 1) * C * 1024
        assert least == min(need, (Q + 2) * C * H * W * 4)
    for H, W, Q, C, r in ((64, 96, 4, 1, 1), (64, 96, 1, 1, 2), (600, 96, 1, 1, 1)):
        need, _ = _sizes(L, _p(H, W, Q, C, r))
        assert need == (Q + 2) * C * H * W * 4
