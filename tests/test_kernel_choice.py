"""CPU: which kernels a context runs, as the library chooses them from the
grid and as its settings change them (no device work)."""
import ctypes

import pytest

from paper_2608_04085_amd import rtcnop

NAMES = {v: k for k, v in rtcnop.TILES.items()}


class Bare:
    """A context without a workspace, through the C ABI."""

    def __init__(self, nx, ny, nb, recon=0):
        self.L, self.h = rtcnop.load(), ctypes.c_void_p()
        g = rtcnop.RtGrid(nx, ny, nb, 0, 0.5, 1.0)
        p = rtcnop.RtPhys(1.4, -0.1, 2.0, 1.0, 0.5, 0.01, 2.5, 0.4, 3, recon)
        assert self.L.rt_create(ctypes.byref(g), ctypes.byref(p), None, ctypes.byref(self.h)) == 0

    def __del__(self):
        self.L.rt_destroy(self.h)

    @property
    def fold(self):
        v = ctypes.c_int32()
        assert self.L.rt_get_fold(self.h, ctypes.byref(v)) == 0
        return v.value

    def set_fold(self, on):
        assert self.L.rt_set_fold(self.h, on) == 0

    @property
    def kernels(self):
        m, s, a = ctypes.c_int32(), ctypes.c_int32(), ctypes.c_int32()
        assert self.L.rt_get_columns(self.h, ctypes.byref(m)) == 0
        assert self.L.rt_get_tiles(self.h, ctypes.byref(s), ctypes.byref(a)) == 0
        m = m.value
        step = "columns" if m & rtcnop.COLUMNS_STEP else NAMES[s.value]
        adj = "columns" if m & rtcnop.COLUMNS_ADJOINT else "fused" if m & rtcnop.FUSED_ADJOINT else NAMES[a.value]
        return f"{step}/{adj}"


@pytest.mark.parametrize("grid", [(64, 128, 1), (256, 512, 1), (512, 512, 1), (512, 1024, 8)])
def test_setting_the_fold_and_back_leaves_the_default_kernels(grid):
    c = Bare(*grid)
    default, fold = c.kernels, c.fold
    assert default.endswith(("fused", "columns"))
    c.set_fold(fold)
    assert (c.kernels, c.fold) == (default, fold)
    for _ in range(2):
        c.set_fold(1 - fold)
        assert c.fold == 1 - fold
        c.set_fold(fold)
        assert (c.kernels, c.fold) == (default, fold)
    # kernels that the caller chose: folding takes the tiles, and unfolding
    # keeps them
    assert c.L.rt_set_columns(c.h, rtcnop.FUSED_ADJOINT) == 0
    c.set_fold(0)
    assert c.kernels.endswith("/fused")
    for on in (1, 0):
        c.set_fold(on)
        assert c.kernels.split("/")[1] in rtcnop.TILES and c.fold == on


# The kernels of grids of which each form is the fastest: measured times of
# the given-dt step and of the adjoint in us, (columns, tiles) and (columns,
# fused, tile pair)
@pytest.mark.parametrize("grid,want", [
    ((16, 64, 1024), "16x15/fused"),      # 67, 42; 141, 83, 88
    ((16, 32, 4096), "16x15/fused"),      # 130, 90; 273, 167, 216
    ((5, 248, 1095), "16x15/16x15"),      # 459, 147; 954, 272, 258
    ((3, 10, 39250), "16x15/16x15"),      # 385, 297; 888, 633, 449
    ((9, 481, 144), "16x15/16x15"),       # 73, 40; 159, 92, 76
    ((3, 9, 1064), "8x8w/8x8w"),          # 22, 11; 42, 24, 19
    ((24, 48, 2048), "columns/fused"),    # 99, 125; 213, 206, 292
    ((44, 902, 54), "columns/columns"),   # 59, 78; 125, 186, 205
    ((56, 2, 9059), "columns/columns"),   # 27, 223; 61, 465, 286
    ((77, 149, 16), "columns/fused"),     # 14, 15 (16x8); a tile rule of few rounds took the latter
    ((64, 128, 40), "columns/columns"),
    ((128, 256, 64), "columns/columns"),
    ((61, 40, 3), "8x8w/fused"),
])
def test_default_kernels_of_narrow_grids_and_large_batches(grid, want):
    assert Bare(*grid).kernels == want
