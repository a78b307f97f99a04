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
