"""GPU: the folded sweep of the tile kernels, which no grid runs by default,
against the two-kernel sweep and the default kernels (the same bits)."""
import numpy as np
import pytest

from paper_2608_04085_amd import inputs
from paper_2608_04085_amd.config import CKPT_STORE_ALL, CKPT_UNIFORM, RTConfig

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile", ["8x8w", "32x8", "16x15"])
def test_folded_sweep_has_the_bits_of_the_default_kernels(tile):
    # members of different step counts, several segments, a ragged last one
    from paper_2608_04085_amd import rtcnop
    cfg = RTConfig(nx=40, ny=72, batch=2)
    uv = inputs.seed_batch(cfg, [3, 4], rms=1e-3)
    uv[1] *= 40.0
    default = rtcnop.Context(cfg, max_steps=2048)
    want = [x.cpu().numpy() for x in default.grad_u0(uv, 0.2, rtcnop.Policy(CKPT_UNIFORM, 5))]
    assert default.kernels == "8x8w/fused" and want[2][0] != want[2][1]
    r = rtcnop.Context(cfg, max_steps=2048, tile=tile)
    for on, fold in ((True, True), (False, True), (True, False)):
        r.set_overlap(on)
        r.set_fold(fold)
        assert r.kernels == f"{tile}/{tile}" and r.fold == fold
        for pol in (rtcnop.Policy(CKPT_UNIFORM, 5), rtcnop.Policy(CKPT_STORE_ALL, 1)):
            for a, b in zip(r.grad_u0(uv, 0.2, pol), want):
                np.testing.assert_array_equal(a.cpu().numpy(), b)
    r.check_error()
