"""GPU: rt_step takes nothing from the workspace that an earlier call left
there: the CFL step of its result is right whatever the workspace holds."""
import numpy as np
import pytest
import torch

from paper_2608_04085_amd.config import RTConfig

pytestmark = pytest.mark.gpu


def host(t):
    return t.detach().cpu().numpy()


# one part of a member and many, of either step kernel: strips of one-row
# segments of a narrow grid are more than its 8x8 tiles; more than 256 and
# more than 2048 parts, which a block reads at once
@pytest.mark.parametrize("nx,ny,nb,tile", [(3, 2, 2, None), (5, 300, 1, "columns"), (64, 128, 3, None),
                                           (250, 254, 1, "16x15"), (130, 250, 9, "columns"), (61, 40, 3, "8x8"),
                                           (1000, 1100, 1, "columns"), (500, 300, 1, "8x8")])
def test_cfl_step_of_the_result_whatever_the_workspace_holds(nx, ny, nb, tile):
    from paper_2608_04085_amd import rtcnop
    cfg = RTConfig(nx=nx, ny=ny, batch=nb)
    r = rtcnop.Context(cfg, max_steps=8, tile=tile if tile in rtcnop.TILES else None)
    if tile == "columns":
        r.set_columns(rtcnop.COLUMNS_STEP)
    g = torch.Generator(device="cuda").manual_seed(5)
    U = r.init_state(0.03 * torch.randn(r.shape_uv, dtype=torch.float64, device="cuda", generator=g))
    dt = 0.5 * r.cfl_dt(U)
    want = r.step(U, dt)
    nxt = host(r.cfl_dt(want))
    # bytes that read as tiny, huge and not-a-number doubles
    for byte in (0x01, 0x7E, 0xFF):
        r.ws.fill_(byte)
        got, n = r.step(U, dt, want_next=True)
        assert torch.equal(got, want)
        np.testing.assert_array_equal(host(n), nxt, err_msg=f"workspace of bytes {byte:#x}")
