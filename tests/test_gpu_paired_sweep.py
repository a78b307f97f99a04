"""GPU: the reverse sweep that runs the next segment's steps beside the adjoint
steps, in the same launches, against the sweep that runs them one after the
other (the same bits), for each tile shape and at the edges of the segments."""
import numpy as np
import pytest
import torch

from paper_2608_04085_amd import inputs
from paper_2608_04085_amd.config import CKPT_UNIFORM, RECON_BALANCED, RTConfig, paper_preset

pytestmark = pytest.mark.gpu

CASES = [RTConfig(nx=3, ny=2, batch=2), RTConfig(nx=61, ny=40, batch=3), RTConfig(nx=130, ny=250), RTConfig(nx=250, ny=254),
         paper_preset(62, batch=3).with_(recon=RECON_BALANCED), RTConfig(nx=5, ny=9, batch=1100)]


def host(t):
    return t.detach().cpu().numpy()


@pytest.mark.parametrize("mode", ["frozen", "differentiated"])
@pytest.mark.parametrize("cfg", CASES, ids=[f"{c.nx}x{c.ny}x{c.batch}" for c in CASES])
def test_paired_sweep_has_the_bits_of_the_one_after_the_other(cfg, mode):
    # members of different speeds end at different steps; the last segment is
    # whole, ragged or one step, with one step re-computed beside each adjoint
    # step, fewer (the rest follow) or none (segments of two after one step)
    from paper_2608_04085_amd import rtcnop
    amp = 3e-2 if cfg.lx == 0.5 else 1e-1
    uv = amp * np.random.default_rng(cfg.nx).standard_normal((cfg.batch, 2, cfg.ny, cfg.nx))
    uv = inputs.mask_components(uv, cfg.comp_mask) * np.linspace(0.1, 1.0, cfg.batch)[:, None, None, None]
    r = rtcnop.Context(cfg, max_steps=64)
    r.set_columns(rtcnop.FUSED_ADJOINT)
    r.set_dt_mode(mode)
    T = 10.4 * float(host(r.cfl_dt(r.init_state(uv))).min())
    n = int(host(r.integrate(r.init_state(uv), T)[2]).max())
    want = None
    for interval in (1, 2, 3, n - 1, n // 2, (n + 1) // 2):
        for on in (False, True):
            r.set_overlap(on)
            pool = torch.full(((r.pool_bytes(CKPT_UNIFORM, interval, n) + 256) // 8,), float("nan"),
                              dtype=torch.float64, device=r.device)
            got = [host(x) for x in r.grad_u0(uv, T, rtcnop.Policy(CKPT_UNIFORM, interval), pool=pool)]
            if want is None:
                want = got
            for a, b in zip(got, want):
                np.testing.assert_array_equal(a, b, err_msg=f"interval {interval} overlap {on} of {n} steps")
    r.check_error()
