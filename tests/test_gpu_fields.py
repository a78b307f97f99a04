"""GPU: reductions, projection and updates of velocity fields at the edges of
their rules: odd and even sizes (one or two elements a load), arrays that do
not start on 16 bytes, blocks with and without a full round of loads."""
import numpy as np
import pytest
import torch

from oracle.rto import Oracle
from paper_2608_04085_amd.config import RTConfig

pytestmark = pytest.mark.gpu

SHAPES = [(3, 3, 1), (5, 7, 3), (70, 37, 2), (64, 128, 1), (127, 131, 5), (258, 513, 2), (512, 1024, 1)]


def host(t):
    return t.detach().cpu().numpy()


def context(cfg):
    from paper_2608_04085_amd import rtcnop
    return rtcnop.Context(cfg, max_steps=8)


def shifted(a):
    """The array on the device, 8 bytes past an aligned address."""
    buf = torch.empty(a.size + 1, dtype=torch.float64, device="cuda")
    v = buf[1:].view(a.shape)
    v.copy_(torch.from_numpy(a))
    return v


@pytest.mark.parametrize("aligned", [True, False])
@pytest.mark.parametrize("nx,ny,nb", SHAPES)
def test_field_operations(nx, ny, nb, aligned):
    cfg = RTConfig(nx=nx, ny=ny, batch=nb)
    r = context(cfg)
    rng = np.random.default_rng(nx + ny)
    a, b = rng.standard_normal((2, nb, 2, ny, nx))
    al = rng.standard_normal(nb)
    da, db = (torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda()) if aligned else (shifted(a), shifted(b))
    # sums: at most 64 additions in a chain (16 per accumulator and block, the
    # rest trees), each with half an ulp of the sum of magnitudes
    la, lb = a.astype(np.longdouble), b.astype(np.longdouble)
    axes = (1, 2, 3)
    got = host(r.dot(da, db))
    assert np.all(np.abs(got - np.sum(la * lb, axes)) <= 64 * 1.2e-16 * np.sum(np.abs(la * lb), axes))
    assert np.array_equal(host(r.max_abs(da)), np.max(np.abs(a), axes))
    # x + alpha y: one rounding (fused) or two
    for alpha, col in ((al, al.reshape(-1, 1, 1, 1)), (-0.75, -0.75)):
        got = host(r.axpy(da, torch.from_numpy(alpha) if isinstance(alpha, np.ndarray) else alpha, db))
        assert np.all(np.abs(got - (a + col * b)) <= 2.3e-16 * (np.abs(a) + 2 * np.abs(col * b)))
    # the projection keeps its input and gives the oracle's scaled field: the
    # norm's sum (64 halves of an ulp on each side), square roots, quotient
    o = Oracle.from_config(cfg)
    for norm in (0, 1, 2):
        for kind in (0, 1):
            for delta in (0.5, 1e6):
                got, m = r.project_to_constraint(da, delta, norm, kind)
                ref, mo = o.project_to_constraint(a, delta, norm, kind)
                assert np.allclose(host(m), mo, rtol=1e-13, atol=0), (norm, kind)
                assert np.allclose(host(got), ref, rtol=1e-13, atol=0), (norm, kind, delta)
    assert np.array_equal(host(da), a)


def test_projection_in_place_and_masks():
    # the in-place entry gives the bits of the other; a component that does
    # not take part is zero in the result and out of the norm, whatever it holds
    import ctypes
    from paper_2608_04085_amd import rtcnop
    cfg = RTConfig(nx=30, ny=17, batch=2).with_(comp_mask=1)
    r = context(cfg)
    u = torch.randn(2, 2, 17, 30, dtype=torch.float64, device="cuda")
    u[:, 1, 3, 4] = float("nan")
    out, m = r.project_to_constraint(u, 0.25)
    w, mw = u.clone(), torch.empty_like(m)
    assert rtcnop.load().rt_project_to_constraint(r._h, ctypes.c_void_p(w.data_ptr()), 0.25, 0, 0,
                                                  ctypes.c_void_p(mw.data_ptr())) == 0
    assert torch.equal(out, w) and torch.equal(m, mw)
    assert not out[:, 1].any() and bool(torch.isfinite(out).all())
