"""GPU: which kernels a call launches, and how often, where a rule decides it
and either choice gives right results, by the names the profiler reports (in
a file that runs late: a profiler once used stays attached to the process)."""
import numpy as np
import pytest
import torch

from paper_2608_04085_amd.config import RTConfig

pytestmark = pytest.mark.gpu


def launched(call):
    """What call returns, and how often it launched each kernel (names up to the argument list)."""
    from torch.profiler import ProfilerActivity, profile
    call()
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as p:
        out = call()
        torch.cuda.synchronize()
    names = {}
    for e in p.key_averages():
        if "k_" in e.key:
            k = e.key[e.key.index("k_"):].split("(")[0].split("<")[0]
            names[k] = names.get(k, 0) + e.count
    assert names, "the profiler reported no kernel"
    return out, names


# lines with a large prime factor: a few of them (the direct kernels' blocks
# are more and shorter), many (the chip is full either way), and others
@pytest.mark.parametrize("nx,ny,nb,rows,cols", [
    (2042, 64, 1, "k_dft_rows", "k_dft_cols_split"), (2042, 2, 1, "k_dft_rows", "k_dft_cols_power"),
    (64, 2042, 1, "k_dft_rows_split", "k_dft_cols_power"), (2042, 64, 16, "k_dft_rows_split", "k_dft_cols_split"),
    (64, 2042, 16, "k_dft_rows_split", "k_dft_cols_split"), (16, 1006, 1, "k_dft_rows_split", "k_dft_cols_split"),
    (302, 300, 1, "k_dft_rows_split", "k_dft_cols_split"), (256, 256, 1, "k_dft_rows_split", "k_dft_cols_split")])
def test_two_stage_or_direct_spectra(nx, ny, nb, rows, cols):
    from paper_2608_04085_amd import rtcnop
    r = rtcnop.Context(RTConfig(nx=nx, ny=ny, batch=nb), max_steps=8)
    f = np.random.default_rng(nx + ny).standard_normal((nb, ny, nx))
    d = torch.from_numpy(f).cuda()
    got, names = launched(lambda: r.power_spectrum_2d(d))
    assert names == {rows: 1, cols: 1}
    # (the bound of the spectra's own test: n^1.5 1.2e-16 at the worst)
    E = np.abs(np.fft.rfft2(f)) ** 2
    assert np.all(np.abs(got.cpu().numpy().reshape(E.shape) - E) <= 1e-12 * E.max(axis=(1, 2), keepdims=True))


# differentiated steps: the launch that corrects lambda follows the last
# adjoint step alone while all tiles of the sweep are few, else every one
@pytest.mark.parametrize("nx,ny,nb,each", [(64, 128, 1, False), (61, 40, 3, False), (256, 256, 4, False),
                                           (256, 256, 5, True), (128, 128, 64, True), (520, 1100, 1, True)])
def test_launches_that_correct_lambda(nx, ny, nb, each):
    from paper_2608_04085_amd import rtcnop
    from paper_2608_04085_amd.config import CKPT_UNIFORM
    cfg = RTConfig(nx=nx, ny=ny, batch=nb)
    uv = 3e-2 * np.random.default_rng(nx).standard_normal((nb, 2, ny, nx)) * np.linspace(0.1, 1.0, nb)[:, None, None, None]
    r, tiles = rtcnop.Context(cfg, max_steps=64), rtcnop.Context(cfg, max_steps=64, tile="16x15")
    for c in (r, tiles):
        c.set_dt_mode("differentiated")
    T = 5.4 * float(r.cfl_dt(r.init_state(uv)).min())
    pol = rtcnop.Policy(CKPT_UNIFORM, 3)
    pool = torch.empty(r.pool_bytes(CKPT_UNIFORM, 3, 16) + 256, dtype=torch.uint8, device="cuda")
    got, names = launched(lambda: [x.cpu().numpy() for x in r.grad_u0(uv, T, pol, pool=pool)])
    assert names["k_dt_correct"] == (int(got[2].max()) if each else 1)
    # against the tile pair, which differs in the grouping of mu's sum alone:
    # 1e-16 times the root of its terms, over a few steps
    want = [x.cpu().numpy() for x in tiles.grad_u0(uv, T, pol, pool=pool)]
    np.testing.assert_array_equal(got[2], want[2])
    assert np.max(np.abs(got[1] - want[1])) <= 1e-11 * np.max(np.abs(want[1]))


@pytest.mark.parametrize("nx,ny,nb", [(64, 128, 1), (40, 72, 3)])
def test_rounds_of_a_march_whose_steps_shrink(nx, ny, nb):
    # a state at rest of even sound speed and uneven pressure: the flow that
    # starts takes the steps to less than half of the first
    from paper_2608_04085_amd import rtcnop
    cfg = RTConfig(nx=nx, ny=ny, batch=nb)
    r = rtcnop.Context(cfg, max_steps=1024)
    x, y = (np.arange(n) / n for n in (nx, ny))
    lp = np.exp(2.3 * np.sin(4 * np.pi * x) * np.sin(6 * np.pi * y)[:, None])
    U = r.init_state(torch.zeros(r.shape_uv, dtype=torch.float64))
    for b in range(nb):
        U[b, 0] = torch.from_numpy(lp)
        U[b, 3] = torch.from_numpy(2.5 * lp / 0.4) * (1.0 - 0.3 * b)
    dt0 = float(r.cfl_dt(U).min())
    for steps in (20, 100):
        (UT, _, n, _), names = launched(lambda: r.integrate(U, steps * dt0))
        assert int(n.max()) > 1.5 * steps
        # each round ends where the steps left at the last size suggest (2 %
        # more), so what remains shrinks at least threefold: 100 in five rounds
        assert names["k_report"] <= 6
        r.set_graphs(False)
        want = r.integrate(U, steps * dt0)
        r.set_graphs(True)
        assert torch.equal(UT, want[0]) and torch.equal(n, want[2])
    # a march beyond the step log is still refused
    few = rtcnop.Context(cfg, max_steps=int(n.max()) - 1)
    with pytest.raises(rtcnop.RTError) as e:
        few.integrate(U, 100 * dt0)
    assert e.value.code == -3
