"""GPU: the column kernels and the fused adjoint against the tile kernels (the
same bits: all evaluate the same expressions) and against the oracle, at the
edges of their strips, row segments and tiles and of the grid."""
import numpy as np
import pytest
import torch

from oracle.rto import Oracle
from paper_2608_04085_amd import inputs
from paper_2608_04085_amd.config import CKPT_REVOLVE, CKPT_UNIFORM, RECON_BALANCED, RTConfig, paper_preset

pytestmark = pytest.mark.gpu

# one strip with its halos wrapping onto itself, a full strip of the adjoint
# (58 columns) and of the step (60), one column more, two strips and a bit;
# segments of one row (small batches), of several rows (64 members), and whole
# columns (1100 members)
CASES = [
    RTConfig(nx=3, ny=2),
    RTConfig(nx=58, ny=3, batch=2),
    RTConfig(nx=59, ny=5),
    RTConfig(nx=60, ny=61),
    RTConfig(nx=61, ny=40, batch=3),
    RTConfig(nx=130, ny=37, batch=64),
    RTConfig(nx=5, ny=9, batch=1100),
    paper_preset(62, batch=40).with_(recon=RECON_BALANCED),
    # a row that is one wavefront
    RTConfig(nx=64, ny=2),
    RTConfig(nx=64, ny=37, batch=70),
    paper_preset(64, batch=3).with_(recon=RECON_BALANCED),
]
IDS = [f"{c.nx}x{c.ny}x{c.batch}-{c.recon}" for c in CASES]


def host(t):
    return t.detach().cpu().numpy()


def contexts(cfg, max_steps=256):
    from paper_2608_04085_amd import rtcnop
    cols = rtcnop.Context(cfg, max_steps=max_steps)
    cols.set_columns(rtcnop.COLUMNS_STEP | rtcnop.COLUMNS_ADJOINT)
    tiles = rtcnop.Context(cfg, max_steps=max_steps, tile="16x15")
    cols.set_fold(False)
    assert tiles.columns == 0 and cols.kernels == "columns/columns"
    return cols, tiles


def states(cfg):
    rng = np.random.default_rng(cfg.nx * 1000 + cfg.ny)
    amp = 3e-2 if cfg.lx == 0.5 else 1e-1
    uv = amp * rng.standard_normal((cfg.batch, 2, cfg.ny, cfg.nx))
    return inputs.mask_components(uv, cfg.comp_mask)


@pytest.mark.parametrize("cfg", CASES, ids=IDS)
def test_step_by_columns_has_the_bits_of_the_tiles_and_matches_the_oracle(cfg):
    cols, tiles = contexts(cfg)
    U = tiles.init_state(states(cfg))
    for _ in range(2):
        U = tiles.step(U)
    dt = tiles.cfl_dt(U)
    Uc, nc = cols.step(U, dt, want_next=True)
    Ut, nt = tiles.step(U, dt, want_next=True)
    np.testing.assert_array_equal(host(Uc), host(Ut))
    np.testing.assert_array_equal(host(nc), host(nt))
    np.testing.assert_array_equal(host(cols.step(U, dt)), host(Ut))
    cols.check_error()
    members = sorted({0, cfg.batch - 1})
    o = Oracle.from_config(cfg.with_(batch=len(members)))
    want = o.step(np.ascontiguousarray(host(U)[members]), np.ascontiguousarray(host(dt)[members]))
    for k in range(4):
        assert np.max(np.abs(host(Uc)[members][:, k] - want[:, k])) <= 1e-13 * np.max(np.abs(want[:, k]))


@pytest.mark.parametrize("cfg", CASES, ids=IDS)
@pytest.mark.parametrize("kernel", ["columns", "fused"])
def test_one_launch_adjoint_has_the_bits_of_the_tiles_and_matches_the_oracle(cfg, kernel):
    from paper_2608_04085_amd import rtcnop
    cols, tiles = contexts(cfg)
    if kernel == "fused":
        cols.set_columns(rtcnop.FUSED_ADJOINT)
    assert cols.kernels.endswith(kernel)
    U = tiles.init_state(states(cfg))
    for _ in range(2):
        U = tiles.step(U)
    dt = tiles.cfl_dt(U)
    lam = torch.from_numpy(np.random.default_rng(7).standard_normal(U.shape)).cuda()
    got = cols.step_adjoint(U, dt, lam)
    np.testing.assert_array_equal(host(got), host(tiles.step_adjoint(U, dt, lam)))
    cols.check_error()
    members = sorted({0, cfg.batch - 1})
    o = Oracle.from_config(cfg.with_(batch=len(members)))
    want = o.step_vjp(*(np.ascontiguousarray(host(x)[members]) for x in (U, dt, lam)))
    for k in range(4):
        assert np.max(np.abs(host(got)[members][:, k] - want[:, k])) <= 1e-12 * np.max(np.abs(want[:, k]))


@pytest.mark.parametrize("cfg", [CASES[1], CASES[5], CASES[7]], ids=[IDS[1], IDS[5], IDS[7]])
def test_march_and_gradient_by_columns_have_the_bits_of_the_tiles(cfg):
    # members of different step counts, the step log, and snapshots written
    # by the step kernel
    from paper_2608_04085_amd import rtcnop
    uv = states(cfg) * np.linspace(0.1, 1.0, cfg.batch)[:, None, None, None]
    cols, tiles = contexts(cfg, max_steps=512)
    T = 20.3 * float(host(tiles.cfl_dt(tiles.init_state(uv))).min())
    a = cols.integrate(cols.init_state(uv), T, log_cap=512)
    b = tiles.integrate(tiles.init_state(uv), T, log_cap=512)
    n = host(a[2])
    np.testing.assert_array_equal(n, host(b[2]))
    np.testing.assert_array_equal(host(a[0]), host(b[0]))
    for m in range(cfg.batch):
        np.testing.assert_array_equal(host(a[3])[m, : n[m]], host(b[3])[m, : n[m]])
    pol = rtcnop.Policy(CKPT_UNIFORM, 4)
    Ra, ga, _ = cols.grad_u0(uv, T, pol)
    Rb, gb, _ = tiles.grad_u0(uv, T, pol)
    np.testing.assert_array_equal(host(Ra), host(Rb))
    np.testing.assert_array_equal(host(ga), host(gb))


def test_unphysical_state_is_reported_by_the_column_kernels():
    from paper_2608_04085_amd import rtcnop
    cfg = RTConfig(nx=70, ny=20)
    cols, _ = contexts(cfg)
    lam = torch.ones(1, 4, cfg.ny, cfg.nx, dtype=torch.float64)
    for var, value in ((3, -1.0), (0, -0.5), (0, float("nan")), (2, float("inf"))):
        U = cols.init_state(states(cfg))
        U[0, var, 13, 61] = value
        for call in (lambda: cols.step(U, torch.tensor([1e-4])), lambda: cols.step_adjoint(U, torch.tensor([1e-4]), lam)):
            call()
            with pytest.raises(rtcnop.RTError) as e:
                cols.check_error()
            assert e.value.code == -4
            cols.check_error()  # the flag is cleared


# a grid, ragged in both directions, for each tile shape of the fused adjoint
# beyond the smallest (which the cases above run on): 16x8, 16x16, 24x16 and
# 32x16 tiles in one round of blocks, and 32x16 in two
FUSED = [(126, 255, 1, 0), (250, 255, 1, 1), (310, 250, 1, 0), (255, 510, 1, 1), (255, 510, 2, 0)]


@pytest.mark.parametrize("nx,ny,batch,recon", FUSED)
def test_fused_adjoint_shapes_have_the_bits_of_the_tiles(nx, ny, batch, recon):
    from paper_2608_04085_amd import rtcnop
    cfg = RTConfig(nx=nx, ny=ny, batch=batch, recon=recon)
    tiles = rtcnop.Context(cfg, max_steps=64, tile="16x15")
    fused = rtcnop.Context(cfg, max_steps=64)
    fused.set_columns(rtcnop.FUSED_ADJOINT)
    U = tiles.step(tiles.init_state(states(cfg)))
    dt = tiles.cfl_dt(U)
    lam = torch.from_numpy(np.random.default_rng(8).standard_normal(U.shape)).cuda()
    np.testing.assert_array_equal(host(fused.step_adjoint(U, dt, lam)), host(tiles.step_adjoint(U, dt, lam)))
    fused.check_error()


@pytest.mark.parametrize("cfg", [CASES[0], CASES[4], CASES[7], RTConfig(nx=126, ny=255)],
                         ids=[IDS[0], IDS[4], IDS[7], "126x255"])
def test_differentiated_steps_by_the_fused_adjoint_match_the_tiles(cfg):
    # the sum behind the step sizes' derivative is grouped by tile: equal to
    # its rounding, about 1e-16 times the square root of its 1e2 to 1e5 terms,
    # which 20 steps and the correction's cancellation leave far below 1e-11
    from paper_2608_04085_amd import rtcnop
    uv = states(cfg) * np.linspace(0.1, 1.0, cfg.batch)[:, None, None, None]
    out = []
    for mask in (0, rtcnop.FUSED_ADJOINT):
        r = rtcnop.Context(cfg, max_steps=256, tile="16x15")
        r.set_columns(mask)
        r.set_dt_mode("differentiated")
        T = 12.4 * float(host(r.cfl_dt(r.init_state(uv))).min())
        out.append([host(x) for x in r.grad_u0(uv, T, rtcnop.Policy(CKPT_UNIFORM, 4))])
    np.testing.assert_array_equal(out[1][0], out[0][0])
    np.testing.assert_array_equal(out[1][2], out[0][2])
    assert np.max(np.abs(out[1][1] - out[0][1])) <= 1e-11 * np.max(np.abs(out[0][1]))


def test_default_kernels_by_grid_size():
    from paper_2608_04085_amd import rtcnop
    for cfg, want in ((RTConfig(nx=64, ny=128), "8x8w/fused"), (RTConfig(nx=256, ny=512), "32x16/fused"),
                      (RTConfig(nx=512, ny=512), "columns/fused"),
                      (RTConfig(nx=512, ny=1024, batch=8), "columns/columns")):
        r = rtcnop.Context(cfg, max_steps=8)
        assert r.kernels == want, (cfg, r.kernels)
        r.set_tiles("16x16", "32x8")
        assert r.kernels == "16x16/32x8" and r.columns == 0
        r.set_columns(rtcnop.COLUMNS_ADJOINT | rtcnop.FUSED_ADJOINT)
        assert r.kernels == "16x16/columns"
        r.set_fold(True)
        assert r.kernels == "16x16/32x8" and r.fold
    with pytest.raises(rtcnop.RTError):
        r.set_columns(8)


@pytest.mark.parametrize("cfg", [RTConfig(nx=61, ny=40, batch=3), RTConfig(nx=250, ny=255)], ids=["61x40x3", "250x255"])
def test_cfl_step_after_each_step_starts_from_cleared_slots(cfg):
    # rt_step's dt_next comes from slots that the kernel that read them clears:
    # calls in a row, after states of larger and of smaller signal speed, and
    # through both step kernels
    from paper_2608_04085_amd import rtcnop
    r = rtcnop.Context(cfg, max_steps=8)
    fast, slow = r.init_state(30.0 * states(cfg)), r.init_state(states(cfg))
    dt = 0.5 * r.cfl_dt(fast)
    for mask in (rtcnop.FUSED_ADJOINT, rtcnop.COLUMNS_STEP):
        r.set_columns(mask)
        for U in (slow, fast, slow, slow):
            Un, nxt = r.step(U, dt, want_next=True)
            np.testing.assert_array_equal(host(nxt), host(r.cfl_dt(Un)))


@pytest.mark.parametrize("nx,ny,nb", [(61, 40, 2), (130, 37, 3), (70, 21, 5), (300, 100, 70)])
def test_groups_of_columns_side_by_side_have_the_bits_of_one_stream(nx, ny, nb):
    # the binomial sweep in column kernels: two even groups, three members in
    # one stream, uneven groups, launches of more than one wavefront per SIMD
    from paper_2608_04085_amd import rtcnop
    cfg = RTConfig(nx=nx, ny=ny, batch=nb)
    uv = states(cfg) * np.linspace(0.1, 1.0, nb)[:, None, None, None]
    r = rtcnop.Context(cfg, max_steps=64)
    r.set_columns(rtcnop.COLUMNS_STEP | rtcnop.COLUMNS_ADJOINT)
    T = 12.4 * float(host(r.cfl_dt(r.init_state(uv))).min())
    want = [host(x) for x in r.grad_u0(uv, T, rtcnop.Policy(CKPT_UNIFORM, 1))]
    for on in (False, True, True):
        r.set_overlap(on)
        got = [host(x) for x in r.grad_u0(uv, T, rtcnop.Policy(CKPT_REVOLVE, pool_bytes=5 * 32 * nx * ny * nb))]
        for a, b in zip(got, want):
            np.testing.assert_array_equal(a, b)
    r.check_error()


@pytest.mark.parametrize("cfg", [RTConfig(nx=3, ny=2, batch=2), RTConfig(nx=9, ny=7), RTConfig(nx=61, ny=40, batch=3),
                                 RTConfig(nx=250, ny=254), paper_preset(62, batch=3).with_(recon=RECON_BALANCED),
                                 RTConfig(nx=520, ny=1100)],
                         ids=["3x2x2", "9x7", "61x40x3", "250x254", "62x62x3-balanced", "520x1100"])
def test_step_size_correction_by_the_next_launch_matches_the_tiles(cfg):
    # Members end at different steps; the cell of largest speed lies anywhere,
    # also in the halo of tiles that wrap onto themselves; 520x1100 has more
    # tiles than a launch corrects from.  The sum behind mu is grouped by tile:
    # 1e-11 as above; the policies agree to the bit.
    from paper_2608_04085_amd import rtcnop
    uv = states(cfg) * np.linspace(0.1, 1.0, cfg.batch)[:, None, None, None]
    out = []
    for mask in (0, rtcnop.FUSED_ADJOINT):
        r = rtcnop.Context(cfg, max_steps=64, tile="16x15")
        r.set_columns(mask)
        r.set_dt_mode("differentiated")
        T = (12.4 if cfg.cells < 100000 else 3.4) * float(host(r.cfl_dt(r.init_state(uv))).min())
        for pol in (rtcnop.Policy(CKPT_UNIFORM, 1), rtcnop.Policy(CKPT_UNIFORM, 3),
                    rtcnop.Policy(CKPT_REVOLVE, pool_bytes=3 * 32 * cfg.cells * cfg.batch)):
            out.append([host(x) for x in r.grad_u0(uv, T, pol)])
        r.check_error()
    for o in out[1:3]:
        np.testing.assert_array_equal(o[1], out[0][1])
    for o in out[4:]:
        np.testing.assert_array_equal(o[1], out[3][1])
    np.testing.assert_array_equal(out[3][2], out[0][2])
    assert np.max(np.abs(out[3][1] - out[0][1])) <= 1e-11 * np.max(np.abs(out[0][1]))
