"""GPU: the spectra of lines that are split in two stages, and of prime and
longer ones that are not."""
import numpy as np
import pytest
import torch

from paper_2608_04085_amd.config import RTConfig

pytestmark = pytest.mark.gpu


def host(t):
    return t.detach().cpu().numpy()


@pytest.mark.parametrize("nx,ny,nb", [(4, 4, 1), (6, 251, 2), (127, 64, 3), (254, 9, 1), (1022, 49, 1), (2048, 6, 2),
                                      (2049, 4, 1), (2054, 3, 1), (12, 2048, 1), (8, 2050, 1)])
def test_spectra_of_split_prime_and_long_lines(nx, ny, nb):
    cfg = RTConfig(nx=nx, ny=ny, batch=nb)
    from paper_2608_04085_amd import rtcnop
    r = rtcnop.Context(cfg, max_steps=8)
    f = np.random.default_rng(nx * ny).standard_normal((nb, 2, ny, nx))
    d = torch.from_numpy(f).cuda()
    # a coefficient is a sum of n terms with an error below n halves of an ulp
    # of the sum of magnitudes, sqrt(n) of the largest mode: n^1.5 1.2e-16 in
    # the worst case and far less as errors cancel; 1e-12 for each n here
    for row in (0, ny - 1):
        E = np.abs(np.fft.rfft(f[:, 1, row], axis=-1)) ** 2
        got = host(r.row_spectrum(d, row, component=1))
        assert np.all(np.abs(got - E) <= 1e-12 * E.max(axis=-1, keepdims=True)), row
    E = np.abs(np.fft.rfft2(f[:, 0])) ** 2
    got = host(r.power_spectrum_2d(d, component=0)).reshape(E.shape)
    assert np.all(np.abs(got - E) <= 1e-12 * E.max(axis=(1, 2), keepdims=True))
