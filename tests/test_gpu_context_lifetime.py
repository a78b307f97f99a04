"""GPU: creating and destroying contexts does not wait for other streams'
work, and contexts that come and go (also in several threads) march as one
that stays."""
import gc
import threading

import numpy as np
import pytest
import torch

from paper_2608_04085_amd import inputs
from paper_2608_04085_amd.config import RTConfig

pytestmark = pytest.mark.gpu


def host(t):
    return t.detach().cpu().numpy()


@pytest.mark.parametrize("marched", [False, True])
def test_destroying_a_context_does_not_wait_for_another_stream(marched):
    from paper_2608_04085_amd import rtcnop
    a = torch.randn(4096, 4096, dtype=torch.float64, device="cuda")
    o = torch.empty_like(a)
    torch.mm(a, a, out=o)
    side, done = torch.cuda.Stream(), torch.cuda.Event()
    cfg = RTConfig(nx=40, ny=72)
    r = rtcnop.Context(cfg, max_steps=256)
    if marched:
        r.integrate(r.init_state(inputs.seed_batch(cfg, [0], rms=1e-3)), 0.05)
    gc.collect()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        for _ in range(100):  # a few ms each at the least
            torch.mm(a, a, out=o)
        done.record()
    del r
    waited = done.query()
    torch.cuda.synchronize()
    assert not waited


def test_contexts_that_come_and_go_in_threads_march_alike():
    # step counts, speeds and flags come through host memory that a destroyed
    # context leaves to the next: batches of one and of several pages
    from paper_2608_04085_amd import rtcnop
    cfgs = [RTConfig(nx=16, ny=24, batch=b) for b in (1, 3, 400)]
    uvs = [3e-2 * np.random.default_rng(c.batch).standard_normal((c.batch, 2, c.ny, c.nx)) for c in cfgs]

    def march(k):
        r = rtcnop.Context(cfgs[k], max_steps=256)
        U, t, n, _ = r.integrate(r.init_state(uvs[k]), 0.08)
        return host(U), host(n)

    want = [march(k) for k in range(3)]
    assert all(int(n.min()) > 5 for _, n in want)
    bad = []

    def work(first):
        with torch.cuda.stream(torch.cuda.Stream()):
            for i in range(9):
                k = (first + i) % 3
                U, n = march(k)
                if not (np.array_equal(U, want[k][0]) and np.array_equal(n, want[k][1])):
                    bad.append((first, i))

    threads = [threading.Thread(target=work, args=(f,)) for f in range(3)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad
