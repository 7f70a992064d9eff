"""GPU test of the server's admission estimate: without the share it keeps for
the pool's rounding, it covers the bytes that the setup and solve of a system
take from the pool (one request, a fresh pool)."""

import time

import numpy as np
import pytest

from test_gpu_block_lu import TwoLevel

pytestmark = pytest.mark.gpu


def _request(name):
    if name == "builder":
        from paper_1709_05660_amd import Problem
        from synth import config, fourier_coefficients
        s = config("c0_2d_16x4")
        return Problem(s, fourier_coefficients(s.dim, s.seed))
    p = TwoLevel({"small": [17] * 300, "smallest": [2] * 600, "ragged": [33, 81, 145] * 12, "large": [800, 513]}[name], 9)
    p.b = np.random.default_rng(1).standard_normal(p.n)
    return p


@pytest.mark.parametrize("precision", ["fp64", "bf16"])
@pytest.mark.parametrize("name", ["builder", "small", "smallest", "ragged", "large"])
def test_estimate_covers_the_pool(name, precision):
    from paper_1709_05660_amd import Server
    p = _request(name)
    srv = Server(hbm_budget_bytes=4 << 30, max_slots=1)
    ticket = srv.submit(p, precision=precision, rtol=1e-6, restart=5, maxit=5)
    end = time.time() + 60
    while srv.poll(ticket)[0] == 2 and time.time() < end:
        time.sleep(0.001)
    stats = srv.stats()
    srv.close()
    taken = stats["pool_peak_in_use_bytes"]
    # the estimate is 5/4 of its sum and 96 pages; each of the pool's about 100 arrays is rounded up to 256 bytes
    bare = (stats["peak_bytes"] - 96 * 4096) / 1.25
    print(name, precision, "taken", taken, "estimate", bare, flush=True)
    assert taken - 100 * 256 <= bare
