"""GPU test of the choice between the blocks' two inversions in a plain setup:
Gauss-Jordan for a few blocks beside a coarsest Gauss-Jordan chain, the LU
elsewhere.  A Schwarz application has the bits of the forced inversion."""

import numpy as np
import pytest

from gpu_common import dev, host

pytestmark = pytest.mark.gpu

PAIRED, LU = 6, 7


@pytest.mark.parametrize("nx,ny,levels,patch,variant", [
    (16, 16, 2, 4, PAIRED),    # coarsest mesh 8x8 (407 waiting rows): the chain; 16 blocks of up to 372 dofs
    (64, 64, 4, 4, PAIRED),    # the same with 336
    (32, 8, 2, 4, LU),         # 16x4: banded
    (64, 64, 4, 2, LU)])       # 8x8, six rounds of blocks of 112 dofs
def test_inversion_of_a_plain_setup(nx, ny, levels, patch, variant, tmp_path):
    from paper_1709_05660_amd import MG, Problem
    from synth import ProblemSpec, fourier_coefficients
    s = ProblemSpec(dim=2, nx=nx, ny=ny, levels=levels, patch=patch, lx=0.25 * (nx >> (levels - 1)),
                    transient=True, seed=5)
    p = Problem(s, fourier_coefficients(2, 5))
    r = dev(np.random.default_rng(6).standard_normal(p.n))
    db = str(tmp_path / "tune.db")
    mg = MG(p, precision="fp64")
    z = {None: host(mg.apply(levels - 1, 4, r))}
    mg.autotune(db)
    mg.close()
    lines = [line.split() for line in open(db).read().split("\n") if line]
    for v in (PAIRED, LU):
        with open(db, "w") as f:
            for k, x in lines:
                if k.startswith("gj3:"):
                    x = v
                elif k.startswith("gjg:"):
                    k = k.rsplit(":", 1)[0] + f":{v}"
                f.write(f"{k} {x}\n")
        mg = MG(p, precision="fp64")
        assert mg.autotune(db) == 0
        mg.refactor()
        z[v] = host(mg.apply(levels - 1, 4, r))
        mg.close()
    assert not np.array_equal(z[PAIRED], z[LU])
    assert np.array_equal(z[None], z[variant])
