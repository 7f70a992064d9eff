"""GPU tests of how exact the Schwarz blocks' inverses are: blocks whose rows
differ so much that pivots chosen by unscaled magnitudes lose digits, and the
16-bit rows against the rounding of each entry."""

import numpy as np
import pytest
import scipy.linalg as sl

from gpu_common import csr_of, dev, host
from test_gpu_block_lu import SIZES, TwoLevel, _say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("transient", [True, False])
def test_interface_blocks_keep_the_digits_of_row_scaled_pivots(transient):
    """Blocks with the equations of both materials: LAPACK's inverse of the
    block with its rows scaled is at least 25 times closer to the refined
    solution than that of the plain block, and the library's within ten times
    the former."""
    from paper_1709_05660_amd import MG, Problem
    from synth import ProblemSpec, fourier_coefficients
    p = Problem(ProblemSpec(dim=2, nx=32, ny=8, levels=2, patch=4, transient=transient, lx=4.0, seed=5),
                fourier_coefficients(2, 5))
    J = csr_of(p, 1).tocsr()
    scale = 0.5 ** np.frexp(abs(J).max(1).toarray().ravel())[1]
    r = np.random.default_rng(0).standard_normal(p.n) / scale
    mg = MG(p, precision="fp64")
    z = host(mg.apply(1, 4, dev(r)))
    mg.close()
    ptr, dof, own, _ = p.patches(1)
    found = 0
    for k in range(len(ptr) - 1):
        d, o = dof[ptr[k]:ptr[k + 1]], own[ptr[k]:ptr[k + 1]].astype(bool)
        B, b = J[d][:, d].toarray(), r[d]
        S, c = B * scale[d][:, None], b * scale[d]
        lu = sl.lu_factor(S)
        x = sl.lu_solve(lu, c)
        for _ in range(4):
            x = x.astype(np.longdouble)
            x = x + sl.lu_solve(lu, np.asarray(c - S.astype(np.longdouble) @ x, float))
        x = np.asarray(x, float)[o]
        err = lambda y: np.linalg.norm(y - x) / np.linalg.norm(x)
        plain, scaled, here = err((np.linalg.inv(B) @ b)[o]), err((np.linalg.inv(S) @ c)[o]), err(z[d[o]])
        if plain < 25 * scaled:
            continue
        found += 1
        _say("interface block", k, len(d), "plain", plain, "scaled", scaled, "here", here)
        assert here <= 10 * scaled
    assert found >= 1


@pytest.mark.parametrize("name", ["panels", "128", "256", "384", "512", "800"])
@pytest.mark.parametrize("precision", ["bf16", "fp16"])
def test_rows_in_16_bits_against_their_rounding(name, precision):
    """|error| <= u |B^-1| |r| in the norm, u half a unit in the last of 8 or 11
    bits, with FP16's smallest step under the columns' scales, and 1e2 eps cond
    of the FP32 inverse."""
    from paper_1709_05660_amd import MG
    p = TwoLevel(SIZES[name], 7 + len(name))
    r = np.random.default_rng(3).standard_normal(p.n) * abs(p.A).max(1).toarray().ravel()
    mg = MG(p, precision=precision)
    y = host(mg.apply(1, 6, dev(r)))
    mg.close()
    ref, cond = p.schwarz(r)
    bound, end = np.zeros(p.n), 0
    for a, b in p.ranges:
        W = np.abs(np.linalg.inv(p.A[a:b, a:b].toarray()))[max(a, end) - a:]
        bound[max(a, end):b] = (2.0 ** -9 if precision == "bf16" else 2.0 ** -12) * (W @ np.abs(r[a:b]))
        if precision == "fp16":
            bound[max(a, end):b] += 2.0 ** -25 * (W.max(0) @ np.abs(r[a:b]))
        end = max(end, b)
    tol = (np.linalg.norm(bound) / np.linalg.norm(ref)) + 1e2 * 2.0 ** -23 * cond
    err = np.linalg.norm(y - ref) / np.linalg.norm(ref)
    _say("16-bit rows", name, precision, "rel err", err, "tol", tol, "of it rounding", tol - 1e2 * 2.0 ** -23 * cond)
    assert err <= tol
