"""GPU tests of the coarsest inverse on the builder's operators of long meshes:
more panels than a wave keeps in registers, and rows that wait for their pivot
over many of them (their factors reach panels far back).  Reference: LAPACK's
solution refined in extended precision.  Errors are taken in the unknowns of
the equilibrated operator (powers of two); the bound is 1e2 eps times its
condition number."""

import numpy as np
import pytest
import scipy.sparse as sp

from test_gpu_coarse import OneLevel, _say

pytestmark = pytest.mark.gpu


def equilibrated(A):
    """Exponents of rows and columns after four passes over the largest entries."""
    C = A.tocoo()
    n, e = A.shape[0], np.frexp(np.abs(C.data))[1]
    r, c = np.zeros(n, int), np.zeros(n, int)
    for _ in range(4):
        for own, at in ((r, C.row), (c, C.col)):
            top = np.full(n, -10 ** 6)
            np.maximum.at(top, at[C.data != 0], (e + r[C.row] + c[C.col])[C.data != 0])
            own -= np.where(top > -10 ** 6, top >> 1, 0)
    return 2.0 ** r, 2.0 ** c


# 1,674 to 3,426 free dofs (105 to 215 panels)
@pytest.mark.parametrize("dim,mesh,transient", [(2, (24, 6), False), (2, (24, 6), True), (2, (16, 6), False),
                                                (2, (24, 8), True),
                                                (3, (16, 2, 2), True)])
def test_long_coarsest_operator_against_lapack(dim, mesh, transient):
    import torch

    from paper_1709_05660_amd import MG, Problem
    from synth import ProblemSpec, fourier_coefficients
    s = ProblemSpec(dim=dim, nx=2 * mesh[0], ny=2 * mesh[1], nz=2 * mesh[2] if dim == 3 else 1, levels=2, patch=2,
                    lx=(0.25 if dim == 2 else 0.5) * mesh[0], transient=transient, seed=3)
    p = Problem(s, fourier_coefficients(dim, 3))
    rp, ci, v, shape = p.csr(0)
    A = sp.csr_matrix((v, ci, rp), shape=shape)
    r, c = equilibrated(A)
    E = (sp.diags(r) @ A @ sp.diags(c)).toarray()
    rng = np.random.default_rng(4)
    B = rng.standard_normal((3, A.shape[0])) / r
    mg = MG(OneLevel(A.copy()), precision="fp64")
    X = [mg.apply(0, 5, torch.as_tensor(b).cuda()).cpu().numpy() for b in B]
    mg.refactor()
    again = mg.apply(0, 5, torch.as_tensor(B[0]).cuda()).cpu().numpy()
    mg.close()
    inv = np.linalg.inv(E)
    tol = 1e2 * 2.0 ** -52 * np.linalg.norm(E, 2) * np.linalg.norm(inv, 2)
    for b, x in zip(B, X):
        y = inv @ (r * b)
        for _ in range(4):
            y = y + inv @ np.asarray(r * b - E.astype(np.longdouble) @ y.astype(np.longdouble), float)
        err = np.linalg.norm(x / c - y) / np.linalg.norm(y)
        _say("long coarse", mesh, "time step" if transient else "steady", A.shape[0], "rel err", err, "tol", tol,
             "lapack inverse", np.linalg.norm(inv @ (r * b) - y) / np.linalg.norm(y))
        assert err <= tol
    assert np.array_equal(again, X[0])
