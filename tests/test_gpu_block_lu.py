"""GPU tests of the Schwarz blocks' inversion at the edges of its size classes
(16-column panels, rows a lane, panels a wave, the largest block), through the C ABI: a two-level hierarchy whose patches are runs
of consecutive dofs of a seeded saddle-point matrix, one Schwarz application
against numpy's block solves.  The bound is 1e2 eps cond(B), with eps of the
working matrices, over the largest block's cond, plus the storage rounding of
the 16-bit forms."""

import ctypes as C
import sys

import numpy as np
import pytest
import scipy.sparse as sp

pytestmark = pytest.mark.gpu


def _say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def _csr(dst, A, keep):
    A = sp.csr_matrix(A)
    A.sort_indices()
    rp = np.ascontiguousarray(A.indptr, dtype=np.int64)
    ci = np.ascontiguousarray(A.indices, dtype=np.int32)
    v = np.ascontiguousarray(A.data, dtype=np.float64)
    keep += [rp, ci, v]
    dst.nrows, dst.ncols = A.shape
    dst.nnz = A.nnz
    dst.rowptr = rp.ctypes.data_as(C.POINTER(C.c_int64))
    dst.colind = ci.ctypes.data_as(C.POINTER(C.c_int32))
    dst.val = v.ctypes.data_as(C.POINTER(C.c_double))


class TwoLevel:
    """Level 1: patches of the given sizes, each overlapping the one before by
    a third of the smaller (the earlier one owns the overlap); level 0: a
    diagonal operator of four dofs."""

    def __init__(self, sizes, seed):
        from paper_1709_05660_amd import _lib as L
        rng = np.random.default_rng(seed)
        ranges, a = [], 0
        for i, m in enumerate(sizes):
            if i:
                a = ranges[-1][1] - min(m, sizes[i - 1]) // 3
            ranges.append((a, a + m))
        n = ranges[-1][1]
        # zero diagonals on every fifth dof (row pivoting), rows of very different scales
        i = np.arange(n)
        A = sp.diags(np.where(i % 5 == 4, 0.0, 6.0 + rng.uniform(size=n))).tolil()
        for d in (1, 2, 3, 7, 13):
            for r in range(n - d):
                if not (r % 5 == 4 and (r + d) % 5 == 4) and rng.uniform() < 0.7:
                    A[r, r + d] = rng.uniform(-1.0, 1.0)
                    A[r + d, r] = rng.uniform(-1.0, 1.0)
        for r in range(4, n, 5):     # the zero-diagonal dofs couple firmly to the one before
            A[r, r - 1] = A[r - 1, r] = 2.0
        self.A = sp.csr_matrix(sp.diags(10.0 ** rng.integers(-4, 5, n)) @ A.tocsr())
        self.ranges = ranges
        self.n, self.nlevels, self.keep = n, 2, []
        self.levels = (L.LevelC * 2)()
        _csr(self.levels[0].J, sp.identity(4), self.keep)
        _csr(self.levels[1].J, self.A, self.keep)
        P = sp.csr_matrix((np.ones(4), (np.arange(4) * (n // 4), np.arange(4))), shape=(n, 4))
        _csr(self.levels[1].P, P, self.keep)
        _csr(self.levels[1].R, P.T, self.keep)
        ptr = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
        dof = np.concatenate([np.arange(a, b) for a, b in ranges]).astype(np.int32)
        owned, end = [], 0
        for a, b in ranges:
            owned.append((np.arange(a, b) >= end).astype(np.uint8))
            end = max(end, b)
        owned = np.concatenate(owned)
        kind = np.zeros(len(sizes), np.uint8)
        self.keep += [ptr, dof, owned, kind]
        p = self.levels[1].patches
        p.npatch = len(sizes)
        p.ptr = ptr.ctypes.data_as(C.POINTER(C.c_int64))
        p.dof = dof.ctypes.data_as(C.POINTER(C.c_int32))
        p.owned = owned.ctypes.data_as(C.POINTER(C.c_uint8))
        p.kind = kind.ctypes.data_as(C.POINTER(C.c_uint8))

    def schwarz(self, r):
        """The restricted Schwarz application and the largest row-scaled cond."""
        y, end, cond = np.zeros(self.n), 0, 1.0
        for a, b in self.ranges:
            B = self.A[a:b, a:b].toarray()
            s = 1.0 / np.abs(B).max(1)
            B = B * s[:, None]
            x = np.linalg.solve(B, r[a:b] * s)
            y[max(a, end):b] = x[max(a, end) - a:]
            cond = max(cond, np.linalg.cond(B))
            end = max(end, b)
        return y, cond


SIZES = {
    "panels": [1, 2, 15, 16, 17, 31, 33, 63, 64, 65],
    "128": [127, 128, 17, 100],
    "256": [129, 255, 256],
    "384": [257, 383, 384, 372, 90],
    "385": [385, 40],
    "512": [320, 511, 512],
    "800": [513, 799, 800, 16],
}


@pytest.mark.parametrize("name,precision", [(k, "fp64") for k in SIZES] + [(k, "fp32") for k in SIZES] +
                         [("384", "bf16"), ("384", "fp16"), ("800", "bf16")])
def test_blocks_inverted_at_size_edges(name, precision):
    import torch

    from paper_1709_05660_amd import MG
    p = TwoLevel(SIZES[name], 7 + len(name))
    mg = MG(p, precision=precision)
    rng = np.random.default_rng(3)
    scale = np.abs(p.A).max(1).toarray().ravel()
    r = rng.standard_normal(p.n) * scale
    op = 4 if precision == "fp64" else 6
    y = mg.apply(1, op, torch.as_tensor(r, device="cuda")).cpu().numpy()
    mg.refactor()
    again = mg.apply(1, op, torch.as_tensor(r, device="cuda")).cpu().numpy()
    mg.close()
    ref, cond = p.schwarz(r)
    eps = 2.0 ** -52 if precision == "fp64" else 2.0 ** -23
    tol = 1e2 * eps * cond
    if precision in ("bf16", "fp16"):
        # rows of m entries rounded to 8 or 11 bits of the row's largest scaled one: random errors
        tol += 4 * (2.0 ** -8 if precision == "bf16" else 2.0 ** -11) * cond ** 0.5
    err = np.linalg.norm(y - ref) / np.linalg.norm(ref)
    _say("blocks", name, precision, "rel err", err, "tol", tol, "cond", cond)
    assert err <= tol
    assert np.array_equal(y, again)
