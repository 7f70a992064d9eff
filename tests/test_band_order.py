"""CPU tests of the ordering of the coarsest operator for its banded elimination
(compiled from its source): positions, the panels' rows and columns, and the
recognition of patterns with too few rows for a panel's columns, which the
elimination must not be given (a panel without a waiting row)."""

import os
import subprocess

import numpy as np
import pytest
import scipy.sparse as sp

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1709_05660_amd", "csrc")

MAIN = """
#include <cstdio>
#include "fsi_order.h"
template <class V> static void line(const V &v) {
  for (auto x : v) printf("%d ", (int)x);
  printf("\\n");
}
int main() {
  int n, nnz;
  if (scanf("%d %d", &n, &nnz) != 2) return 1;
  std::vector<int64_t> rp(n + 1);
  std::vector<int> ci(nnz);
  for (auto &v : rp) { int x; if (scanf("%d", &x) != 1) return 1; v = x; }
  for (auto &v : ci) if (scanf("%d", &v) != 1) return 1;
  const fsi::BandOrder b = fsi::band_order(n, rp, ci, 16);
  printf("%d %d %.17g %.17g\\n", b.window, (int)b.full, fsi::band_time(b, n), fsi::chain_time(n));
  line(b.colpos); line(b.rowpos); line(b.hi); line(b.cend);
}
"""


@pytest.fixture(scope="module")
def order(tmp_path_factory):
    d = tmp_path_factory.mktemp("order")
    src, exe = str(d / "main.cpp"), str(d / "main")
    open(src, "w").write(MAIN)
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", CSRC, src, os.path.join(CSRC, "fsi_order.cpp"), "-o", exe],
                   check=True)

    def run(A):
        A = sp.csr_matrix(A)
        A.sort_indices()
        text = " ".join(map(str, [A.shape[0], A.nnz, *A.indptr, *A.indices]))
        out = subprocess.run([exe], input=text, check=True, capture_output=True, text=True).stdout.splitlines()
        window, full, *run.times = map(float, out[0].split())
        return (int(window), bool(full), *(np.array(x.split(), int) for x in out[1:]))

    return run


def starved(rows, wide, narrow):
    """`rows` rows alone reach the first `wide` > rows columns; the others share the last `narrow`."""
    n = wide + narrow
    A = np.zeros((n, n))
    for i in range(n):
        if i < rows:
            A[i, :wide] = A[i, wide + i % narrow] = 1
        else:
            A[i, wide + (i + np.arange(-4, 5)) % narrow] = 1
    return A


# (27, 64, 64): 48 rows for the first 64 columns, so no row is left before the fourth panel
@pytest.mark.parametrize("shape", [(27, 64, 64), (32, 64, 64)])
def test_too_few_rows_for_the_columns_are_recognised(order, shape):
    A = starved(*shape)
    assert np.linalg.matrix_rank(A * np.random.default_rng(0).uniform(1, 2, A.shape)) < len(A)
    window, full, colpos, rowpos, hi, cend = order(A)
    short = hi < np.minimum(16 * (np.arange(len(hi)) + 1), len(A))
    print(shape, "window", window, "hi", hi, "short at", np.nonzero(short)[0])
    assert short.any() and not full


@pytest.mark.parametrize("n,half", [(1, 1), (16, 3), (17, 5), (130, 20), (401, 33)])
def test_orders_of_banded_patterns(order, n, half):
    rng = np.random.default_rng(n)
    i, j = np.indices((n, n))
    A = (np.abs(i - j) <= half) & ((rng.uniform(size=(n, n)) < 0.4) | (i == j))
    p = rng.permutation(n)
    A = A[p][:, p].astype(float)
    window, full, colpos, rowpos, hi, cend = order(A)
    assert full and sorted(colpos) == list(range(n)) and sorted(rowpos) == list(range(n))
    B = np.zeros((n, n))
    B[np.ix_(rowpos, colpos)] = A
    for k in range(len(hi)):
        lo, up = 16 * k, min(16 * (k + 1), n)
        assert not B[hi[k]:, :up].any() and not B[:hi[k], cend[k]:].any()
        assert lo < hi[k] <= lo + window


# measured on the device (us): the banded elimination and the Gauss-Jordan chain
@pytest.mark.parametrize("mesh,transient,band,chain", [
    ((16, 4), False, 980, 2600), ((24, 6), False, 3622, 11029), ((24, 8), True, 7130, 21144),
    ((8, 8), False, 2944, 2732), ((8, 6), True, 1335, 1780), ((8, 2, 2), False, 1427, 2149),
    ((8, 2, 4), False, 11953, 9082), ((10, 4, 2), True, 15867, 13527), (120, None, 190, 237), (384, None, 941, 681)])
def test_the_faster_inverse_is_chosen(order, mesh, transient, band, chain):
    """The builder's coarsest operators of these meshes (their free block), and dense ones."""
    if transient is None:
        A = np.ones((mesh, mesh))
    else:
        from paper_1709_05660_amd import Problem
        from synth import ProblemSpec, fourier_coefficients
        dim = len(mesh)
        s = ProblemSpec(dim=dim, nx=2 * mesh[0], ny=2 * mesh[1], nz=2 * mesh[2] if dim == 3 else 1, levels=2, patch=2,
                        lx=(0.25 if dim == 2 else 0.5) * mesh[0], transient=transient, seed=3)
        rp, ci, v, shape = Problem(s, fourier_coefficients(dim, 3)).csr(0)
        P = sp.csr_matrix((np.ones(len(ci)), ci, rp), shape=shape)
        free = ~((np.diff(P.indptr) == 1) & (np.diff(P.tocsc().indptr) == 1))
        A = P[free][:, free]
    window = order(A)[0]
    est_band, est_chain = order.times
    print(mesh, "window", window, "estimates", est_band, est_chain, "measured", band, chain)
    assert (est_band > est_chain) == (band > chain)
    assert abs(est_band / band - 1) < 0.15 and abs(est_chain / chain - 1) < 0.15
