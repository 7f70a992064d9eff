"""GPU tests of coarsest operators that have no inverse: each is reported, by
the step of the coarsest level, and a later operator of the same pattern that
has one is inverted."""

import numpy as np
import pytest

from test_band_order import starved
from test_gpu_coarse import OneLevel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(27, 64, 64), (32, 64, 64)])
def test_pattern_without_rows_for_its_columns_is_reported(shape):
    import scipy.sparse as sp

    from paper_1709_05660_amd import MG, FsiError
    A = starved(*shape) * np.random.default_rng(1).uniform(1, 2, (sum(shape[1:]),) * 2)
    with pytest.raises(FsiError) as e:
        MG(OneLevel(sp.csr_matrix(A)), precision="fp64")
    assert "coarsest" in str(e.value)


def block_triangular(nblock, lower):
    """Dense 16 x 16 blocks on the diagonal (one panel of the elimination each), and full ones beside them on one
    side: the rows of a block are pivots before those of the next begin."""
    A = np.kron(np.eye(nblock), np.ones((16, 16))) + np.kron(np.eye(nblock, k=-1 if lower else 1), np.ones((16, 16)))
    return A * np.random.default_rng(nblock).uniform(1, 2, A.shape) + 30 * np.eye(16 * nblock)


@pytest.mark.parametrize("lower", [False, True])
@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.inf])
def test_entry_that_is_not_finite_is_reported(lower, bad):
    import scipy.sparse as sp
    import torch

    from paper_1709_05660_amd import MG, FsiError
    A = sp.csr_matrix(block_triangular(4, lower))
    for at in (0, 16 * 16 + 3, 5 * 16 * 16 + 7, A.nnz - 1):
        p = OneLevel(A.copy())
        p.val[at] = bad
        with pytest.raises(FsiError) as e:
            MG(p, precision="fp64")
        assert "coarsest" in str(e.value)
    mg = MG(OneLevel(A), precision="fp64")
    val = A.data.copy()
    val[16 * 16 + 3] = bad
    mg.set_jvalues(0, torch.as_tensor(val).cuda())
    with pytest.raises(FsiError):
        mg.refactor()
    mg.set_jvalues(0, torch.as_tensor(A.data).cuda())
    mg.refactor()
    b = np.random.default_rng(2).standard_normal(A.shape[0])
    x = mg.apply(0, 5, torch.as_tensor(b).cuda()).cpu().numpy()
    mg.close()
    ref = np.linalg.solve(A.toarray(), b)
    assert np.linalg.norm(x - ref) <= 1e2 * 2.0 ** -52 * np.linalg.cond(A.toarray()) * np.linalg.norm(ref)
