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
