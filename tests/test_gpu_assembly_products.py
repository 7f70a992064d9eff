"""GPU test of the element Jacobian's products away from the seeded state for
the element kind that the assembly's own off-state test leaves out (3D,
steady): the checker's assembly is the reference."""

import pytest

import test_gpu_assembly as base

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,kw", base.CASES[2:3])
def test_steady_3d_products_off_state(name, kw):
    base.test_device_assembly_off_state_against_checker(name, kw)
