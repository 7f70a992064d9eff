"""GPU test of the dynamic LDS limits of the blocks' inversion kernels: a limit
belongs to the kernel, which handles of several sizes and setup threads share,
so setting a smaller system up must not lower it under a launch of a larger
one."""

import ctypes as C

import pytest

from test_gpu_block_lu import TwoLevel

pytestmark = pytest.mark.gpu


class FuncAttributes(C.Structure):
    _fields_ = [("binary_version", C.c_int), ("cache_mode_ca", C.c_int), ("const_size", C.c_size_t),
                ("local_size", C.c_size_t), ("max_dynamic_shared", C.c_int), ("max_threads", C.c_int),
                ("num_regs", C.c_int), ("carveout", C.c_int), ("ptx_version", C.c_int), ("shared_size", C.c_size_t)]


def dynamic_limit(lib, kernel):
    hip = C.CDLL("libamdhip64.so")
    a = FuncAttributes()
    assert hip.hipFuncGetAttributes(C.byref(a), C.c_void_p(C.addressof(C.c_char.in_dll(lib, kernel)))) == 0
    return a.max_dynamic_shared


# (precision, mangled type and arguments, smallest and largest block of the class, bytes a row)
@pytest.mark.parametrize("precision,inst,small,large,row", [
    ("fp64", "IdLi6ELi2E", 257, 384, 2 * 18 * 8), ("fp64", "IdLi8ELi2E", 385, 512, 2 * 18 * 8),
    ("fp64", "IdLi13ELi1E", 513, 800, 18 * 8), ("fp32", "IfLi13ELi2E", 513, 800, 2 * 20 * 4)])
def test_limit_admits_the_largest_of_the_class(precision, inst, small, large, row):
    from paper_1709_05660_amd import MG, lib
    name = f"_ZN3fsi11k_lu_blocks{inst}EEvPT_PKlPKiS4_PiS7_S6_"
    handles = [MG(TwoLevel([m], 5), precision=precision) for m in (large, small)]
    limit = dynamic_limit(lib(), name)
    print(precision, inst, "limit", limit, "a row", row, flush=True)
    assert limit >= row * large
    for mg in handles:
        mg.refactor()
        mg.close()
