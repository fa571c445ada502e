"""The rules that choose a call's kernels, queried on the host (no GPU): each
choice is a launch the runtime accepts and the kernel's on-chip memory holds."""
import ctypes as C

import pytest

import paper_2609_35800_amd as hg

THREADS, BLOCK_TOKENS = 256, 128  # a workgroup of the quantize kernels


def select_with_values(slices, n, D, bits):
    f = hg.library().hg_test_select_with_values
    f.argtypes, f.restype = [C.c_uint64, C.c_uint64, C.c_int, C.c_int], C.c_int
    return bool(f(slices, n, D, bits))


@pytest.mark.parametrize("n", [1, 128, 129, 1000])
@pytest.mark.parametrize("D", [64, 128, 256])
def test_selection_with_the_values_stays_under_the_launch_limit(n, D):
    """The launch of the values with the selection has one workgroup a slice more
    than the values alone; a launch of 2^32 work-items or more is refused."""
    per_slice = -(-n // BLOCK_TOKENS) + 1
    most = (2**32 - 1) // THREADS // per_slice
    assert select_with_values(most, n, D, 2) and not select_with_values(most + 1, n, D, 2)
    assert not select_with_values(2**23, n, D, 2) or 2**23 * per_slice * THREADS < 2**32
