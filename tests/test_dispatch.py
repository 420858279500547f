"""Which bf16 kernels a call takes, and the size of their launches: host arithmetic of the library, no GPU."""
import ctypes

import pytest

FIELDS = ("few_rows", "small_gradients", "joint", "merged", "seg_tiles", "bins2", "bins1", "threads")


def paths(A, d, f, E, V):
    """The kernels of a bf16 call with A rows (flexmoe_debug_bf16_paths)."""
    from paper_2304_03946_amd import binding
    fn = binding.load_library().flexmoe_debug_bf16_paths
    fn.restype, fn.argtypes = None, [ctypes.c_int] * 5 + [ctypes.c_void_p]
    out = (ctypes.c_longlong * len(FIELDS))()
    fn(A, d, f, E, V, out)
    return dict(zip(FIELDS, out))


@pytest.mark.parametrize("d", [8, 16, 24, 32])
@pytest.mark.parametrize("E", [4, 16, 256])
@pytest.mark.parametrize("columns", [2 ** 29, 2 ** 30 - 2048, 2 ** 30, 2 ** 30 + 2 ** 29, 2 ** 31 - 2 ** 19])
def test_weight_gradients_of_very_many_columns_can_be_launched(d, E, columns):
    """All experts' columns: a product of its own is two threads each, both in one launch are four.  HIP runs a grid of 2^32 threads
    and more modulo 2^32, without an error."""
    f = columns // E // 8 * 8
    for A in (1, 64, 4096):
        p = paths(A, d, f, E, E)
        assert p["threads"] < 2 ** 32, p
    assert paths(64, d, 512, E, E)["joint"]
