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


# sizes on either side of each line between the 128 x 128 and the 256 x 256 weight-gradient tiles: at most three tiles of 256 x 256 and a share
# of 180 K tiles x tiles per compute unit; four tiles and 100; more and 20; little padding; 112 rows per expert
@pytest.mark.parametrize("A,d,f,E,small", [
    (491520, 192, 768, 12, True), (491520 + 5 * 32, 192, 768, 12, False), (204800, 256, 1024, 8, True), (204832, 256, 1024, 8, False),
    (400000, 512, 512, 8, False), (20480, 512, 1024, 8, True), (20512, 512, 1024, 8, False), (1 << 20, 384, 1536, 8, True),
    (1 << 20, 128, 8192, 8, True), (112 * 64, 2048, 8192, 64, True), (112 * 64 + 1, 2048, 8192, 64, False)])
def test_line_of_the_weight_gradient_tiles(A, d, f, E, small):
    assert paths(A, d, f, E, E)["small_gradients"] == small


def test_weight_gradients_of_layers_wider_than_byte_offsets():
    """32 rows of 2^26 columns and more: the 128 x 128 tiles count 32-bit offsets in bytes, the 256 x 256 ones in elements."""
    for d, f in ((8, 2 ** 26), (8, 70_000_000), (2 ** 26 + 8, 8)):
        assert not paths(32, d, f, 1, 1)["small_gradients"]
    assert paths(32, 8, 2 ** 26 - 8, 1, 1)["small_gradients"]
