"""Several arrays in one allocation: no exception and no allocation on the host (the calls that use it are C entries),
every array on its own 256 bytes, a size beyond the address space and more arrays than it holds reported by status."""
import ctypes

import pytest

import _host


@pytest.fixture(scope="module")
def slab(tmp_path_factory):
    lib = _host.load("host_alloc", tmp_path_factory.mktemp("host"))

    def call(counts):
        n = len(counts)
        arr = (ctypes.c_size_t * max(n, 1))(*counts)
        at = (ctypes.c_size_t * max(n, 1))()
        size = ctypes.c_size_t()
        st = lib.slab(ctypes.c_int(n), arr, ctypes.byref(size), at)
        return st, size.value, list(at)[:n]
    return call


@pytest.mark.parametrize("n", [1, 7, 28])
def test_no_heap_and_no_overlap(slab, n):
    counts = [(37 * i) % 90 for i in range(n)]   # an empty array among them
    st, size, at = slab(counts)
    assert st == 0
    ends = [a + 8 * max(c, 1) for a, c in zip(at, counts)]
    assert all(a % 256 == 0 for a in at) and ends[-1] <= size
    assert all(e <= a for e, a in zip(ends, at[1:]))


def test_too_much_is_a_status(slab):
    assert slab([1, (1 << 61) + 5])[0] > 0        # 2^64 bytes and more
    assert slab([1 << 60, 1 << 60, 1 << 60])[0] > 0
    assert slab([1] * 64)[0] > 0
