"""Arrays read from the library's pinned memory: views, copies by one thread and copies by several, on both sides of the
size where the copy changes."""
import ctypes as C

import numpy as np
import pytest

from paper_2502_09138_amd.tracker import _THREADED_COPY_BYTES, _host_array

LIMIT = _THREADED_COPY_BYTES // 4


@pytest.mark.parametrize("dtype", [np.uint32, np.int32, np.float32])
@pytest.mark.parametrize("count", [0, 1, 77, LIMIT - 1, LIMIT, LIMIT + 3])
def test_views_and_copies(dtype, count):
    bits = np.random.default_rng(count).integers(0, 1 << 32, max(count, 1), dtype=np.uint64).astype(np.uint32)
    source = bits.view(dtype)
    pointer = source.ctypes.data_as(C.POINTER(C.c_uint32))
    own = _host_array(pointer, count, dtype, True)
    view = _host_array(pointer, count, dtype, False)
    for a in (own, view):
        assert a.shape == (count,) and a.dtype == dtype and a.flags.writeable and a.flags.c_contiguous
        np.testing.assert_array_equal(a.view(np.uint32), bits[:count])   # NaN patterns included
    assert own.flags.owndata and not np.shares_memory(own, source)
    assert count == 0 or np.shares_memory(view, source)
