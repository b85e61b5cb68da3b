"""Where the kernels that decode the packed weight themselves read its index stream: never past a row's words, whatever spans and
chunks the reduction ends on.  The library's own address arithmetic, on the host."""
import ctypes

import pytest

import paper_2409_09708_amd as nm
from paper_2409_09708_amd.binding import load_library


@pytest.mark.parametrize("N,M", [(1, 4), (3, 4), (1, 8), (2, 8), (3, 8), (4, 8), (1, 16), (2, 16), (4, 16)])
@pytest.mark.parametrize("wide", [False, True])
def test_index_words_end_with_the_row(N, M, wide):
    words = load_library().nm_internal_direct_index_words
    words.restype, words.argtypes = ctypes.c_int64, [ctypes.c_int32] * 3 + [ctypes.c_int64]
    whole = 8 if wide else 16  # the last chunk of the wide form may be half of one
    for K in [k for k in range(64, 1100, whole) if k % M == 0]:
        assert words(wide, N, M, K) == nm.nm_index_bytes(1, K, N, M) // 4, K
