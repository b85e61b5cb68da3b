"""Which dX multiplies a transposed copy of the weight: the choice knows the output type and many tokens.  The library's own rule, on
the host, at shapes where both forms were timed far apart."""
import ctypes

import pytest

from paper_2409_09708_amd.binding import load_library

ONE, COPY = 0, 1


# (T, O, K): tokens, reduction, width; float32, bfloat16
@pytest.mark.parametrize("T,O,K,f32,bf16", [
    (1576, 768, 2048, ONE, ONE), (7205, 576, 1600, ONE, ONE), (13056, 1792, 640, ONE, ONE), (11876, 3456, 544, ONE, ONE),
    (1656, 640, 2216, ONE, ONE), (197, 3072, 768, COPY, COPY), (1576, 4096, 1024, COPY, COPY), (197, 768, 768, COPY, COPY),
    (65, 2304, 768, COPY, COPY), (1576, 768, 768, COPY, COPY), (3152, 512, 512, COPY, COPY), (8, 1024, 1024, COPY, COPY)])
def test_the_faster_form_is_chosen(T, O, K, f32, bf16):
    lib, i64 = load_library(), ctypes.c_int64
    assert lib.nm_backward_input_workspace_bytes(O, K, T) == 0 < lib.nm_backward_input_scratch_bytes(O, K, T)
    copies = [lib.nm_internal_backward_input_copies(i64(O), i64(K), i64(T), b) for b in (0, 1)]
    assert copies == [f32, bf16]
