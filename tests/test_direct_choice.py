"""Which form of the kernel that decodes the packed weight itself a plain call takes, at shapes where the two were timed far apart."""
import pytest

from gpu_util import product_route


# one round of blocks of one span of 256: the first form (two spans of the other took 1.1 to 1.25 of its time); more blocks, one span
# of the other, or a chunk that is half past K: the second
@pytest.mark.parametrize("T,K,O,N,M,wide", [
    (507, 208, 893, 4, 16, False), (1155, 208, 370, 4, 16, False), (143, 256, 2632, 3, 8, False), (669, 256, 568, 3, 8, False),
    (600, 256, 1100, 3, 8, True), (1664, 256, 768, 4, 8, True), (1025, 64, 1096, 4, 8, True), (1579, 1000, 1001, 2, 8, True)])
def test_forms(T, K, O, N, M, wide):
    kernel, tile = product_route("plain", T, K, O, N, M)
    assert kernel == "direct" and (tile[:2] == (64, 128)) == wide
