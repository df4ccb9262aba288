"""Calls that a line of the dispatch once sent to the slower of two kernels (the measured times stand at launch_forward), and
the claims that tests on the GPU make about the kernels their calls are sent to."""
import pytest

from tests import dispatch


@pytest.mark.parametrize("b, n, hq, hkv, d, seqlens, shares", [
    (2, 1900, 14, 2, 128, True, 2), (2, 1900, 14, 2, 64, True, 2), (2, 1600, 16, 8, 64, True, 2), (4, 1700, 8, 8, 128, True, 2),
    (4, 1700, 8, 2, 128, True, 1), (2, 1400, 20, 4, 128, True, 1),                                  # one KV head to an XCD
    (1, 1900, 28, 4, 64, False, 2), (1, 1900, 28, 4, 128, False, 1), (1, 1700, 32, 8, 64, False, 1),
])
def test_split_where_nearly_every_place_is_taken(b, n, hq, hkv, d, seqlens, shares):
    assert dispatch.forward(b, n, hq, hkv, d, 128, seqlens=seqlens).shares == shares
