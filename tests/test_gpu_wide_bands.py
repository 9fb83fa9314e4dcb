"""Bands in which every 32-bit offset is an ordinary pixel: the regularizers' 64-bit
addresses at the index 0x0c000000, which the buffer path keeps for "no pixel". The
reference and its tolerance are those of test_gpu_regularizer_sweep.py; every
element of u, s, t, y1, y3, y4 is compared after five iterations (an odd count: the
states are those of the side that the initial point does not write)."""
import pytest

from gpu_helpers import announce
from test_gpu_regularizer_sweep import check

pytestmark = pytest.mark.gpu


def test_the_buffer_paths_missing_pixel_is_a_pixel_here():
    announce("a band of 12289 x 16384 pixels: pixel (12288, 0) has the index 0x0c000000")
    assert 12288 * 16384 == 0x0C000000
    check(3, (1, 12289, 16384), scale=0.02)
