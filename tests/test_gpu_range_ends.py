"""Kernels at ends of their ranges that the tests of the ranges leave out: the
last interval of the Rys tables (T below 60) and its asymptotic form, and guess
gradients with more than eight chunks (over 256 row blocks of 32)."""
from __future__ import annotations

import pytest

import test_gpu_boys
import test_gpu_guess_net

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [59.0, 59.5, 59.99, 59.999999, 60.0, 60.000001, 61.0])
def test_last_interval_of_the_quadrature(T):
    test_gpu_boys.test_argument_of_every_class(T)


@pytest.mark.parametrize("counts", [(900, 3700, 3800), (0, 8193, 0)])
def test_more_than_eight_chunks(counts):
    assert sum(-(-c // 32) for c in counts) > 256
    test_gpu_guess_net.test_row_blocks_and_chunks(counts)
