"""Symmetries of the library's taps that the direct correlation folds its sum by.

For integer offsets A(-q, z) = A(q, z), and A(q, -z) is the conjugate of
A(-q, z): h_z[-d] = h_z[d] for |d| < L/2 and h_-z = conj(h_z).  The library
integrates both signs and both sides separately by FP64 quadrature, so the
identities hold to its accuracy (1e-12, five orders below one FP32 rounding).
"""

import numpy as np
import pytest

from paper_1806_01556_amd import fdas


@pytest.mark.parametrize("z", [0, 1, 7, 8, 21, 42, 63, 64])
def test_taps_symmetric_in_distance_and_conjugate_in_drift(z):
    h, g = fdas.template_taps(z), fdas.template_taps(-z)
    assert np.max(np.abs(g - np.conj(h))) < 1e-12
    assert np.max(np.abs(h[1:] - h[1:][::-1])) < 1e-12  # h[0] is the tap at d = -L/2
