"""CPU: the magnitude up to which the fp32 path takes pixels apart into bf16 parts."""

import ctypes

import numpy as np
import pytest

F = np.float32


def limit(w, b):
    from paper_2009_04509_amd import binding
    f = binding.lib._ZN7pointid18conv_fc1_f32_limitEPKfS1_
    f.restype = ctypes.c_float
    p = ctypes.POINTER(ctypes.c_float)
    w, b = np.ascontiguousarray(w, F), np.ascontiguousarray(b, F)
    return f(w.ctypes.data_as(p), b.ctypes.data_as(p))


@pytest.mark.parametrize("scale", [1e-30, 0.01, 1.0, 1e4, 1e37])
def test_conv_sums_stay_in_range(scale):
    """Pixels below the limit: the conv's largest sum, its parts' 1.02 times that and
    the bias stay below a quarter of fp32's range, and no pixel rounds to infinity in bf16."""
    rng = np.random.default_rng(1)
    w, b = rng.normal(0, scale, (48, 25)).astype(F), rng.normal(0, scale, 48).astype(F)
    x = float(limit(w, b))
    assert 0 < x <= 2.0**126
    top = (x * 1.02 * np.abs(w.astype(np.float64)).sum(1) + 1.02 * np.abs(b)).max()
    assert top <= 2.0**126 * (1 + 1e-6)
    if scale >= 1:
        assert top >= 2.0**125                           # and the limit is no lower than it has to be


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan, 3.4e38])
def test_no_pixel_where_weights_leave_no_room(value):
    w, b = np.ones((48, 25), F), np.zeros(48, F)
    b[7] = value
    assert limit(w, b) == 0
    w[9, 3], b[7] = value, 0
    assert limit(w, b) == 0 or value == 3.4e38
