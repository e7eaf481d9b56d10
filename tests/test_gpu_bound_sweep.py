"""trial_bound never exceeds a trial's exact distance: at every float that a
uniform of the generator rounds to (2^-53 to 1, 4.4e8 of them), for the largest
uniform that rounds to it, with coefficients over the range that dipole ends
have, among them those that single precision rounds up (or whose reciprocal it
does) by the most."""
import ctypes
import os

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

LIB = os.path.join(os.path.dirname(os.path.abspath(__file__)), "native", "libtrial_bounds.so")


@pytest.mark.parametrize("inverse", [0, 1])
def test_bound_is_never_above_the_distance(inverse):
    import torch  # noqa: F401  (its HIP runtime serves the process)

    lib = ctypes.CDLL(LIB)
    up = 1.0 + 2.0 ** -24 + 2.0 ** -50    # rounds up to 1 + 2^-23
    down = 1.0 + 2.0 ** -24 - 2.0 ** -50  # rounds down to 1: its reciprocal comes out large
    coefs = [s * m for s in (2.0 ** -20, 2.0 ** -6, 1.0, 2.0 ** 9, 2.0 ** 40) for m in (up, down, 1.3, 1.9999999)]
    arr = (ctypes.c_double * len(coefs))(*coefs)
    above, worst = ctypes.c_uint64(), ctypes.c_float()
    print(f"case bound sweep inverse={inverse}", flush=True)
    assert lib.trial_bound_sweep(arr, len(coefs), inverse, ctypes.byref(above), ctypes.byref(worst)) == 0
    assert above.value == 0
    assert worst.value > 1.0 - 2.0 ** -16  # and is close to it: few cycles need the exact comparison
