"""The polynomials of the largest eigenvalue's closed form, as the device code
evaluates them (constants read from its header, each step rounded as an FMA)."""
import os
import re

import numpy as np

from paper_2408_02758_amd import build as B

L = np.longdouble


def test_float64_polynomial_is_as_exact_as_the_library():
    """c = cos(acos(r) / 3) over r in [-1, 1]: the polynomial's rms error is below that
    of correctly rounded acos and cos one after the other, and it has no bias.

    Bounds: acos rounds by up to 2^-52 (rms 2^-53 / sqrt(3) of values above 1,
    times c' = sin(acos / 3) / 3 <= 0.29) and cos by 2^-54: together 4.4e-17; a
    bias of 1e-17 is a sixth of a rounding."""
    text = open(os.path.join(B.CSRC, "ftle_device_math.h")).read()
    k = [float(v) for v in re.search(r"kEigPoly\[20\] = \{([^}]*)\}", text).group(1).split(",")]
    centre = float(re.search(r"kEigCentre = ([^;]*);", text).group(1))
    r = np.random.default_rng(0).uniform(-1, 1, 200000)
    u = np.sqrt(0.5 * (1.0 + r)) - centre
    c = np.full_like(u, k[-1])
    for a in k[-2::-1]:
        c = (c.astype(L) * u + a).astype(np.float64)
    err = (c - np.cos(np.arccos(r.astype(L)) / 3)).astype(np.float64)
    print(f"rms {np.sqrt(np.mean(err ** 2)):.2e}, bias {err.mean():.1e}")
    assert np.sqrt(np.mean(err ** 2)) <= 4.4e-17
    assert abs(err.mean()) <= 1e-17
