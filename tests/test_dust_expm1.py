"""The dust emission's e^u - 1 against 80-bit arithmetic (2^-64 units, rounded
once here): within the 1.6 units of 2^-53 of it that its comment states, over
its whole range, around the places where the multiple of ln 2 changes, and to
the smallest arguments."""
import numpy as np
import pytest

LN2 = np.log(np.longdouble(2))


def _arguments(name):
    rng = np.random.default_rng(3)
    if name == "range":
        return rng.uniform(0.0, 700.0, 400000)
    if name == "small":
        return 10.0 ** rng.uniform(-30.0, 1.0, 400000)
    k = rng.integers(0, 1009, 200000)
    near = (LN2 * (k + 0.5 * rng.integers(0, 2, k.size))).astype(np.float64)  # multiples and halves
    return np.abs(near * (1.0 + rng.integers(-40, 41, k.size) * 2.0 ** -52))


@pytest.mark.skipif(np.finfo(np.longdouble).nmant < 63, reason="needs 80-bit long doubles")
@pytest.mark.parametrize("name", ["range", "small", "multiples"])
def test_expm1(E, name):
    u = _arguments(name)
    u = u[(u > 0.0) & (u < 700.0)]
    ref = np.expm1(u.astype(np.longdouble))
    off = np.abs(E.expm1(u).astype(np.longdouble) - ref) / ref * np.longdouble(2) ** 53
    assert float(off.max()) <= 1.6, (float(off.max()), float(u[off.argmax()]))
