"""Dust emission where its terms leave the middle of their range: wavelengths
far into the Wien and Rayleigh-Jeans ends, opacities near the smallest and
largest doubles (scaled by a power of two, the emissivity by its inverse:
nothing else changes), a table whose first entries underflow, one wavelength; on
the CPU harness and on the GPU against the oracle.  T carries a few units of
2^-53 (1e-12 as for the other spectra); a wavelength with b/T = u carries u
times T's error, 2e-12 for u <= 700."""
import numpy as np
import pytest

CASES = {"wide": (np.geomspace(1e-2, 1e6, 40), 0), "one": (np.array([3.0]), 0),
         "far_wien": (np.geomspace(0.01, 0.3, 7), 0), "faint": (np.geomspace(1.0, 1000.0, 20), -700),
         "strong": (np.geomspace(1.0, 1000.0, 20), 690)}


def _case(orc, name):
    """Arguments of the call, and the oracle's temperatures and spectra."""
    lam, shift = CASES[name]
    dlam, ka = 0.1 * lam, lam ** -1.3
    temps = np.array([1.0005, 1.7, 2.5, 9.0, 20.0, 77.7, 300.0, 4321.0, 6e4, 9.99e4])
    L = np.array([orc.mbb_sum(lam, dlam, ka, t) for t in temps])
    L = L[(L > 1e-60) & (L < 1e60)]
    box, n = (0.0, float(L.size), 0.0, 1.0, 0.0, 1.0), (L.size, 1, 1)
    out = orc.dust_emission(box, n, np.ones(L.size), L[None, :], lam, dlam, ka, 1.0)
    return (box, n, np.ones(L.size), L, lam, dlam, np.ldexp(ka, shift), np.ldexp(1.0, -shift)), out


def _compare(name, T, em, T_o, em_o):
    np.testing.assert_allclose(T, T_o, rtol=1e-12)
    # a term is formed with the opacity it is given, before the emissivity
    # scales it back: with 2^-700 in the opacity it is a normal number only
    # where the spectrum is 2^700 above the smallest ones
    floor = np.ldexp(1e-290, max(0, -CASES[name][1]))
    big = em_o > floor
    np.testing.assert_allclose(em[big], em_o[big], rtol=2e-12)
    assert np.all(em[~big] <= 2.0 * floor)


@pytest.mark.parametrize("name", sorted(CASES))
def test_wide_spectra_on_the_harness(E, orc, name):
    (box, n, rho, L, lam, dlam, ka, eps), out = _case(orc, name)
    _compare(name, *E.dust_emission(box, n, rho, 0, L[None, :], lam, dlam, ka, eps), *out)


@pytest.mark.gpu
@pytest.mark.parametrize("name", sorted(CASES))
def test_wide_spectra_on_the_gpu(orc, name):
    import torch
    from paper_1410_1629_amd import binding as B
    (box, n, rho, L, lam, dlam, ka, eps), out = _case(orc, name)
    dev = lambda a: torch.as_tensor(a, dtype=torch.float64, device="cuda")
    em = torch.empty((lam.size, L.size), dtype=torch.float64, device="cuda")
    T = torch.empty(L.size, dtype=torch.float64, device="cuda")
    B.dust_emission({"box": box, "n": n}, dev(rho), 0, dev(L[None, :]), lam, dlam, ka, eps, em, T)
    _compare(name, T.cpu().numpy(), em.cpu().numpy(), *out)
