"""A cell re-emits what it absorbed.  Its spectrum is L t_i / S with S the sum
of the same terms t_i: the sum of n terms, the quotient L / S and the product
with each term round by at most (n - 1) + 1 + 1 units of 2^-53, so the
spectrum's exact sum lies within (n + 2) 2^-53 of L, however unlike the terms
are (a faint Wien term beside a Rayleigh-Jeans one makes the sum's curvature in
T hundreds of times its slope squared)."""
import math

import numpy as np
import pytest


def _case(orc, n_lambda, seed):
    """Wavelengths spread at random over 0.1 - 1000 um, and cells of 3 - 3000 K."""
    rng = np.random.default_rng(1000 * n_lambda + seed)
    lam = np.sort(10.0 ** rng.uniform(-1.0, 3.0, n_lambda))
    dlam, ka = 0.1 * lam, lam ** -1.5
    L = np.array([orc.mbb_sum(lam, dlam, ka, t) for t in 10.0 ** rng.uniform(math.log10(3.0), math.log10(3000.0), 300)])
    L = L[(L > 1e-200) & (L < 1e200)]
    return (0.0, float(L.size), 0.0, 1.0, 0.0, 1.0), L, lam, dlam, ka


def _off(em, L):
    """Largest deviation of a cell's exact sum from L, in 2^-53 of L."""
    return max(abs(math.fsum(em[:, m]) - L[m]) / L[m] for m in range(L.size)) * 2.0 ** 53


@pytest.mark.parametrize("n_lambda", [1, 2, 3, 4, 8, 60])
def test_cells_reemit_what_they_absorbed_on_the_harness(E, orc, n_lambda):
    for seed in range(8):
        box, L, lam, dlam, ka = _case(orc, n_lambda, seed)
        _, em = E.dust_emission(box, (L.size, 1, 1), np.ones(L.size), 0, L[None, :], lam, dlam, ka, 1.0)
        assert _off(em, L) <= n_lambda + 2, seed


@pytest.mark.gpu
@pytest.mark.parametrize("n_lambda", [1, 2, 3, 4, 8, 60])
def test_cells_reemit_what_they_absorbed_on_the_gpu(orc, n_lambda):
    import torch
    from paper_1410_1629_amd import binding as B
    dev = lambda a: torch.as_tensor(a, dtype=torch.float64, device="cuda")
    for seed in range(8):
        box, L, lam, dlam, ka = _case(orc, n_lambda, seed)
        em = torch.empty((n_lambda, L.size), dtype=torch.float64, device="cuda")
        B.dust_emission({"box": box, "n": (L.size, 1, 1)}, dev(np.ones(L.size)), 0, dev(L[None, :]), lam, dlam, ka, 1.0,
                        em, None)
        assert _off(em.cpu().numpy(), L) <= n_lambda + 2, seed
