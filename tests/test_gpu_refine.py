"""The second sort of the queued peel rays where one tile holds one long run of
equal keys (a point source's emission rays), around the sort's turns of 8192
rays and its wavefronts of 64: every ray is walked once.  The same call
without a queue walks each ray where it arises.  FP64 walks agree to rounding
and sums of n contributions of one sign differ by at most n 2^-53 (2e-12 for
2e4): 1e-11; one ray lost or walked twice is 1/n, at least 4e-5."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("flags", [1, 3])
@pytest.mark.parametrize("n_pkg", [1, 2, 63, 64, 65, 1025, 8191, 8192, 8193, 24577])
def test_long_runs_walk_every_ray_once(n_pkg, flags):
    import torch
    from paper_1410_1629_amd import binding as B
    from paper_1410_1629_amd import workloads as W
    p = W.small_problem("refine", (8, 8, 8), (-1, 1, -1, 1, -1, 1), kappa=1.0, albedo=0.6, g=0.3, n_packages=n_pkg,
                        precision=0, flags=flags, seed=9, detectors=[W.frame(10.0, 40.0, 24, 20, 1.2, 1.1)])
    rho = B.density_tensor(p)
    queued, inline = (torch.empty(B.image_shape(p), dtype=torch.float64, device="cuda") for _ in range(2))
    a = B.run_photons(p, rho, queued)
    b = B.run_photons(p, rho, inline, peel_queue=-1)
    assert a["peels"] == b["peels"] and a["x_peel"] == b["x_peel"]
    assert float((queued - inline).abs().sum()) <= 1e-11 * float(inline.abs().sum())
    assert float(inline.sum()) > 0.0
