"""Kept device memory goes back without being asked for: after calls that do not
use it, and at the end of any call, small ones too, that finds less than half
of the device's memory free."""
import pytest

pytestmark = pytest.mark.gpu
LARGE = 1 << 29  # the run's peel-ray queue alone takes 1.7 GB
KEEP_CALLS = 32


def _free():
    import torch
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def _large_run(B, W):
    """A run that leaves more than LARGE bytes behind; returns the free memory before it."""
    import torch
    p = W.spiral(n_packages=1_000_000)
    rho = B.density_tensor(p)
    images = torch.empty(B.image_shape(p), dtype=torch.float64, device="cuda")
    B.release_workspaces()
    before = _free()
    B.run_photons(dict(p, flags=3), rho, images)
    assert _free() < before - LARGE
    return before


def _small_call(B, W):
    """A call of a few rays and about a kilobyte of device memory."""
    import torch
    p = W.small_problem("few", (4, 4, 4), rho=W.lognormal_density((4, 4, 4), 1.0, seed=1))
    rho = B.density_tensor(p)
    o, k = (torch.as_tensor(a, device="cuda") for a in W.random_rays(100, p["box"], seed=9))
    tau = torch.empty(100, dtype=torch.float64, device="cuda")
    return lambda: B.trace_path(p, rho, 1.0, 0, o, k, tau, crossings=False)


def test_memory_goes_when_calls_do_not_use_it():
    from paper_1410_1629_amd import binding as B
    from paper_1410_1629_amd import workloads as W
    call = _small_call(B, W)
    before = _large_run(B, W)
    for _ in range(KEEP_CALLS):
        call()
    assert _free() < before - LARGE
    call()
    assert _free() > before - LARGE // 2
    B.release_workspaces()


def test_memory_goes_when_the_device_fills():
    import torch
    from paper_1410_1629_amd import binding as B
    from paper_1410_1629_amd import workloads as W
    call = _small_call(B, W)
    before = _large_run(B, W)
    call()
    assert _free() < before - LARGE
    held = torch.empty(_free() - torch.cuda.mem_get_info()[1] // 2 + (8 << 30), dtype=torch.uint8, device="cuda")
    call()
    now = _free()
    del held
    torch.cuda.empty_cache()
    assert now > torch.cuda.mem_get_info()[1] // 2 - (8 << 30) + LARGE
    assert _free() > before - LARGE // 2
