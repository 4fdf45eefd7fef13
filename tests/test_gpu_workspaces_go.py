"""Kept device memory goes back without being asked for: after calls that do not
use it, and at the end of any call, small ones too, that finds less than half
of the device's memory free."""
import hiprt
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


def test_a_recorded_run_plans_without_the_kept_memory():
    """A run that is recorded into a graph cannot take kept blocks or give them back: its chunks are those that the
    memory beside them allows.  (Nothing of the graphs is run.)"""
    import ctypes as C
    import torch
    from paper_1410_1629_amd import binding as B
    from paper_1410_1629_amd import workloads as W
    hip = hiprt.load()
    stream = torch.cuda.Stream()
    p = W.cube(n_packages=30_000_000, precision=1)
    p["flags"] = 3
    rho = B.density_tensor(p)
    images = torch.empty(B.image_shape(p), dtype=torch.float64, device="cuda")

    def nodes():
        graph, n = C.c_void_p(), C.c_size_t(0)
        assert hip.hipStreamBeginCapture(C.c_void_p(stream.cuda_stream), 0) == 0
        try:
            B.run_photons(p, rho, images, stats=False, stream=stream)
        finally:
            ended = hip.hipStreamEndCapture(C.c_void_p(stream.cuda_stream), C.byref(graph))
        assert ended == 0 and hip.hipGraphGetNodes(graph, None, C.byref(n)) == 0
        assert hip.hipGraphDestroy(graph) == 0
        return n.value

    nodes()  # what a first recording sets up
    B.run_photons(dict(p, n_packages=1000), rho, images, stats=False, peel_queue=(24 << 30) // 74)
    free = _free()
    held = torch.empty(free - (24 << 30), dtype=torch.uint8, device="cuda")  # 24 GiB free, about as much kept
    beside = nodes()
    B.release_workspaces()
    more = torch.empty(_free() - (24 << 30), dtype=torch.uint8, device="cuda")
    assert more.numel() > 20 << 30
    alone = nodes()
    del held, more
    torch.cuda.empty_cache()
    assert beside == alone
    B.release_workspaces()
    assert nodes() < alone  # with all memory free the run takes fewer chunks
