"""Runs on a device that others have filled: a run that fits in what is free
beside them runs, whatever the library keeps and whatever path it would take
with more memory."""
import pytest

pytestmark = pytest.mark.gpu
GB = 1 << 30


def _hold(free):
    """Tensors that leave `free` bytes of the device (the first one's size in device memory is not quite its own)."""
    import torch
    held = []
    for _ in range(3):
        torch.cuda.synchronize()
        more = torch.cuda.mem_get_info()[0] - free
        if more > 1 << 22:
            held.append(torch.empty(more, dtype=torch.uint8, device="cuda"))
    assert abs(torch.cuda.mem_get_info()[0] - free) < 1 << 24
    return held


@pytest.fixture(autouse=True)
def _clean():
    import torch
    from paper_1410_1629_amd import binding as B
    B.release_workspaces()
    torch.cuda.empty_cache()
    yield
    B.release_workspaces()
    torch.cuda.empty_cache()


def test_a_kept_block_is_not_spent_on_less_than_the_run_needs():
    """A run with little free beside what is kept works as if nothing were kept: its queue takes as many rays."""
    import torch
    from paper_1410_1629_amd import binding as B
    from paper_1410_1629_amd import workloads as W
    p = dict(W.cube(n_packages=30_000_000, precision=1), flags=3)
    rho = B.density_tensor(p)
    adj = torch.ones(B.image_shape(p), dtype=torch.float64, device="cuda")
    grad = torch.empty(rho.numel(), dtype=torch.float64, device="cuda")
    B.backward_density(dict(p, n_packages=1000), rho, adj, grad, stats=False, peel_queue=24 * GB // 70)
    kept = B.kept_bytes()
    assert kept > 23 * GB
    # of 28 GB the event scratch takes about 7, and a quarter of the rest is the queue's
    held = _hold(4 * GB)
    beside = B.backward_density(p, rho, adj, grad)
    del held
    B.release_workspaces()
    torch.cuda.empty_cache()
    held = _hold(4 * GB + kept)
    alone = B.backward_density(p, rho, adj, grad)
    del held
    assert beside["packages"] == alone["packages"] == 30_000_000
    # which rays a full queue leaves out depends on their order
    assert abs(beside["x_queue"] - alone["x_queue"]) <= 0.02 * alone["x_queue"]


def test_a_run_without_room_for_the_stages_goes_without():
    """A grid that fills nine tenths of what is free leaves no room for the package lists of a run in stages."""
    import torch
    from paper_1410_1629_amd import binding as B
    from paper_1410_1629_amd import workloads as W
    n = 3_700_000  # their lists take 0.56 GB, of the 0.4 GB beside the densities
    p = dict(W.cube(n_packages=n, precision=0), n=(800, 800, 800), flags=3)
    rho = torch.ones(800 ** 3, dtype=torch.float64, device="cuda")  # 4.1 GB, and as much for the library's copy
    images = torch.empty(B.image_shape(p), dtype=torch.float64, device="cuda")
    held = _hold(4_500_000_000)
    st = B.run_photons(p, rho, images, peel_queue=100000)
    del held
    assert st["packages"] == n and float(images.sum()) > 0.0
