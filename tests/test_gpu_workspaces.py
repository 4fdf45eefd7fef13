"""Device memory kept between calls: calls of different sizes on two streams
and two threads give what each gives alone, and the memory goes back."""
import threading

import pytest

pytestmark = pytest.mark.gpu


def _call(B, W, n, seed, stream):
    import torch
    p = W.small_problem("ws", (n, n + 1, n - 2), rho=W.lognormal_density((n, n + 1, n - 2), 1.0, seed=seed),
                        n_packages=20000 + 1000 * n, flags=7, seed=seed)
    with torch.cuda.stream(stream):
        rho = B.density_tensor(p)
        images, absorbed, _ = B.render(p, rho=rho, stats=False)
        grad = torch.empty(rho.numel(), dtype=torch.float64, device="cuda")
        B.backward_density(p, rho, torch.ones_like(images), grad, stats=False)
        stream.synchronize()
    return images.cpu(), absorbed.cpu(), grad.cpu()


def test_two_streams_and_threads():
    import torch
    from paper_1410_1629_amd import binding as B
    from paper_1410_1629_amd import workloads as W
    jobs = [(9, 1), (40, 2), (12, 3), (33, 4), (9, 5), (25, 6)]
    alone = {j: _call(B, W, *j, torch.cuda.current_stream()) for j in jobs}
    got, errors = {}, []

    def work(mine):
        try:
            stream = torch.cuda.Stream()
            for j in mine:
                got[j] = _call(B, W, *j, stream)
        except Exception as e:  # shown by the assertion below
            errors.append(e)

    threads = [threading.Thread(target=work, args=(m,)) for m in (jobs[::2], jobs[1::2])]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    for j in jobs:
        for a, b in zip(got[j], alone[j]):  # sums of the same terms in another order
            assert float((a - b).abs().sum()) <= 1e-11 * float(b.abs().sum()), j


def test_memory_goes_back():
    import torch
    from paper_1410_1629_amd import binding as B
    from paper_1410_1629_amd import workloads as W
    p = W.spiral(n_packages=1_000_000)
    rho = B.density_tensor(p)
    B.release_workspaces()
    images = torch.empty(B.image_shape(p), dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    B.run_photons(dict(p, flags=3), rho, images)
    torch.cuda.synchronize()
    assert torch.cuda.mem_get_info()[0] < before - (1 << 29)  # the peel-ray queue alone takes 1.7 GB
    B.release_workspaces()
    torch.cuda.synchronize()
    assert torch.cuda.mem_get_info()[0] > before - (1 << 28)
