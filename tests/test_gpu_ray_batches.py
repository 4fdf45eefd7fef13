"""trace_path and peel_off choose their walk by the number of rays (crossings
per step, rays per wavefront, the caller's own densities or a bricked copy):
a ray's optical depth is the same to the bit in every batch, and peel-off
images differ only by the order of their additions."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _grid(W, kind, precision):
    box, n = (-1, 1, -1, 1, -0.5, 0.5), (37, 21, 30)
    if kind == "tree":
        blob = lambda x, y, z: np.exp(-3.0 * (x * x + y * y + z * z))
        return W.tree_problem("rays_tree", box, W.adaptive_tree(box, blob, 1e-3, 15), blob, 1.0, 0.5, 0.3, [W.point()],
                              [W.frame(10.0, 30.0, 16, 16, 1.0, 1.0)], 1, precision)
    p = W.small_problem("rays", n, box, rho=W.lognormal_density(n, 1.0, seed=3, f32=precision == 1),
                        precision=precision)
    if kind == "rect":
        p["planes"] = tuple(W.power_law_planes(box[2 * a], box[2 * a + 1], n[a], 6.0) for a in range(3))
    return p


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("kind", ["regular", "rect", "tree"])
def test_batches_agree(kind, precision):
    import torch
    from paper_1410_1629_amd import binding as B
    from paper_1410_1629_amd import workloads as W
    p = _grid(W, kind, precision)
    rho = B.density_tensor(p)
    most = (1 << 20) + 3
    o, k = (torch.as_tensor(a, device="cuda") for a in W.random_rays(most, p["box"], seed=9))
    perm = torch.randperm(most, generator=torch.Generator().manual_seed(1)).cuda()
    o, k = o[perm].contiguous(), k[perm].contiguous()
    first, tau0 = 700, None
    for n in (first, (1 << 18) - 1, 1 << 18, most):
        tau = torch.empty(n, dtype=torch.float64, device="cuda")
        B.trace_path(p, rho, 1.3, precision, o[:n].contiguous(), k[:n].contiguous(), tau)
        tau0 = tau if tau0 is None else tau0
        assert torch.equal(tau[:first], tau0), n
    w = torch.rand(most, dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(2))
    dets = [W.frame(10.0, t, 16, 16, 1.0, 1.0) for t in (20.0, 90.0)]
    for n in (first, (1 << 20) - 1, most):  # two rays per event
        whole, parts = (torch.zeros(2 * 256, dtype=torch.float64, device="cuda") for _ in range(2))
        B.peel_off(p, rho, 1.3, 0.4, precision, o[:n].contiguous(), k[:n].contiguous(), w[:n].contiguous(), dets, whole)
        for a in range(0, n, 150001):
            s = slice(a, min(n, a + 150001))
            B.peel_off(p, rho, 1.3, 0.4, precision, o[s].contiguous(), k[s].contiguous(), w[s].contiguous(), dets, parts)
        assert float((whole - parts).abs().sum()) <= 1e-10 * float(parts.sum()), n  # 1e6 terms: n 2^-53
