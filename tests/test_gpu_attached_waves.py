"""The attached gradient's two forms (one wavefront per SIMD for calls of fewer
packages than it has lanes, two above, shared evenly between the wavefronts
up to their lanes) around the line between them, against the same call in
chunks that all take the first form.  Every package's arithmetic is the
same, so counts are equal and gradients differ by the order of their
additions: at most 1e5 terms per cell, each a unit of 2^-53 of the partial
sums, whose cancelled parts stay below 100 times the result: 1e-9.  A lost
package is 1e-5."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
LANES = 256 * 256  # of one wavefront per SIMD


@pytest.mark.parametrize("kind", ["regular", "rect", "tree"])
@pytest.mark.parametrize("n_pkg", [LANES - 1, LANES, LANES + 1, 2 * LANES - 63, 2 * LANES + 1])
def test_two_wavefronts_per_simd(kind, n_pkg):
    import torch
    from paper_1410_1629_amd import binding as B
    from paper_1410_1629_amd import workloads as W
    box, n = (-1, 1, -1, 1, -0.5, 0.5), (9, 8, 7)
    dets = [W.frame(10.0, 40.0, 12, 10, 1.2, 1.1)]
    if kind == "tree":
        blob = lambda x, y, z: np.exp(-3.0 * (x * x + y * y + z * z))
        p = W.tree_problem("waves", box, W.adaptive_tree(box, blob, 2e-2, 9), blob, 2.0, 0.6, 0.4, [W.point()], dets,
                           n_pkg, 0, flags=3)
    else:
        rho = np.exp(0.5 * np.random.default_rng(5).standard_normal((n[2], n[1], n[0])))
        p = W.small_problem("waves", n, box, rho=rho, detectors=dets, kappa=1.0, albedo=0.6, g=0.4, n_packages=n_pkg,
                            precision=0, flags=3, seed=21)
    if kind == "rect":
        p["planes"] = tuple(W.power_law_planes(box[2 * a], box[2 * a + 1], n[a], 5.0) for a in range(3))
    rho = B.density_tensor(p)
    adj = torch.ones(B.image_shape(p), dtype=torch.float64, device="cuda")
    one, parts = (torch.empty(rho.numel(), dtype=torch.float64, device="cuda") for _ in range(2))
    a = B.backward_density(p, rho, adj, one, attached=True)
    b = B.backward_density(p, rho, adj, parts, attached=True, max_chunk=LANES // 2)
    for k in ("x_path", "x_locate", "x_peel", "events", "packages", "peels", "deposits"):
        assert a[k] == b[k], (k, a[k], b[k])
    assert float((one - parts).abs().sum()) <= 1e-9 * float(parts.abs().sum())
    assert float(parts.abs().sum()) > 0.0
