"""The optics and luminosity gradients of wavelengths summed in parts (from
8192 packages of a wavelength in one chunk), around the lines where a part
is added and where a chunk cuts a wavelength, against the same call in chunks
of one part.  The sums' terms are the same; n <= 2e4 terms of both signs
whose magnitudes add up to at most 1e3 times the result differ by 2e4 2^-53 1e3
= 2e-9: 5e-9.  A lost package is 1/n, 5e-5."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("chunk", [0, 15001])
@pytest.mark.parametrize("n_pkg", [4095, 8191, 8192, 8193, 12289, 20001])
def test_parts_add_up(n_pkg, chunk):
    import torch
    from paper_1410_1629_amd import binding as B
    from paper_1410_1629_amd import workloads as W
    p = W.small_problem("parts", (8, 7, 6), kappa=[1.0, 0.6, 0.8], albedo=[0.6, 0.4, 0.5], g=[0.4, -0.2, 0.0],
                        sources=[W.point((0.1, 0.0, -0.1), [1.0, 0.5, 0.0]), W.expdisk(0.4, 0.15, [0.7, 1.1, 0.0])],
                        detectors=[W.frame(10.0, 40.0, 12, 10, 1.2, 1.1)], n_packages=n_pkg, precision=0, flags=3,
                        seed=23)
    rho = B.density_tensor(p)
    adj = torch.as_tensor(np.random.default_rng(3).uniform(0.5, 1.5, B.image_shape(p)), device="cuda")
    out = []
    for kw in ({"max_chunk": chunk} if chunk else {}, {"max_chunk": 4000}):
        g = [torch.empty(n, dtype=torch.float64, device="cuda") for n in (3, 3, 6)]
        B.backward(p, rho, adj, None, *g, **kw)
        out.append(g)
    for a, b in zip(*out):
        assert float(b.abs().sum()) > 0.0
        assert float((a - b).abs().sum()) <= 5e-9 * float(b.abs().sum())
