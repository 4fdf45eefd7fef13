"""The life cycle in stages (runs of at least 2^20 packages without an
absorbed tally, and the adjoint's first replay): the same packages, walks and
contributions as the lane machine, which runs the same call in chunks below
that size.  Every package's arithmetic is the same to the bit, so counts are
equal and sums differ only by the order of their additions: n of them of one
sign by at most n 2^-53, 1e-10 for the 1e6 contributions of one pixel, and a
gradient's mixed signs by the same bound on the sum of magnitudes."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# Room for every ray: FP32 rays beyond a queue are walked in other times than
# queued ones, and which rays those are depends on the chunks.
QUEUE = 1 << 26
ITEMS = (1 << 20) + 777  # just over the smallest chunk in stages; lists below it go to the lane machine


def _problem(W, kind, precision, n_pkg):
    rng = np.random.default_rng(5)
    box, n = (-1, 1, -1, 1, -0.5, 0.5), (19, 17, 11)
    kw = dict(n_packages=n_pkg, precision=precision, flags=3, seed=77)
    dets = [W.frame(10.0, 40.0, 24, 20, 1.2, 1.1), W.frame(10.0, 90.0, 16, 16, 0.8, 0.8)]
    if kind == "instruments":
        dets = [W.sed(10.0, 30.0), W.perspective((0.3, 0.2, 0.1), (0.0, 0.0, 0.0), (0, 0, 1), 12, 12, 0.5, 0.5)]
    if kind == "tree":
        blob = lambda x, y, z: np.exp(-3.0 * (x * x + y * y + z * z))
        return W.tree_problem("stages_tree", box, W.adaptive_tree(box, blob, 2e-3, 15), blob, 4.0, 0.6, 0.4,
                              [W.point()], dets, n_pkg, precision, flags=3)
    rho = np.exp(rng.standard_normal((n[2], n[1], n[0])) - 0.5)
    if precision == 1:
        rho = W.as_f32_values(rho)
    if kind == "lambdas":  # several wavelengths, one of them dark, direct and scattered light apart
        kw.update(kappa=[2.0, 1.0, 0.5], albedo=[0.8, 0.5, 0.0], g=[0.6, 0.0, -0.3], n_packages=n_pkg // 3 + 1,
                  flags=3 | W.FLAG_SPLIT, sources=[W.point(lum=[1.0, 0.0, 2.0]), W.expdisk(0.3, 0.1, lum=[0.5, 0.0, 1.0])])
    else:
        kw.update(kappa=2.0, albedo=0.7, g=0.5)
    p = W.small_problem("stages", n, box, rho=rho, detectors=dets, **kw)
    if kind == "rect":
        p["planes"] = tuple(W.power_law_planes(box[2 * a], box[2 * a + 1], n[a], 5.0) for a in range(3))
    return p


def _rel(a, b):
    return float((a - b).abs().sum() / b.abs().sum())


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("kind", ["regular", "rect", "tree", "lambdas", "instruments"])
def test_stages_match_the_lane_machine(kind, precision):
    import torch
    from paper_1410_1629_amd import binding as B
    from paper_1410_1629_amd import workloads as W
    p = _problem(W, kind, precision, ITEMS)
    rho = B.density_tensor(p)
    images, lanes = (torch.empty(B.image_shape(p), dtype=torch.float64, device="cuda") for _ in range(2))
    a = B.run_photons(p, rho, images, peel_queue=QUEUE)
    b = B.run_photons(p, rho, lanes, max_chunk=1 << 19, peel_queue=QUEUE)
    for k in ("x_path", "x_locate", "x_peel", "events", "packages", "peels"):
        assert a[k] == b[k], (k, a[k], b[k])
    for k in ("absorbed", "escaped", "truncated"):
        assert abs(a[k] - b[k]) <= 1e-10 * a["emitted"], (k, a[k], b[k])
    assert _rel(images, lanes) < 1e-10
    # pass A of the adjoint in stages
    adj = torch.as_tensor(np.random.default_rng(1).standard_normal(images.numel()), device="cuda").view_as(images)
    ga, gb = (torch.empty(rho.numel(), dtype=torch.float64, device="cuda") for _ in range(2))
    a = B.backward_density(p, rho, adj, ga, peel_queue=QUEUE)
    b = B.backward_density(p, rho, adj, gb, max_chunk=1 << 19, peel_queue=QUEUE)
    for k in ("x_path", "x_locate", "x_peel", "events", "packages", "peels", "deposits"):
        assert a[k] == b[k], (k, a[k], b[k])
    assert _rel(ga, gb) < 1e-9  # the terms' magnitudes sum to some ten times the result's


@pytest.mark.parametrize("cap", [1, 100000])
def test_stages_with_a_full_queue(cap):
    """Rays beyond the queue's capacity are walked by the event kernels; FP64, so both walks agree."""
    import torch
    from paper_1410_1629_amd import binding as B
    from paper_1410_1629_amd import workloads as W
    p = _problem(W, "regular", 0, ITEMS)
    rho = B.density_tensor(p)
    images, ref = (torch.empty(B.image_shape(p), dtype=torch.float64, device="cuda") for _ in range(2))
    a = B.run_photons(p, rho, images, peel_queue=cap)
    b = B.run_photons(p, rho, ref, peel_queue=QUEUE)
    for k in ("x_path", "x_locate", "x_peel", "events", "packages", "peels"):
        assert a[k] == b[k], (k, a[k], b[k])
    assert a["x_queue"] < b["x_queue"]
    assert _rel(images, ref) < 1e-10
    adj = torch.ones_like(images)
    ga, gb = (torch.empty(rho.numel(), dtype=torch.float64, device="cuda") for _ in range(2))
    B.backward_density(p, rho, adj, ga, peel_queue=cap)
    B.backward_density(p, rho, adj, gb, peel_queue=QUEUE)
    assert _rel(ga, gb) < 1e-9


def test_stages_against_the_oracle(orc):
    import torch
    from paper_1410_1629_amd import binding as B
    from paper_1410_1629_amd import workloads as W
    p = _problem(W, "regular", 0, ITEMS)
    rho = B.density_tensor(p)
    images = torch.empty(B.image_shape(p), dtype=torch.float64, device="cuda")
    B.run_photons(p, rho, images)
    ref = np.asarray(orc.run(p, threads=16)[0]).ravel()
    assert np.abs(images.cpu().numpy().ravel() - ref).sum() < 1e-10 * np.abs(ref).sum()
