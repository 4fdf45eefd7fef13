"""The life cycle in stages through many orders: several wavelengths, all the
orders the stages take with a full list left over, the tape, the launch
options; against the lane machine, which runs the same call in chunks below
the size that stages need.  Counts and the tape's entries are equal to the
bit; sums add the same terms in another order, at most 1e6 of one sign per
pixel (1e-10), a gradient's mixed signs within ten times that."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

QUEUE = 1 << 27  # room for every ray of a chunk
STAGE_MIN, STAGE_ORDERS = 1 << 20, 12  # lists below this go to the lane machine, and so does what is left after these
N_PKG = 1 << 21
BOX = (-1, 1, -1, 1, -0.5, 0.5)
COUNTS = ("x_path", "x_locate", "x_peel", "events", "packages", "peels")


def _problem(W, precision, n_lambda, n_pkg, **kw):
    n = (19, 17, 11)
    rho = np.exp(np.random.default_rng(5).standard_normal((n[2], n[1], n[0])) - 0.5)
    dets = [W.frame(10.0, 40.0, 24, 20, 1.2, 1.1)]
    args = dict(rho=W.as_f32_values(rho) if precision == 1 else rho, detectors=dets, n_packages=n_pkg,
                precision=precision, flags=3, seed=77, kappa=4.0, albedo=0.95, g=0.5)
    if n_lambda == 3:  # the middle wavelength dark
        args.update(kappa=[4.0, 1.0, 6.0], albedo=[0.95, 0.5, 0.9], g=[0.6, 0.0, -0.3], flags=3 | W.FLAG_SPLIT,
                    sources=[W.point(lum=[1.0, 0.0, 2.0]), W.expdisk(0.3, 0.1, lum=[0.5, 0.0, 1.0])])
    args.update(kw)
    return W.small_problem("orders", n, BOX, **args)


def _run(B, p, rho, **kw):
    import torch
    images = torch.empty(B.image_shape(p), dtype=torch.float64, device="cuda")
    return images, B.run_photons(p, rho, images, peel_queue=QUEUE, **kw)


def _rel(a, b):
    return float((a - b).abs().sum() / b.abs().sum())


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n_lambda", [1, 3])
def test_every_order_with_a_full_list_left(n_lambda, precision):
    import torch
    from paper_1410_1629_amd import binding as B
    from paper_1410_1629_amd import workloads as W
    # every package has at most one event more than the stages take
    p = _problem(W, precision, n_lambda, N_PKG, w_min=0.0, max_scatter=STAGE_ORDERS + 1)
    rho = B.density_tensor(p)
    images, a = _run(B, p, rho)
    lanes, b = _run(B, p, rho, max_chunk=1 << 19)
    born = N_PKG * (2 if n_lambda == 3 else 1)
    # lists never grow, so the one after the last staged order holds at least the events beyond STAGE_ORDERS full lists
    assert a["events"] - STAGE_ORDERS * born >= STAGE_MIN
    for k in COUNTS:
        assert a[k] == b[k], (k, a[k], b[k])
    for k in ("absorbed", "escaped", "truncated"):
        assert abs(a[k] - b[k]) <= 1e-10 * a["emitted"], (k, a[k], b[k])
    assert _rel(images, lanes) < 1e-10
    adj = torch.as_tensor(np.random.default_rng(1).standard_normal(images.numel()), device="cuda").view_as(images)
    ga, gb = (torch.empty(rho.numel(), dtype=torch.float64, device="cuda") for _ in range(2))
    a = B.backward_density(p, rho, adj, ga, peel_queue=QUEUE)
    b = B.backward_density(p, rho, adj, gb, max_chunk=1 << 19, peel_queue=QUEUE)
    for k in COUNTS + ("deposits",):
        assert a[k] == b[k], (k, a[k], b[k])
    assert _rel(ga, gb) < 1e-9


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n_lambda", [1, 3])
def test_the_tape_is_the_lane_machines(n_lambda, precision):
    import torch
    from paper_1410_1629_amd import binding as B
    from paper_1410_1629_amd import workloads as W
    p = _problem(W, precision, n_lambda, STAGE_MIN + 777, w_min=1e-3, max_scatter=20, albedo=[0.8] * n_lambda)
    rho = B.density_tensor(p)
    tapes = [torch.zeros(B.tape_bytes(p), dtype=torch.uint8, device="cuda") for _ in range(2)]
    _, a = _run(B, p, rho, tape=tapes[0])
    _, b = _run(B, p, rho, tape=tapes[1], max_chunk=1 << 19)
    assert a["events"] == b["events"] > 3 * p["n_packages"]
    assert torch.equal(*tapes)


@pytest.mark.parametrize("options", [{"event_batch": 1}, {"event_batch": 64}, {"launch_blocks": 1},
                                     {"event_batch": 7, "launch_blocks": 3}])
def test_launch_options_change_no_package(options):
    from paper_1410_1629_amd import binding as B
    from paper_1410_1629_amd import workloads as W
    p = _problem(W, 1, 1, N_PKG)
    rho = B.density_tensor(p)
    images, a = _run(B, p, rho)
    other, b = _run(B, p, rho, **options)
    for k in COUNTS:
        assert a[k] == b[k], (k, a[k], b[k])
    assert _rel(other, images) < 1e-10
