"""The life cycle in stages on the CPU harness, every memory access checked:
the same packages, walks and contributions as the lane machine.  Every
package's arithmetic is the same to the bit, so counts and the tape (one entry
per event, no sums) are equal; images and gradients add the same terms in
another order, n of them of one sign within n 2^-53 of each other: 1e-11 for
the 1e4 terms of these runs, 1e-10 where a gradient's signs are mixed."""
import numpy as np
import pytest

BOX = (-1, 1, -1, 1, -0.5, 0.5)
COUNTS = ("x_path", "x_locate", "x_peel", "events", "packages", "peels", "deposits", "x_queue")


@pytest.fixture(autouse=True)
def _lane_machine_after(E):
    yield
    E.set_stages(0)


def _problem(W, kind, precision, n_pkg=700, **more):
    rng = np.random.default_rng(5)
    n = (9, 7, 6)
    dets = [W.frame(10.0, 40.0, 12, 10, 1.2, 1.1), W.frame(10.0, 90.0, 8, 8, 0.8, 0.8)]
    if kind == "instruments":
        dets = [W.sed(10.0, 30.0), W.perspective((0.3, 0.2, 0.1), (0.0, 0.0, 0.0), (0, 0, 1), 9, 9, 0.5, 0.5)]
    if kind == "tree":
        blob = lambda x, y, z: np.exp(-3.0 * (x * x + y * y + z * z))
        return dict(W.tree_problem("stages_tree", BOX, W.adaptive_tree(BOX, blob, 2e-2, 9), blob, 4.0, 0.6, 0.4,
                                   [W.point()], dets, n_pkg, precision, flags=3), **more)
    rho = np.exp(rng.standard_normal((n[2], n[1], n[0])) - 0.5)
    if precision == 1:
        rho = W.as_f32_values(rho)
    kw = dict(kappa=2.0, albedo=0.7, g=0.5, n_packages=n_pkg, flags=3)
    if kind == "lambdas":  # several wavelengths, one of them dark, direct and scattered light apart
        kw.update(kappa=[2.0, 1.0, 0.5], albedo=[0.8, 0.5, 0.0], g=[0.6, 0.0, -0.3], n_packages=n_pkg // 3 + 1,
                  flags=3 | W.FLAG_SPLIT, sources=[W.point(lum=[1.0, 0.0, 2.0]), W.expdisk(0.3, 0.1, lum=[0.5, 0.0, 1.0])])
    p = W.small_problem("stages", n, BOX, rho=rho, detectors=dets, precision=precision, seed=77, **kw)
    if kind == "rect":
        p["planes"] = tuple(W.power_law_planes(BOX[2 * a], BOX[2 * a + 1], n[a], 5.0) for a in range(3))
    return dict(p, **more)


def _rel(a, b):
    return float(np.abs(a - b).sum() / np.abs(b).sum())


def _both(E, p, stages, tape=False, **kw):
    """(images, stats, gradient, gradient's stats, tape) of the lane machine and in stages."""
    out = []
    adj = None
    for s in ((0, 0), stages):
        E.set_stages(*s)
        t = E.new_tape(p) if tape else None
        img, _, st = E.run(p, tape=t, **kw)
        if adj is None:
            adj = np.random.default_rng(1).standard_normal(img.shape)
        g, gst = E.grad(p, adj, **kw)
        out.append((img, st, g, gst, t))
    return out


def _same(lanes, staged):
    (img0, st0, g0, gst0, t0), (img1, st1, g1, gst1, t1) = lanes, staged
    for k in COUNTS:
        assert st1[k] == st0[k] and gst1[k] == gst0[k], k
    for k in ("absorbed", "escaped", "truncated"):
        assert abs(st1[k] - st0[k]) <= 1e-11 * st0["emitted"], k
    assert img0.sum() > 0.0 and _rel(img1, img0) < 1e-11
    assert np.abs(g0).sum() > 0.0 and _rel(g1, g0) < 1e-10
    if t0 is not None:
        assert np.array_equal(t0, t1)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("kind", ["regular", "rect", "tree", "lambdas", "instruments"])
@pytest.mark.parametrize("stages", [(1, 12), (1, 2), (150, 12)])
def test_stages_match_the_lane_machine(E, W, kind, precision, stages):
    _same(*_both(E, _problem(W, kind, precision), stages, tape=True))


@pytest.mark.parametrize("kind", ["regular", "lambdas"])
def test_all_orders_end_in_the_lane_machine(E, W, kind):
    """Every order runs in stages and the last list still has packages: none has more than one event after them."""
    p = _problem(W, kind, 0, n_pkg=300, w_min=0.0, max_scatter=13, albedo=[0.95] * (3 if kind == "lambdas" else 1))
    lanes, staged = _both(E, p, (1, 12))
    _same(lanes, staged)
    born = p["n_packages"] * (2 if kind == "lambdas" else 1)
    assert staged[1]["events"] > 12 * born


@pytest.mark.parametrize("kind", ["regular", "rect", "tree"])
def test_opaque_walls_that_absorb_everything(E, W, kind):
    """Cells of infinite density and albedo 0 (FP64): a leg into one is absorbed whole, also where its walk ends
    inside a block of crossings.  (With scattered light the walk that starts at such a cell's face has no depth.)"""
    p = _problem(W, kind, 0, n_pkg=400, albedo=[0.0])
    rho = np.array(p["rho"], dtype=np.float64)
    if kind == "tree":
        rho[::7] = np.inf
    else:
        rho = rho.reshape(6, 7, 9)
        rho[:, :, -1] = rho[0] = np.inf
    p["rho"] = rho
    out = []
    for s in ((0, 0), (1, 12)):
        E.set_stages(*s)
        out.append(E.run(p))
    (img0, _, st0), (img1, _, st1) = out
    assert np.isfinite(img0).all() and st0["absorbed"] > 0.9 * st0["emitted"]
    for k in COUNTS:
        assert st1[k] == st0[k], k
    for k in ("absorbed", "escaped", "truncated"):
        assert abs(st1[k] - st0[k]) <= 1e-11 * st0["emitted"], k
    assert np.abs(img1 - img0).sum() <= 1e-11 * img0.sum()  # the tree's source is walled in: no light


@pytest.mark.parametrize("cap", [1, 500])
def test_a_full_queue_is_walked_by_the_events(E, W, cap):
    """FP64, so the walks in the queue and here agree; which rays they take does not."""
    p = _problem(W, "lambdas", 0)
    E.set_stages(0)
    img0, _, st0 = E.run(p, peel_queue=1 << 16)
    adj = np.random.default_rng(1).standard_normal(img0.shape)
    g0, _ = E.grad(p, adj, peel_queue=1 << 16)
    E.set_stages(1, 12)
    img1, _, st1 = E.run(p, peel_queue=cap)
    g1, _ = E.grad(p, adj, peel_queue=cap)
    assert st1["x_queue"] < st0["x_queue"] and st1["x_peel"] == st0["x_peel"]
    assert _rel(img1, img0) < 1e-11 and _rel(g1, g0) < 1e-10


@pytest.mark.parametrize("more", [dict(flags=1), dict(flags=2), dict(flags=0), dict(first_package=(1 << 33) + 5),
                                  dict(max_scatter=1), dict(max_scatter=2, w_min=0.0), dict(w_min=0.5),
                                  dict(albedo=[1.0, 0.0, 0.3], g=[0.0, 0.9, -0.9], max_scatter=30)])
def test_run_options(E, W, more):
    """Peel-off at emission or scattering alone or not at all, packages of a later range, ends by count and weight."""
    p = _problem(W, "lambdas", 0, n_pkg=400, **more)
    p["flags"] = p["flags"] | W.FLAG_SPLIT if p["flags"] & 3 else 0
    E.set_stages(0)
    img0, _, st0 = E.run(p)
    E.set_stages(1, 12)
    img1, _, st1 = E.run(p)
    for k in COUNTS:
        assert st1[k] == st0[k], k
    for k in ("absorbed", "escaped", "truncated"):
        assert abs(st1[k] - st0[k]) <= 1e-11 * st0["emitted"], k
    assert np.abs(img1 - img0).sum() <= 1e-11 * img0.sum()
    assert (img0.sum() > 0.0) == bool(p["flags"] & 3)


@pytest.mark.parametrize("max_chunk", [64, 257])
def test_chunks(E, W, max_chunk):
    _same(*_both(E, _problem(W, "lambdas", 1), (1, 12), tape=True, max_chunk=max_chunk))


def test_stages_against_the_oracle(E, orc, W):
    p = _problem(W, "lambdas", 0)
    E.set_stages(1, 12)
    img, _, _ = E.run(p)
    img_o, _, _ = orc.run(p)
    assert _rel(img, img_o) < 1e-11
    adj = np.random.default_rng(3).standard_normal(img.shape)
    g, _ = E.grad(p, adj)
    g_o, _, _ = orc.grad(p, adj)
    assert _rel(g, g_o) < 1e-9
