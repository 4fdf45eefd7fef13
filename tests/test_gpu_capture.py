"""A call on one stream while another stream is recorded into a graph (in the
global mode, where a query of any event ends a recording): the recording goes
on, the call gives what it gives alone, and the graph does its own work.
Device memory that calls on a third stream left behind is there to be taken,
so the calls look at its state."""
import ctypes as C

import hiprt
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _calls(B, W):
    """Name -> (call into its output, output) of every entry point that does not wait."""
    import torch
    n = (16, 15, 14)
    p = W.small_problem("capture", n, rho=W.lognormal_density(n, 1.0, seed=1), n_packages=3000, precision=0, flags=3,
                        seed=3, detectors=[W.frame(10.0, 30.0, 16, 16, 1.0, 1.0)])
    rho = B.density_tensor(p)
    o, k = (torch.as_tensor(a, device="cuda") for a in W.random_rays(5000, p["box"], seed=9))
    new = lambda *shape: torch.zeros(shape, dtype=torch.float64, device="cuda")
    w, adj, lum = new(5000) + 1.0, new(*B.image_shape(p)) + 1.0, rho.view(1, -1).clone()
    lam = np.geomspace(1.0, 100.0, 5)
    tau, frames, images, grad, em = (new(5000), new(256), new(*B.image_shape(p)), new(rho.numel()),
                                     new(5, rho.numel()))
    calls = {
        "trace_path": (lambda: B.trace_path(p, rho, 1.0, 0, o, k, tau, crossings=False), tau),
        "peel_off": (lambda: B.peel_off(p, rho, 1.0, 0.3, 0, o, k, w, p["detectors"], frames), frames),
        "run_photons": (lambda: B.run_photons(p, rho, images, stats=False), images),
        "backward_density": (lambda: B.backward_density(p, rho, adj, grad, stats=False), grad),
        "dust_emission": (lambda: B.dust_emission(p, rho, 0, lum, lam, 0.1 * lam, lam ** -1.5, 1.0, em), em),
    }
    return calls, (p, rho, o, k, w, adj, lum)


@pytest.mark.parametrize("name", ["trace_path", "peel_off", "run_photons", "backward_density", "dust_emission"])
def test_a_recording_goes_on_beside_a_call(name):
    import torch
    from paper_1410_1629_amd import binding as B
    from paper_1410_1629_amd import workloads as W
    hip = hiprt.load()
    calls, keep = _calls(B, W)
    call, out = calls[name]
    recorded, beside, other = (torch.cuda.Stream() for _ in range(3))
    x, y = torch.ones(1000, device="cuda"), torch.zeros(1000, device="cuda")
    y.add_(x)  # the kernel of the recording is loaded
    with torch.cuda.stream(other):
        call()
    torch.cuda.synchronize()
    alone = out.clone()
    out.zero_()
    y.zero_()
    torch.cuda.synchronize()
    graph, exe = C.c_void_p(), C.c_void_p()
    assert hip.hipStreamBeginCapture(C.c_void_p(recorded.cuda_stream), 0) == 0
    with torch.cuda.stream(recorded):
        y.add_(x)
    failed = None
    with torch.cuda.stream(beside):
        try:
            call()
        except Exception as e:
            failed = e
    with torch.cuda.stream(recorded):
        y.add_(x)
    ended = hip.hipStreamEndCapture(C.c_void_p(recorded.cuda_stream), C.byref(graph))
    hip.hipGetLastError()
    assert failed is None and ended == 0, (failed, ended)
    torch.cuda.synchronize()
    assert float((out - alone).abs().sum()) <= 1e-11 * float(alone.abs().sum())  # sums of the same terms
    assert float(alone.abs().sum()) > 0.0 and float(y.sum()) == 0.0
    assert hip.hipGraphInstantiate(C.byref(exe), graph, None, None, 0) == 0
    for n in (1, 2):
        assert hip.hipGraphLaunch(exe, C.c_void_p(recorded.cuda_stream)) == 0
        torch.cuda.synchronize()
        assert torch.equal(y, 2.0 * n * x)
        call()
        torch.cuda.synchronize()
    assert hip.hipGraphExecDestroy(exe) == 0 and hip.hipGraphDestroy(graph) == 0
