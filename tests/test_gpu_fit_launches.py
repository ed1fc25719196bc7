"""A small group's fit takes at most 250 Adam steps a launch, so that a long fit
leaves the device to other streams between launches; the steps go on from the
state that the last launch left, and the fit has the bits of one launch per
kernel and step."""

import ctypes

import numpy as np
import pytest
import torch

import paper_2512_24840_amd as lasp
from paper_2512_24840_amd.lasp import FitResult
from synth import make_basis, make_spectra, shape_by_name, wave_grid

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")
B, P, MARGIN, DEGREE = 5, 257, 17, 4


@pytest.fixture(scope="module")
def prob():
    shape = shape_by_name("lamost3900", n_pix=P, margin=MARGIN, degree=DEGREE)
    basis, lines = make_basis(shape)
    batch = make_spectra(shape, lines, 78, 0, B)
    return shape, [torch.from_numpy(x).to(DEV) for x in (batch.obs, batch.ivar, basis, batch.init)]


def fit(prob, n_steps, **kw):
    shape, (obs, ivar, basis, init) = prob
    return lasp.fit_group(obs, ivar, wave_grid(shape), basis, init, n_steps, margin=MARGIN,
                          degree=DEGREE, **kw)


@pytest.mark.parametrize("n_steps", [249, 250, 251, 500, 777])
def test_steps_across_launches_equal_single_steps(prob, n_steps):
    print(f"[fit launches] {n_steps} steps", flush=True)
    out = []
    for one in (True, False):
        r = fit(prob, n_steps, want_cov=True, step_graph=one)
        torch.cuda.synchronize()
        out.append({k: getattr(r, k).cpu().numpy()
                    for k in ("params", "status", "chi2", "steps", "cov")})
    for k in out[0]:
        assert np.array_equal(out[0][k], out[1][k], equal_nan=True), k
    assert np.all(out[0]["steps"] == n_steps)


def test_a_launch_takes_at_most_250_steps(prob):
    print("[fit launches] kernels of one captured call", flush=True)
    hip = lasp.load()                       # its HIP runtime's names come with it
    stream = torch.cuda.Stream(device=DEV)
    out = FitResult(torch.empty((B, 5), dtype=torch.float32, device=DEV), None,
                    torch.empty(B, dtype=torch.int32, device=DEV),
                    torch.empty(B, dtype=torch.float64, device=DEV))
    fit(prob, 1, out=out, stream=stream)    # scratch of this stream
    torch.cuda.synchronize()

    def kernels(n_steps):
        st, graph, n = ctypes.c_void_p(stream.cuda_stream), ctypes.c_void_p(), ctypes.c_size_t()
        assert hip.hipStreamBeginCapture(st, 1) == 0
        fit(prob, n_steps, out=out, stream=stream)
        assert hip.hipStreamEndCapture(st, ctypes.byref(graph)) == 0
        assert hip.hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0
        assert hip.hipGraphDestroy(graph) == 0
        return n.value

    base = kernels(250)
    assert [kernels(k) - base for k in (1, 251, 500, 501, 1000)] == [0, 1, 1, 2, 3]
