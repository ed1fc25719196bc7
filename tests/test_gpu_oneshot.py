"""The one-shot evaluation's fused pass prepares its spectra itself; a grouped
fit of zero steps prepares them with k_prepare.  At the same parameters (up to
the rounding of u from its physical values) both give the same chi2 and the
same status, and outputs may take the place of u."""

import numpy as np
import pytest
import torch

import paper_2512_24840_amd as lasp
from synth import BOX_HI, BOX_LO, make_basis, make_spectra, shape_by_name, wave_grid

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.mark.parametrize("name,n_pix,margin,degree", [
    ("lamost3900", 32, 1, 4), ("lamost3900", 257, 17, 4), ("lamost1550", 1550, 64, 8),
    ("lamost3900", 2048, 64, 6), ("lamost3900", 3900, 64, 10), ("lamost3900", 4224, 64, 10),
    ("desi7800", 7800, 64, 10), ("desi7800", 8576, 64, 10)])
def test_oneshot_equals_the_prepared_pass(name, n_pix, margin, degree):
    print(f"[oneshot] {name} n_pix={n_pix} margin={margin} degree={degree}", flush=True)
    arms = {} if n_pix == 7800 else dict(arm_start=(), arm_sigma_kms=())
    shape = shape_by_name(name, n_pix=n_pix, margin=margin, degree=degree, **arms)
    basis, lines = make_basis(shape)
    batch = make_spectra(shape, lines, 71, 0, 5)
    obs, ivar = batch.obs.copy(), batch.ivar.copy()
    obs[1, n_pix // 2] = np.nan
    ivar[2] = 0.0
    ivar[3, 12:] = 0.0
    a = lasp.Arms(shape.arm_start, shape.arm_sigma_kms) if shape.arm_start else None
    kw = dict(margin=margin, degree=degree, arms=a)
    o, iv, bas, init = (torch.from_numpy(x).to(DEV) for x in (obs, ivar, basis, batch.init))
    grid = wave_grid(shape)
    fit = lasp.fit_group(o, iv, grid, bas, init, 0, **kw)
    # u as the fit forms it from the start
    th = batch.init.astype(np.float64)
    th[:, 0] = np.log10(th[:, 0])
    u = torch.from_numpy((2.0 * (th - BOX_LO) / (BOX_HI - BOX_LO) - 1.0).astype(np.float32)).to(DEV)
    res = lasp.forward(o, iv, grid, bas, u, want_grad=True, **kw)
    torch.cuda.synchronize()
    # the device's log10 may round one u elsewhere than numpy's: chi2 to 1e-5
    np.testing.assert_allclose(res["chi2"].cpu().numpy(), fit.chi2.cpu().numpy(), rtol=1e-5)
    assert np.array_equal(res["status"].cpu().numpy(), fit.status.cpu().numpy())
    # without the status and n_eff outputs, and with the gradient over u
    lib = lasp.load()
    import ctypes
    from paper_2512_24840_amd.lasp import make_opts
    for own_u in (True, False):
        opts = make_opts(5, n_pix, **kw)
        v = u.clone()
        grad = torch.empty_like(u) if own_u else v
        chi2 = torch.empty(5, dtype=torch.float64, device=DEV)
        p = [ctypes.c_void_p(t.data_ptr()) for t in (o, iv, bas, v, chi2, grad)]
        g = np.ascontiguousarray(grid)
        assert lib.lasp_forward(p[0], p[1], g.ctypes.data_as(ctypes.c_void_p), p[2], p[3], None,
                                p[4], None, None, p[5], None, None, ctypes.byref(opts)) == 0
        torch.cuda.synchronize()
        assert np.array_equal(chi2.cpu().numpy(), res["chi2"].cpu().numpy())
        assert np.array_equal(grad.cpu().numpy(), res["grad"].cpu().numpy())
