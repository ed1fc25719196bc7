"""The preparation's flux weight: a power of two on every path of its search.

The objective does not depend on the weight, and a power of two leaves every
rounding where it is, so whatever branch finds it -- the bracket over
register counts, the search bit by bit, no weight at all -- the results
equal those of weight 1 bit for bit."""

import numpy as np
import pytest
import torch

import paper_2512_24840_amd as lasp
from synth import make_basis, make_spectra, shape_by_name, wave_grid

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def _rows(batch):
    """Rows whose quantile the bracket finds, and rows it must leave to the
    bitwise search: order statistics on both sides of 2^(b + 1/2) and right beside
    it, few valid pixels, nonpositive and widely scattered fluxes."""
    obs, ivar = batch.obs.copy(), batch.ivar.copy()
    half = obs.shape[1] // 2
    edge = np.float32(np.sqrt(2.0) * 64.0)
    obs[1] = edge * np.linspace(0.99999, 1.00001, obs.shape[1], dtype=np.float32)
    obs[2, :half] = 70.0                        # two values, the median between them
    obs[2, half:] = 120.0
    ivar[2] = ivar[2].max()
    ivar[3, 20:] = 0.0                          # few valid pixels
    obs[4] -= np.float32(np.median(obs[4]))     # median flux near zero
    obs[5] *= np.exp2(np.random.default_rng(5).integers(-12, 13, obs.shape[1])).astype(np.float32)
    obs[6] = 0.0
    obs[7, 3], ivar[7, 9], obs[7, 11] = np.nan, np.inf, -np.inf
    return obs, ivar


@pytest.mark.parametrize("name,n_pix", [("lamost3900", 257), ("lamost3900", 3900),
                                        ("desi7800", 7800), ("desi7800", 8576)])
@pytest.mark.parametrize("quantile", [0.5, 0.9])
def test_every_path_of_the_weight_gives_the_results_of_weight_one(name, n_pix, quantile):
    print(f"[prepare] n_pix={n_pix} quantile={quantile}", flush=True)
    shape = shape_by_name(name, n_pix=n_pix, arm_start=(), arm_sigma_kms=())
    basis, lines = make_basis(shape)
    batch = make_spectra(shape, lines, 61, 0, 9)
    obs, ivar = _rows(batch)
    dev = [torch.from_numpy(a).to(DEV) for a in (obs, ivar, basis)]
    u = torch.from_numpy(np.random.default_rng(4).uniform(-0.6, 0.6, (9, 5))
                         .astype(np.float32)).to(DEV)
    kw = dict(want_model=True, want_grad=True, margin=shape.margin, degree=shape.degree)
    got = [lasp.forward(dev[0], dev[1], wave_grid(shape), dev[2], u, weight_quantile=q, **kw)
           for q in (quantile, 0.0)]
    torch.cuda.synchronize()
    for key in ("chi2", "J", "grad", "model", "n_eff", "status"):
        a, b = (r[key].cpu().numpy() for r in got)
        assert np.array_equal(a, b, equal_nan=True), key
    assert got[0]["status"].cpu().numpy()[7] & lasp.ST_NONFINITE_INPUT
    ok = np.isfinite(obs) & np.isfinite(ivar) & (ivar > 0)
    assert np.array_equal(got[0]["n_eff"].cpu().numpy(), ok.sum(1))
