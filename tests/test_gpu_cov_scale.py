"""The covariance's scale s^2 = chi2 / (n_eff - 5) is summed in FP64 from the
pixels up.

Every 17th pixel (a lane's first) carries the fit and a term of about 1 in
chi2.  The sixteen after it add 0.9 of half a last bit of that term in FP32
each, so a sum over a lane in FP32 loses all of them, 6e-7 of chi2; they are
1e-10 of every other sum.  Against the same spectrum without those pixels the
covariance must change by the change of s^2 alone."""

import numpy as np
import pytest
import torch

import oracle
import paper_2512_24840_amd as lasp
from synth import BOX_HI, BOX_LO, make_basis, make_spectra, shape_by_name, wave_grid

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("oracle_lib")]
DEV = torch.device("cuda:0")


def heavy_and_light(name, n_pix, degree):
    shape = shape_by_name(name, n_pix=n_pix, degree=degree, arm_start=(), arm_sigma_kms=())
    basis, lines = make_basis(shape)
    batch = make_spectra(shape, lines, 76, 0, 1)
    cfg = oracle.Config.from_shape(shape, BOX_LO, BOX_HI)
    u = cfg.normalise(batch.init)[0].astype(np.float32)

    def ev(obs, ivar):
        return oracle.evaluate(cfg, obs, ivar, basis, u.astype(np.float64))

    fpp = ev(np.ones(n_pix, np.float32), np.ones(n_pix, np.float32))["fpp"]
    heavy = np.arange(n_pix) % 17 == 0
    sign = np.random.default_rng(9).choice([-1.0, 1.0], n_pix)
    obs = (100.0 * fpp + np.where(heavy, 0.1 * sign, 10.0)).astype(np.float32)
    ivar = np.where(heavy, 110.0, 0.0).astype(np.float32)
    e = obs - ev(obs, ivar)["model"]
    # a lane's large term, where its rounding to FP32 cannot move it to another
    # binade, and the half of its last bit
    term = (ivar * e ** 2)[heavy]
    mant, ex = np.frexp(term)                       # mant in [1/2, 1)
    half_bit = np.where((mant > 0.52) & (mant < 0.98), 2.0 ** (ex - 1.0 - 24.0), 0.0)
    light = np.where(heavy, 0.0, np.repeat(0.9 * half_bit, 17)[:n_pix])
    both = np.where(heavy, ivar, light / e ** 2).astype(np.float32)
    return shape, basis, u, obs, ivar, both, ev


@pytest.mark.parametrize("name,n_pix,degree", [("lamost1550", 1550, 8), ("lamost3900", 3900, 10),
                                               ("lamost3900", 7800, 10)])
def test_covariance_scale_holds_small_terms(name, n_pix, degree):
    print(f"[cov scale] {n_pix} px", flush=True)
    shape, basis, u, obs, ivar, both, ev = heavy_and_light(name, n_pix, degree)
    a, b = ev(obs, ivar), ev(obs, both)
    grown = b["chi2"] / a["chi2"] - 1.0
    assert grown > 4e-7
    o = torch.from_numpy(np.stack([obs, obs])).to(DEV)
    iv = torch.from_numpy(np.stack([ivar, both])).to(DEV)
    uu = torch.from_numpy(np.stack([u, u])).to(DEV)
    kw = dict(margin=shape.margin, degree=degree, want_cov=True)
    bas = torch.from_numpy(basis).to(DEV)
    for grad in (False, True):           # alone, and after the fused pass
        r = lasp.forward(o, iv, wave_grid(shape), bas, uu, want_grad=grad, **kw)
        torch.cuda.synchronize()
        cov, n = r["cov"].cpu().numpy(), r["n_eff"].cpu().numpy()
        assert not np.any(r["status"].cpu().numpy() & lasp.ST_SINGULAR)
        d = np.arange(5)
        ratio = cov[1, d, d] / cov[0, d, d] * (n[1] - 5) / (n[0] - 5) - 1.0
        # FP32 sums may round otherwise in a lane or two: far below 1e-7
        assert np.all(np.abs(ratio - grown) <= 1e-7), (ratio, grown)
