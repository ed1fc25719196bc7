"""Continuum moments on both sides of each line between the pixel sums and the
node sums, against the FP64 oracle, under the forward pass's bars."""

import numpy as np
import pytest
import torch

import oracle
import paper_2512_24840_amd as lasp
from synth import BOX_HI, BOX_LO, make_basis, make_spectra, shape_by_name, wave_grid

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("oracle_lib")]
DEV = torch.device("cuda:0")


@pytest.mark.parametrize("n_pix,margin,degree", [
    (236, 64, 4), (240, 64, 4), (628, 64, 6), (632, 64, 6), (1175, 64, 8), (1177, 64, 8),
    (1871, 64, 10), (1873, 64, 10), (2017, 80, 10), (4224, 64, 10), (8544, 80, 10)])
def test_forward_matches_the_oracle_beside_each_line(n_pix, margin, degree):
    print(f"[moments] n_pix={n_pix} margin={margin} degree={degree}", flush=True)
    name = "desi7800" if n_pix > 4300 else "lamost3900"
    shape = shape_by_name(name, n_pix=n_pix, margin=margin, degree=degree, arm_start=(),
                          arm_sigma_kms=())
    basis, lines = make_basis(shape)
    batch = make_spectra(shape, lines, 83, 0, 4)
    cfg = oracle.Config.from_shape(shape, BOX_LO, BOX_HI)
    u = (cfg.normalise(batch.init) + np.random.default_rng(6).normal(0, 0.03, (4, 5)))
    u = u.astype(np.float32)
    res = lasp.forward(*(torch.from_numpy(a).to(DEV) for a in (batch.obs, batch.ivar)),
                       wave_grid(shape), torch.from_numpy(basis).to(DEV),
                       torch.from_numpy(u).to(DEV), want_model=True, want_grad=True,
                       margin=margin, degree=degree)
    torch.cuda.synchronize()
    for i in range(4):
        ref = oracle.evaluate(cfg, batch.obs[i], batch.ivar[i], basis, u[i].astype(np.float64))
        rms = np.sqrt(np.mean(ref["model"] ** 2))
        assert np.max(np.abs(res["model"][i].cpu().numpy() - ref["model"])) <= 1e-5 * rms, i
        assert float(res["chi2"][i]) == pytest.approx(ref["chi2"], rel=1e-5), i
        g, gr = res["grad"][i].cpu().numpy(), ref["grad"]
        assert np.linalg.norm(g - gr) <= 1e-5 * np.linalg.norm(gr) + 1e-9, (i, g, gr)
