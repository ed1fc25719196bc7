"""A small FP32 group's Adam steps in one launch, a workgroup per spectrum,
against the same steps as three launches each (step_graph=False): the same
operations in the same order, so every output must agree bit for bit -- at the
edges of the pixel chunks, the block sizes, odd counts of 16-pixel chunks,
one and several arms, spectra without data, and one spectrum past the largest
group that takes the one launch."""

import numpy as np
import pytest
import torch

import paper_2512_24840_amd as lasp
from synth import make_basis, make_spectra, shape_by_name, wave_grid

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.mark.parametrize("name,n_pix,margin,degree,n_spec,n_steps", [
    ("lamost3900", 32, 1, 4, 5, 7), ("lamost3900", 257, 17, 4, 5, 7),
    ("lamost1550", 1550, 64, 8, 5, 30), ("lamost3900", 2048, 64, 6, 5, 1),
    ("lamost3900", 2176, 64, 6, 5, 7), ("lamost3900", 2177, 64, 6, 5, 7),
    ("lamost3900", 3900, 64, 10, 5, 30), ("lamost3900", 4224, 64, 10, 5, 7),
    ("lamost3900", 4225, 64, 10, 5, 7), ("lamost3900", 4352, 64, 10, 5, 7),
    ("lamost3900", 4353, 64, 10, 5, 7), ("desi7800", 7800, 64, 10, 5, 7),
    ("desi7800", 8576, 64, 10, 5, 7), ("lamost3900", 257, 17, 4, 1024, 3),
    ("lamost3900", 257, 17, 4, 1025, 26), ("lamost3900", 4353, 64, 4, 256, 3),
    ("lamost3900", 4353, 64, 4, 257, 26)])
def test_one_launch_equals_three_per_step(name, n_pix, margin, degree, n_spec, n_steps):
    print(f"[fit one launch] {name} n_pix={n_pix} margin={margin} B={n_spec} "
          f"steps={n_steps}", flush=True)
    arms = {} if n_pix == 7800 else dict(arm_start=(), arm_sigma_kms=())
    shape = shape_by_name(name, n_pix=n_pix, margin=margin, degree=degree, **arms)
    basis, lines = make_basis(shape)
    batch = make_spectra(shape, lines, 72, 0, 5)
    rep = -(-n_spec // 5)
    obs, ivar, init = (np.concatenate([x] * rep)[:n_spec]
                       for x in (batch.obs, batch.ivar, batch.init))
    obs[1, n_pix // 2] = np.nan
    ivar[2] = 0.0
    ivar[3, 12:] = 0.0
    init[:, 1] += np.linspace(0.0, 0.2, n_spec, dtype=np.float32)
    a = lasp.Arms(shape.arm_start, shape.arm_sigma_kms) if shape.arm_start else None
    o, iv, bas, ini = (torch.from_numpy(x).to(DEV) for x in (obs, ivar, basis, init))
    out = []
    for one in (True, False):
        r = lasp.fit_group(o, iv, wave_grid(shape), bas, ini, n_steps, margin=margin,
                           degree=degree, arms=a, want_cov=True, step_graph=one)
        torch.cuda.synchronize()
        out.append({k: getattr(r, k).cpu().numpy()
                    for k in ("params", "status", "chi2", "steps", "cov")})
    assert np.all(out[0]["steps"][3:5] == out[1]["steps"][3:5])
    for k in out[0]:
        assert np.array_equal(out[0][k], out[1][k], equal_nan=True), k
