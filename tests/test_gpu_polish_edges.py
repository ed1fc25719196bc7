"""The one-launch Levenberg-Marquardt polish at the edges of its kernel: block
sizes, the lines between the two forms of the continuum moments, odd rows,
several arms and emulator classes, rows without data beside good ones, and each
way its iteration ends (its own stop, a dropped last step, the limit)."""

import numpy as np
import pytest
import torch

import oracle
import paper_2512_24840_amd as lasp
from synth import BOX_HI, BOX_LO, make_basis, make_spectra, shape_by_name, wave_grid

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("oracle_lib")]
DEV = torch.device("cuda:0")
THREE = dict(arm_start=(0, 401, 1100), arm_sigma_kms=(60.0, 40.0, 30.0))
CASES = [
    ("lamost1550", 257, 17, 4, {}, 1), ("lamost1550", 600, 64, 6, {}, 1),
    ("lamost1550", 700, 64, 6, {}, 1), ("lamost1550", 1170, 64, 8, {}, 1),
    ("lamost1550", 1300, 64, 8, {}, 1), ("lamost1550", 1550, 64, 8, THREE, 1),
    ("lamost3900", 1850, 64, 10, {}, 1), ("lamost3900", 2048, 64, 10, {}, 1),
    ("lamost3900", 2049, 64, 10, {}, 1), ("lamost3900", 4224, 64, 10, {}, 1),
    ("lamost3900", 4225, 64, 10, {}, 1), ("desi7800", 7800, 64, 10, None, 1),
    ("desi7800", 8576, 64, 10, {}, 1), ("lamost1550", 801, 64, 6, {}, 3),
    ("lamost3900", 2049, 64, 10, {}, 3)]


@pytest.mark.parametrize("name,n_pix,margin,degree,arms,classes", CASES)
def test_polish_ends_at_a_minimum_whatever_stands_beside_it(name, n_pix, margin, degree, arms,
                                                           classes):
    print(f"[LM edges] n_pix={n_pix} degree={degree} arms={bool(arms) or arms is None} "
          f"classes={classes}", flush=True)
    over = {} if arms is None else {"arm_start": (), "arm_sigma_kms": (), **arms}
    shape = shape_by_name(name, n_pix=n_pix, margin=margin, degree=degree, **over)
    basis, lines = make_basis(shape, n_classes=classes)
    batch = make_spectra(shape, lines, 77, 0, 6)
    cfg = oracle.Config.from_shape(shape, BOX_LO, BOX_HI, n_classes=classes)
    a = lasp.Arms(shape.arm_start, shape.arm_sigma_kms) if shape.arm_start else None
    kw = dict(margin=margin, degree=degree, arms=a, n_classes=classes)
    bas = torch.from_numpy(basis).to(DEV)

    def fit(limit, bad=False):
        obs, ivar, init = batch.obs, batch.ivar, batch.init
        if bad:                             # three rows without a fit between the others
            obs, ivar, init = (np.repeat(x, [1, 2, 1, 2, 1, 2], axis=0) for x in (obs, ivar, init))
            ivar[2], ivar[5, 12:], obs[8] = 0.0, 0.0, np.nan
        r = lasp.fit_group(*(torch.from_numpy(x).to(DEV) for x in (obs, ivar)), wave_grid(shape),
                           bas, torch.from_numpy(init).to(DEV), 0, polish_iters=limit, **kw)
        torch.cuda.synchronize()
        out = {k: getattr(r, k).cpu().numpy() for k in ("params", "status", "chi2")}
        return {k: v[[0, 1, 3, 4, 6, 7]] for k, v in out.items()} if bad else out

    full = fit(200)
    assert not np.any(full["status"] & lasp.ST_POLISH_LIMIT)
    # the oracle's fit from there stays there: the polish promises 1e-3 standard
    # deviations, FP32 sums leave less
    for i in range(6):
        u = cfg.normalise(full["params"][i].astype(np.float64))
        ref = oracle.fit(cfg, batch.obs[i], batch.ivar[i], basis, u)
        sd = np.sqrt(np.diag(ref["cov_u"]))
        assert np.all(np.abs(ref["u"] - u) <= 0.05 * sd + 1e-6), (i, (ref["u"] - u) / sd)
    beside = fit(200, bad=True)
    for k in full:
        assert np.array_equal(beside[k], full[k]), k
    # a smaller limit cuts the same iteration short, or does not touch it
    last = None
    for limit in (1, 2, 3, 4, 6, 9):
        r = fit(limit)
        ended = (r["status"] & lasp.ST_POLISH_LIMIT) == 0
        for k in full:
            assert np.array_equal(r[k][ended], full[k][ended]), (limit, k)
        assert last is None or np.all(r["chi2"] <= last * (1.0 + 1e-6)), limit
        last = r["chi2"]
