"""A forward call with the covariance or the model Jacobian but no gradient is
one kernel that prepares its spectra itself; with the gradient the fused pass
prepares and evaluates them.  Everything that both give has the same bits, over
block sizes, arms, classes and rows without data; and the Jacobian is the
oracle's."""

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
    ("lamost3900", 32, 1, 4, {}, 1), ("lamost3900", 257, 17, 4, {}, 1),
    ("lamost1550", 1550, 64, 8, {}, 1), ("lamost1550", 1550, 64, 8, THREE, 1),
    ("lamost3900", 2048, 64, 10, {}, 1), ("lamost3900", 2049, 64, 6, {}, 1),
    ("lamost3900", 3900, 64, 10, {}, 1), ("lamost3900", 4225, 64, 10, {}, 1),
    ("desi7800", 7800, 64, 10, None, 1), ("desi7800", 8576, 64, 10, {}, 1),
    ("lamost1550", 1550, 64, 8, {}, 3)]


def problem(name, n_pix, margin, degree, arms, classes, n, cid):
    over = {} if arms is None else {"arm_start": (), "arm_sigma_kms": (), **arms}
    shape = shape_by_name(name, n_pix=n_pix, margin=margin, degree=degree, **over)
    basis, lines = make_basis(shape, n_classes=classes)
    batch = make_spectra(shape, lines, cid, 0, n)
    cfg = oracle.Config.from_shape(shape, BOX_LO, BOX_HI, n_classes=classes)
    u = cfg.normalise(batch.init) + np.random.default_rng(6).normal(0, 0.03, (n, 5))
    a = lasp.Arms(shape.arm_start, shape.arm_sigma_kms) if shape.arm_start else None
    kw = dict(margin=margin, degree=degree, arms=a, n_classes=classes)
    return shape, basis, batch, cfg, u.astype(np.float32), kw


@pytest.mark.parametrize("name,n_pix,margin,degree,arms,classes", CASES)
def test_same_bits_as_the_fused_pass(name, n_pix, margin, degree, arms, classes):
    print(f"[cov one-shot] n_pix={n_pix} degree={degree} classes={classes}", flush=True)
    shape, basis, batch, cfg, u, kw = problem(name, n_pix, margin, degree, arms, classes, 7, 80)
    obs, ivar = batch.obs.copy(), batch.ivar.copy()
    obs[1, n_pix // 2] = np.nan
    ivar[2] = 0.0
    ivar[3, 12:] = 0.0
    obs[4] *= -1.0
    u[5, 1] = 2.0                                # out of the box
    obs[6, 3], ivar[6, 5] = np.inf, -1.0
    args = [torch.from_numpy(x).to(DEV) for x in (obs, ivar)]
    args += [wave_grid(shape)] + [torch.from_numpy(x).to(DEV) for x in (basis, u)]
    ref = lasp.forward(*args, want_grad=True, want_model=True, want_jac=True, want_cov=True, **kw)
    for want in (dict(want_cov=True), dict(want_jac=True), dict(want_cov=True, want_model=True),
                 dict(want_cov=True, want_jac=True, want_model=True)):
        for noalloc in (False, True):
            got = lasp.forward(*args, noalloc=noalloc, **want, **kw)
            torch.cuda.synchronize()
            for k, v in got.items():
                # the covariance adds its own SINGULAR: only where it was asked for
                if v is None or (k == "status" and "want_cov" not in want):
                    continue
                a, b = ref[k].cpu().numpy(), v.cpu().numpy()
                assert np.array_equal(a, b, equal_nan=True), (want, noalloc, k)
    plain = lasp.forward(*args, want_model=True, **kw)      # the fused pass alone
    jac = lasp.forward(*args, want_jac=True, **kw)
    torch.cuda.synchronize()
    for k in ("chi2", "J", "n_eff", "status"):
        a, b = plain[k].cpu().numpy(), jac[k].cpu().numpy()
        assert np.array_equal(a, b, equal_nan=True), k


@pytest.mark.parametrize("name,n_pix,margin,degree,arms,classes", [
    ("lamost1550", 1550, 64, 8, THREE, 1), ("lamost3900", 2049, 64, 6, {}, 1),
    ("desi7800", 7800, 64, 10, None, 1), ("lamost1550", 1550, 64, 8, {}, 3)])
def test_jacobian_without_gradient_matches_the_oracle(name, n_pix, margin, degree, arms, classes):
    print(f"[cov one-shot] Jacobian n_pix={n_pix} classes={classes}", flush=True)
    shape, basis, batch, cfg, u, kw = problem(name, n_pix, margin, degree, arms, classes, 3, 81)
    res = lasp.forward(*(torch.from_numpy(x).to(DEV) for x in (batch.obs, batch.ivar)),
                       wave_grid(shape), *(torch.from_numpy(x).to(DEV) for x in (basis, u)),
                       want_jac=True, want_model=True, **kw)
    torch.cuda.synchronize()
    for i in range(3):
        ref = oracle.evaluate(cfg, batch.obs[i], batch.ivar[i], basis, u[i].astype(np.float64))
        rms = np.sqrt(np.mean(ref["model"] ** 2))
        assert np.max(np.abs(res["model"][i].cpu().numpy() - ref["model"])) <= 1e-5 * rms, i
        for t in range(5):
            j, r = res["jac"][i, t].cpu().numpy(), ref["jac"][t]
            assert np.linalg.norm(j - r) <= 1e-5 * np.linalg.norm(r), (i, t)
