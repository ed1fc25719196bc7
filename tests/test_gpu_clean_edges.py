"""The Clean mask at the edges of its layout -- the row's ends, the borders of
a lane's 17 pixels and of a wave's 64 lanes, the smallest and largest rows --
and on rows without valid pixels, against the oracle's, bit for bit."""

import numpy as np
import pytest
import torch

import oracle
import paper_2512_24840_amd as lasp

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("oracle_lib")]
DEV = torch.device("cuda:0")


@pytest.mark.parametrize("n_pix,margin", [(32, 1), (1087, 64), (2048, 64), (3900, 64), (4224, 64),
                                          (8576, 64)])
def test_clean_mask_at_layout_edges(n_pix, margin):
    print(f"[clean edges] n_pix={n_pix}", flush=True)
    rng = np.random.default_rng(n_pix)
    model = (100.0 + 10.0 * np.sin(np.arange(n_pix) / 7.0))[None].repeat(6, 0).astype(np.float32)
    obs = model + rng.normal(0, 1.0, model.shape).astype(np.float32)
    ivar = np.ones_like(obs)
    at = np.array([j for j in (0, 16, 17, 33, 1087, 1088, 2175, 2176, n_pix - 2, n_pix - 1)
                   if j < n_pix])
    obs[0, at] += 40.0                          # outliers on the borders
    for k in range(3):                          # same-sign shoulders across them
        obs[1, np.clip(at + k, 0, n_pix - 1)] += 30.0 / (k + 1)
        obs[1, np.clip(at - k, 0, n_pix - 1)] += 30.0 / (k + 1)
    obs[2, at] -= 40.0
    ivar[2, at[::2]] = 0.0
    ivar[3] = 0.0                               # no valid pixel
    ivar[4, 1:] = 0.0                           # one
    obs[5, :: 9] += 25.0                        # over 3 % clipped: the relaxed thresholds
    obs[5, 5], ivar[5, 7], obs[5, 9] = np.nan, np.inf, -np.inf
    grid = 3700.0 * 10.0 ** (1e-4 * np.arange(n_pix))
    dev = [torch.from_numpy(a).to(DEV) for a in (obs, ivar, model)]
    for f_shift in (0.5, 0.2):
        keep, n_masked = lasp.clean_mask(*dev, grid, f_shift, margin=margin)
        torch.cuda.synchronize()
        for i in range(6):
            ref = oracle.clean_mask(obs[i], ivar[i], model[i].astype(np.float64), f_shift)
            got = keep[i].cpu().numpy()
            assert np.array_equal(got, ref["keep"]), (i, f_shift, np.where(got != ref["keep"]))
            assert int(n_masked[i]) == ref["masked"], (i, f_shift)
