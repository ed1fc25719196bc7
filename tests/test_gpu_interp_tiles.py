"""The forward contraction takes several 16-row tiles per workgroup in large
groups: an evaluation in a group at the edges of that rule has the bits of the
same spectra evaluated in groups of one tile each, with and without derivative
rows, in FP32 and BF16x3."""

import numpy as np
import pytest
import torch

import paper_2512_24840_amd as lasp
from synth import make_basis, make_spectra, shape_by_name, wave_grid

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


# 1,024 workgroups make a round: with one column block (n_pix + 2 margin <= 512)
# tiles are grouped from 2,049 tiles on (32,769 rows), with two from 16,385
@pytest.mark.parametrize("precision", ["fp32", "bf16x3"])
@pytest.mark.parametrize("n_pix,n_spec", [(257, 32768), (257, 32769), (257, 49153), (700, 16384),
                                          (700, 16385), (700, 24600), (700, 66001)])
def test_tiles_of_a_workgroup_equal_single_tiles(n_pix, n_spec, precision):
    print(f"[interp tiles] n_pix={n_pix} B={n_spec} {precision}", flush=True)
    shape = shape_by_name("lamost3900", n_pix=n_pix, margin=17, degree=4)
    basis, lines = make_basis(shape)
    batch = make_spectra(shape, lines, 73, 0, 7)
    grid = wave_grid(shape)
    kw = dict(margin=17, degree=4, precision=precision)
    bas = torch.from_numpy(basis).to(DEV)
    idx = torch.arange(n_spec, device=DEV) % 7
    obs = torch.from_numpy(batch.obs).to(DEV)[idx].contiguous()
    ivar = torch.from_numpy(batch.ivar).to(DEV)[idx].contiguous()
    rng = np.random.default_rng(5)
    u = torch.from_numpy(rng.uniform(-0.9, 0.9, (n_spec, 5)).astype(np.float32)).to(DEV)
    for cov in (False, True):
        out = "want_cov" if cov else "want_grad"
        n = n_spec // 4 if cov else n_spec          # four rows per spectrum with derivatives
        big = lasp.forward(obs[:n], ivar[:n], grid, bas, u[:n], **{out: True}, **kw)
        pick = [0, 15, 16, n // 2 - 3, n - 17, n - 16, n - 1]
        for lo in sorted({max(0, min(p, n - 8)) for p in pick}):
            sl = slice(lo, lo + 8)
            one = lasp.forward(obs[sl], ivar[sl], grid, bas, u[sl], **{out: True}, **kw)
            torch.cuda.synchronize()
            for k in one:
                if one[k] is not None:
                    a, b = big[k][sl].cpu().numpy(), one[k].cpu().numpy()
                    assert np.array_equal(a, b, equal_nan=True), (k, lo)
