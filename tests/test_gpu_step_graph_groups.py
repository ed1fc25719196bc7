"""Adam steps from the cached HIP graph, in the groups that take it -- FP32
groups too large for the one-launch fit, and BF16x3 groups -- against the same
steps launched one kernel at a time, bit for bit: chunks with and without a
remainder, replays across calls with other work between them, new arguments and
sizes, a side stream; and against the FP64 oracle."""

import numpy as np
import pytest
import torch

import oracle
import paper_2512_24840_amd as lasp
from synth import BOX_HI, BOX_LO, make_basis, make_spectra, shape_by_name, wave_grid

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("oracle_lib")]
DEV = torch.device("cuda:0")
FIT_TOL = np.array([2.0, 0.005, 0.005, 0.2])
# (pixels, margin, degree, spectra, precision): one more than the one launch
# takes, the largest group of the graph, and BF16x3
GROUPS = [(257, 17, 4, 1025, "fp32"), (257, 17, 4, 4096, "fp32"), (4353, 64, 4, 257, "fp32"),
          (257, 17, 4, 9, "bf16x3"), (1550, 64, 8, 1025, "bf16x3")]


class Problem:
    def __init__(self, n_pix, margin, degree, n_spec, precision):
        self.shape = shape_by_name("lamost1550" if n_pix == 1550 else "lamost3900", n_pix=n_pix,
                                   margin=margin, degree=degree)
        self.basis, lines = make_basis(self.shape)
        self.batch = make_spectra(self.shape, lines, 79, 0, 8)
        idx = np.arange(n_spec) % 8
        init = self.batch.init[idx]
        init[:, 1] += np.linspace(0.0, 0.1, n_spec, dtype=np.float32)
        self.dev = [torch.from_numpy(np.ascontiguousarray(x)).to(DEV)
                    for x in (self.batch.obs[idx], self.batch.ivar[idx], self.basis, init)]
        self.precision = precision

    def fit(self, n_steps, graph, n=None, **kw):
        obs, ivar, basis, init = self.dev
        n = obs.shape[0] if n is None else n
        kw = {"precision": self.precision, "want_cov": True, **kw}
        r = lasp.fit_group(obs[:n], ivar[:n], wave_grid(self.shape), basis, init[:n], n_steps,
                           margin=self.shape.margin, degree=self.shape.degree, step_graph=graph,
                           **kw)
        torch.cuda.current_stream().synchronize()
        return {k: getattr(r, k).cpu().numpy()
                for k in ("params", "status", "chi2", "steps", "cov")}


def same(a, b, tag):
    for k in a:
        assert np.array_equal(a[k], b[k], equal_nan=True), (tag, k)


@pytest.mark.parametrize("group", GROUPS)
def test_replays_equal_single_launches(group):
    print(f"[graph groups] {group}: chunks and remainders", flush=True)
    p = Problem(*group)
    for n_steps in (24, 25, 26, 60):
        same(p.fit(n_steps, True), p.fit(n_steps, False), n_steps)


def test_a_graph_is_kept_and_rebuilt_when_its_arguments_change():
    print("[graph groups] kept across calls; new size, lr, precision; side stream", flush=True)
    p = Problem(*GROUPS[0])
    ref = p.fit(60, False)
    x = torch.ones(1 << 20, device=DEV)
    for rep in range(3):
        same(p.fit(60, True), ref, ("replay", rep))
        x.mul_(1.5).add_(1.0)                   # other work on the same stream
        torch.cuda.synchronize()
    big = Problem(257, 17, 4, 1100, "fp32")
    same(big.fit(50, True), big.fit(50, False), "more spectra")
    same(p.fit(50, True, lr=3e-3), p.fit(50, False, lr=3e-3), "lr")
    same(p.fit(50, True, betas=(0.8, 0.99)), p.fit(50, False, betas=(0.8, 0.99)), "betas")
    same(p.fit(50, True, precision="bf16x3"), p.fit(50, False, precision="bf16x3"), "bf16x3")
    same(p.fit(50, True, n=1024), p.fit(50, False, n=1024), "a size of the one launch between")
    same(p.fit(60, True), ref, "back to the first arguments")
    s = torch.cuda.Stream(device=DEV)
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        same(p.fit(60, True), ref, "side stream")


def test_graph_fits_match_the_oracle():
    print("[graph groups] 500 steps of 1,025 x 1,550 px; oracle LM on 8", flush=True)
    p = Problem(1550, 64, 8, 1025, "fp32")
    got = p.fit(500, True)
    cfg = oracle.Config.from_shape(p.shape, BOX_LO, BOX_HI)
    ref = oracle.fit_many(cfg, p.batch.obs, p.batch.ivar, p.basis, p.batch.init)
    for i in range(0, 1025, 128):
        err = np.abs(got["params"][i].astype(np.float64) - ref[i % 8]["params"])[:4]
        assert np.all(err <= FIT_TOL), (i, err)
