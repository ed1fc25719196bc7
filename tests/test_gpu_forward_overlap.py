"""Outputs of a forward evaluation in the memory of its inputs, or of one
another: the call reads every input before it writes there, so each output has
the bits of the same call with memory of its own for all of them."""

import ctypes

import numpy as np
import pytest
import torch

import paper_2512_24840_amd as lasp
from paper_2512_24840_amd.lasp import make_opts
from synth import BOX_HI, BOX_LO, make_basis, make_spectra, shape_by_name, wave_grid

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")
OUTS = dict(model=("P", torch.float32), chi2=(1, torch.float64), J=(1, torch.float32),
            n_eff=(1, torch.int32), grad=(5, torch.float32), jac=("5P", torch.float32),
            cov=(25, torch.float64), status=(1, torch.int32))


def elements(name, B, P):
    n = OUTS[name][0]
    return B * {"P": P, "5P": 5 * P}.get(n, n)


# which output lies where: (output, place, byte offset in it); a place is an
# input or another output
LAYOUTS = [
    ("model in obs", [("model", "obs", 0)], ("model", "grad")),
    ("model one pixel into ivar", [("model", "ivar+", 4)], ("model",)),
    ("jac over obs and ivar", [("jac", "obs+", 0)], ("model", "jac")),
    ("small ones in obs", [("chi2", "obs", 0), ("J", "obs", 8), ("n_eff", "obs", 12),
                           ("status", "obs", 16)], ("grad",)),
    ("small ones in ivar, covariance", [("chi2", "ivar", 0), ("status", "ivar", 8),
                                        ("n_eff", "ivar", 12)], ("cov", "grad")),
    ("cov in obs", [("cov", "obs", 0)], ("cov", "jac", "model")),
    ("n_eff and status in one place", [("status", "n_eff", 0)], ("cov", "grad")),
    ("all over u and obs", [("grad", "u", 0), ("model", "obs", 0)], ("model", "grad", "cov")),
]


@pytest.mark.parametrize("noalloc", [False, True])
@pytest.mark.parametrize("tag,places,want", LAYOUTS, ids=[x[0] for x in LAYOUTS])
def test_outputs_in_the_place_of_inputs(tag, places, want, noalloc):
    print(f"[overlap] {tag} noalloc={noalloc}", flush=True)
    # more workgroups than are resident at once (16 of 128 threads on each of 256
    # CUs), or what one array of the call without allocation holds
    B, n_pix, margin, degree = (900, 600, 17, 4) if noalloc else (6000, 600, 17, 4)
    shape = shape_by_name("lamost3900", n_pix=n_pix, margin=margin, degree=degree)
    basis, lines = make_basis(shape)
    batch = make_spectra(shape, lines, 75, 0, 6)
    idx = np.arange(B) % 6
    th = batch.init.astype(np.float64)
    th[:, 0] = np.log10(th[:, 0])
    u0 = (2.0 * (th - BOX_LO) / (BOX_HI - BOX_LO) - 1.0)[idx]
    u0 += np.random.default_rng(8).normal(0, 0.03, u0.shape)
    bas = torch.from_numpy(basis).to(DEV)
    grid = np.ascontiguousarray(wave_grid(shape))
    lib = lasp.load()
    names = {"chi2", "J", "n_eff", "status", *want}

    def run(put):
        # obs, ivar and u at the front of blocks with room for any output
        room = 5 * B * n_pix + 64
        blk = {k: torch.zeros(room, dtype=torch.float32, device=DEV) for k in ("obs", "ivar", "u")}
        for k, a in (("obs", batch.obs[idx]), ("ivar", batch.ivar[idx]),
                     ("u", u0.astype(np.float32))):
            blk[k][:a.size] = torch.from_numpy(np.ascontiguousarray(a).ravel()).to(DEV)
        own = {k: torch.zeros(elements(k, B, n_pix), dtype=OUTS[k][1], device=DEV) for k in names}
        at = {k: t.data_ptr() for k, t in {**own, **blk}.items()}
        byte_at = {}
        for out, place, off in put:
            # small outputs side by side in one input: each on its own stretch
            start = off * B if place in ("obs", "ivar") else off
            byte_at[out] = (place.rstrip("+"), start)
            at[out] = at[place.rstrip("+")] + start
        o = make_opts(B, n_pix, margin=margin, degree=degree)
        o.status = ctypes.c_void_p(at["status"])
        p = {k: (ctypes.c_void_p(at[k]) if k in at else None) for k in (*OUTS, "obs", "ivar", "u")}
        fn = lib.lasp_forward_noalloc if noalloc else lib.lasp_forward
        rc = fn(p["obs"], p["ivar"], grid.ctypes.data_as(ctypes.c_void_p),
                ctypes.c_void_p(bas.data_ptr()), p["u"], p["model"], p["chi2"], p["J"],
                p["n_eff"], p["grad"], p["jac"], p["cov"], ctypes.byref(o))
        assert rc == 0, lib.lasp_last_error()
        torch.cuda.synchronize()
        res = {}
        for k in names:
            n, dt = elements(k, B, n_pix), OUTS[k][1]
            if k not in byte_at:
                res[k] = own[k].cpu().numpy()
                continue
            where, start = byte_at[k]
            raw = (blk.get(where) if where in blk else own[where]).view(torch.uint8)
            size = n * torch.empty(0, dtype=dt).element_size()
            res[k] = raw[start:start + size].clone().view(dt).cpu().numpy()
        return res

    ref, got = run([]), run(places)
    for k in names:
        if (k, "n_eff", 0) in places or any(p[1] == k for p in places):
            continue                    # two outputs in one place: either may stand
        assert np.array_equal(ref[k], got[k], equal_nan=True), (k, int(np.sum(ref[k] != got[k])))
