"""The rule for the continuum moments' nodes, compiled from the library's header
for the host: wherever it says that seven nodes hold the moments' polynomials,
their interpolation on every lane's pixels is within its 1e-7 -- the last lane's
too, whose nodes reach past the row, where the polynomials grow."""

import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
NPL, MID = 17, 8            # pixels per lane, its middle


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("nodes")
    src, lib = d / "nodes.cpp", d / "nodes.so"
    src.write_text('#include "lasp_internal.h"\n'
                   'extern "C" int hold(int nd, int P) { return lasp::moment_nodes_hold(nd, P); }\n'
                   'extern "C" double tau(int c) { return lasp::kMomentNodes.tau[c]; }\n')
    subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__",
                    "-I/opt/rocm/include", f"-I{ROOT}/include",
                    f"-I{ROOT}/paper_2512_24840_amd/csrc", str(src), "-o", str(lib)], check=True)
    lib = ctypes.CDLL(str(lib))
    lib.tau.restype = ctypes.c_double
    return lib


def worst(rule, degree, P):
    """Largest interpolation error of T_0 .. T_2D at any pixel of the row."""
    tau = np.array([s * rule.tau(c) for c in range(3) for s in (1.0, -1.0)] + [0.0])
    t = np.arange(NPL) - MID
    lag = np.array([[np.prod([(ti - b) / (a - b) for b in tau if b != a]) for a in tau]
                    for ti in t.astype(float)])
    h, err = 2.0 / P, 0.0
    coef = np.eye(2 * degree + 1)
    j0 = np.arange(0, P, NPL)[:, None]
    x_node = (j0 + MID + tau[None]) * h - 1.0
    j = j0 + np.arange(NPL)[None]
    x = j * h - 1.0
    for k in range(2 * degree + 1):
        p_node = np.polynomial.chebyshev.chebval(x_node, coef[k])
        p = np.polynomial.chebyshev.chebval(x, coef[k])
        err = max(err, np.abs(np.where(j < P, p - p_node @ lag.T, 0.0)).max())
    return err


@pytest.mark.parametrize("degree", [4, 6, 8, 10])
def test_nodes_hold_where_the_rule_says_so(rule, degree):
    nd = degree + 1
    first = next(P for P in range(32, 2176) if rule.hold(nd, P))
    assert all(rule.hold(nd, P) for P in range(first, 8705))
    assert first <= 2016        # wider workgroups, of longer rows, always take nodes
    # every filling of the last lane
    err = [worst(rule, degree, P) for P in range(first, first + 2 * NPL)]
    assert max(err) <= 1e-7, (first, max(err))
