"""Small matrices of 1x1 blocks, all steps in one launch: row counts beside the slices of 64 and the
workgroup's 16 waves, rows short enough for the registers and not, both precisions, sign-bit and dense
probes, moments (doubled and direct) and density, against the oracle.  Graphs of 9,600 rows and more have
so many entries that they take a launch per step; test_gpu_run_rule.py has the largest matrices that run in one
and the first whose vectors do not fit.

Bounds as in the tests of the 9x9 step, with b entries in a row: a moment of p terms is off by at most
4 p^2/2 (b + 5) u || |H_hat| ||_inf ||r||^2, and so is the density, in units of its largest entry (an
entry of few probes may cancel to any size, so none is measured by itself).  FP64 moments: the
parity bar.
"""

import numpy as np
import pytest

from oracle import estimator as est
from tests.gpu_common import banner, check_moments, engine_or_skip
from workloads import rademacher, random_graph, simple_cubic

pytestmark = pytest.mark.gpu

CASES = [("graph", n, s, 24) for n, s in ((5, 3), (63, 4), (64, 65), (65, 130), (1000, 7), (1025, 64), (2100, 20))]
CASES += [("lattice", n, s, 40) for n, s in ((3, 1), (8, 64), (11, 33), (14, 10), (17, 6))]
CASES += [("thin", n, 5, 30) for n in (1000, 1500)]  # rows of 9 to 16 entries
CASES += [("graph", n, 2, 9) for n in (9600, 9601, 19200, 19201)] + [("graph", 300, 5, p) for p in (1, 2, 3, 17, 33)]


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("dense", [False, True])
@pytest.mark.parametrize("model,n,s,p", CASES)
def test_run1(model, n, s, p, dense, prec):
    banner(f"run1 {model} n={n} s={s} p={p} dense={dense} {prec}")
    extra = 3 if model == "thin" else min(12, n // 2)
    H = simple_cubic(n, disorder=0.5, config_id=61) if model == "lattice" else random_graph(n, config_id=61, max_extra=extra)
    R = rademacher(H.n, s, config_id=62)
    if dense:
        R = R * (1.0 + 0.25 * np.cos(np.arange(H.n))[:, None])
    T, mu = 0.2, 0.1
    eng = engine_or_skip()
    eng.set_hamiltonian(H.row_ptr, H.col_idx, H.values, 1, H.e_min, H.e_max, prec)
    eng.set_probes(R)
    o = est.estimate(H, R, T, mu, p, density=True)
    counts = np.diff(H.row_ptr)
    diag = H.block_rows() == H.col_idx
    hat = (2.0 * H.values.reshape(-1) - (H.e_max + H.e_min) * diag) / (H.e_max - H.e_min)
    norm = np.max(np.add.reduceat(np.abs(hat), H.row_ptr[:-1]))
    bound = 4 * 0.5 * p ** 2 * (counts.max() + 5) * 2.0 ** (-53 if prec == "fp64" else -24) * max(norm, 1.0)
    for doubling in (True, False):
        eng.set_moment_doubling(doubling)
        m = eng.fermi_moments(T, mu, p, moments=True)["moments"]
        d = eng.fermi_moments(T, mu, p, moments=True, density=True)
        if prec == "fp64":
            check_moments(m, o["moments"])
            check_moments(d["moments"], o["moments"])
        else:
            assert np.max(np.abs(m - o["moments"]) / o["moments"][:, :1]) < bound
            assert np.max(np.abs(d["moments"] - o["moments"]) / o["moments"][:, :1]) < bound
        assert np.max(np.abs(d["density"] - o["density"])) < bound * np.max(np.abs(o["density"]))
