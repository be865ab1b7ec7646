"""Coefficients and traces at the edges of their kernels: term counts beside groups of four k of one
parity, beside the table sizes held in LDS (2,048 and 8,192 terms) and past them, probe counts beside 64
columns; N, E, F from the stored moments against the oracle's coefficients.

A coefficient is a mean of nq = 4 p samples h: its error is at most nq u max|h|, and the traces weigh
it with sum_c w_c mu_kc.
"""

import numpy as np
import pytest

from oracle.fermi import fermi_coefficient_sets
from tests.gpu_common import banner, engine_or_skip
from workloads import rademacher, simple_cubic

pytestmark = pytest.mark.gpu

CASES = [(p, 3) for p in (1, 2, 3, 4, 7, 8, 9, 255, 1024, 2047, 2048, 2049, 8191, 8192, 8193)]
CASES += [(100, 64), (1000, 65), (257, 200)]


@pytest.mark.parametrize("p,s", CASES)
def test_traces(p, s):
    banner(f"traces p={p} s={s}")
    H = simple_cubic(3, disorder=0.5, config_id=31)
    R = rademacher(H.n, s, config_id=32)
    w = np.linspace(0.5, 1.5, s) / s
    eng = engine_or_skip()
    eng.set_hamiltonian(H.row_ptr, H.col_idx, H.values, H.block_dim, H.e_min, H.e_max, "fp64")
    eng.set_probes(R, w)
    mom = np.asarray(eng.fermi_moments(0.3, 0.2, p, moments=True)["moments"])
    wm = w @ mom
    for T, mu in ((0.3, 0.2), (0.05, -0.4)):
        got = eng.traces_at(T, mu)
        cf = fermi_coefficient_sets(H.e_min, H.e_max, T, mu, p)
        edge = max(abs(H.e_min), abs(H.e_max))
        top = {"N": 2.0, "E": 2.0 * edge, "F": 2.0 * (edge + abs(mu)) + 2.0 * T}
        for i, key in enumerate(("N", "E", "F")):
            bound = 4 * p * 2.0 ** -52 * top[key] * np.sum(np.abs(wm)) + 1e-14
            assert abs(got[key] - np.dot(cf[i], wm)) <= bound, (key, got[key], np.dot(cf[i], wm), bound)
