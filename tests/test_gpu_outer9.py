"""Masked outer products of 9x9 block vectors (density and segment gradient) in FP64 and FP32: block
rows of 1 to 19 blocks (groups of 1 to 6), probe counts beside the 64 (step, probe) pairs of an item
so that its lanes reach over several steps, segments cut at every step count, sign-bit and dense
probes, fewer groups than compute units (eight waves each) and more (four waves).

Sums are FP64 in both types.  FP64: the parity bar.  FP32 vectors: the bound of the step's tests.
"""

import numpy as np
import pytest

from oracle import estimator as est
from tests.gpu_common import banner, check_blocks, engine_or_skip, load_hamiltonian
from tests.test_gpu_step9 import ragged
from workloads import rademacher

pytestmark = pytest.mark.gpu

CASES = [("fp64", 37, s, k) for s in (1, 5, 63, 64, 65, 100, 130) for k in (1, 3, 32)]
CASES += [("fp32", 37, s, 32) for s in (1, 21, 64, 129)] + [("fp64", 1100, 9, 32)]


@pytest.mark.parametrize("prec,nb,s,steps", CASES)
def test_outer9(prec, nb, s, steps):
    banner(f"outer9 {prec} nb={nb} s={s} steps={steps}")
    H = ragged(nb)
    R = rademacher(H.n, s, config_id=78)
    if s % 2 == 1:
        R = R * (1.0 + 0.25 * np.cos(np.arange(H.n))[:, None])
    T, mu, p = 0.2, 0.1, 24
    eng = engine_or_skip()
    load_hamiltonian(eng, H, precision=prec)
    eng.set_probes(R)
    eng.set_tuning("sddmm_steps", steps)
    o = est.estimate(H, R, T, mu, p, density=True, gradient=True)
    g = eng.energy_and_dEdH(T, mu, p)["dFdH"]
    d = eng.fermi_moments(T, mu, p, density=True)["density"]
    if prec == "fp64":
        check_blocks(g, o["dFdH"])
        check_blocks(d, o["density"])
        return
    counts = np.diff(H.row_ptr)
    A = np.zeros((H.n, H.n))
    for i in range(counts.size):
        for z in range(H.row_ptr[i], H.row_ptr[i + 1]):
            A[9 * i:9 * i + 9, 9 * H.col_idx[z]:9 * H.col_idx[z] + 9] = H.values[z]
    bound = 4 * 0.5 * p ** 2 * (9 * counts.max() + 5) * 2.0 ** -24 * np.linalg.norm(np.abs(A), 2)
    assert np.max(np.abs(g - o["dFdH"])) < bound * np.max(np.abs(o["dFdH"]))
    assert np.max(np.abs(d - o["density"])) < bound * np.max(np.abs(o["density"]))
