"""The 9x9 Chebyshev step in FP64 and FP32 at every tile width: block rows whose block counts leave
every remainder of the four-block chunks (1 to 19 blocks), probe counts at and beside the edges of
the 16, 32, 64 and 256-column tiles, sign-bit and dense probes, moments (doubled and direct),
density and gradient, against the oracle.

FP64: the parity bar.  FP32: the rounding of one step is at most (9 b + 4) u |H_hat| |y| per element
(b blocks in a row, u = 2^-24, H_hat rounded once), and T_k of a matrix with spectrum in [-1, 1]
carries an error of a step on with a factor of at most k; so a moment of p terms is off by at most
p^2/2 (9 b + 5) u || |H_hat| ||_2 ||r||^2, and a doubled moment by four times that.
"""

import numpy as np
import pytest

from oracle import estimator as est
from tests.gpu_common import banner, check_blocks, check_moments, engine_or_skip, load_hamiltonian
from workloads import cu_cluster, rademacher
from workloads.bsr import BSR

pytestmark = pytest.mark.gpu


def ragged(nb=37, seed=5):
    """Symmetric block pattern whose rows hold 1 to 19 blocks; H inside [-1, 1] by Gershgorin."""
    rng = np.random.default_rng(seed)
    mask = np.eye(nb, dtype=bool)
    for i in range(1, nb):
        for j in rng.choice(i, size=min(i, int(rng.integers(0, 10))), replace=False):
            mask[i, j] = mask[j, i] = True
    mask[0, 1:] = mask[1:, 0] = False
    rows, cols = np.nonzero(mask)
    vals = rng.standard_normal((rows.size, 9, 9))
    where = {(i, j): z for z, (i, j) in enumerate(zip(rows, cols))}
    for z, (i, j) in enumerate(zip(rows, cols)):
        if i == j:
            vals[z] = 0.5 * (vals[z] + vals[z].T)
        elif i > j:
            vals[z] = vals[where[(j, i)]].T
    rad = np.zeros(nb * 9)
    np.add.at(rad.reshape(nb, 9), rows, np.abs(vals).sum(axis=2))
    vals /= 1.01 * rad.max()
    ptr = np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=nb))]).astype(np.int64)
    return BSR(ptr, cols.astype(np.int32), vals, 9, -1.0, 1.0, meta={})


CASES = [(s, ppl) for s in (1, 16, 17, 33, 64, 100, 130) for ppl in (1, 2, 4)] + [(256, -1), (250, -1), (288, -1)]


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("s,ppl", CASES)
def test_step9_tiles(prec, s, ppl):
    banner(f"step9 {prec} s={s} ppl={ppl}")
    H = ragged()
    counts = np.diff(H.row_ptr)
    assert counts.min() == 1 and set(counts % 4) == {0, 1, 2, 3}
    dense = s % 2 == 1
    R = rademacher(H.n, s, config_id=77)
    if dense:
        R = R * (1.0 + 0.25 * np.cos(np.arange(H.n))[:, None])
    T, mu, p = 0.2, 0.1, 24
    eng = engine_or_skip()
    load_hamiltonian(eng, H, precision=prec)
    eng.set_probes(R)
    eng.set_tuning("ppl", ppl)
    o = est.estimate(H, R, T, mu, p, density=True, gradient=True)
    A = np.zeros((H.n, H.n))
    for i in range(counts.size):
        for z in range(H.row_ptr[i], H.row_ptr[i + 1]):
            A[9 * i:9 * i + 9, 9 * H.col_idx[z]:9 * H.col_idx[z] + 9] = H.values[z]
    bound = 4 * 0.5 * p ** 2 * (9 * counts.max() + 5) * 2.0 ** -24 * np.linalg.norm(np.abs(A), 2)
    for doubling in (True, False):
        eng.set_moment_doubling(doubling)
        m = eng.fermi_moments(T, mu, p, moments=True)
        g = eng.energy_and_dEdH(T, mu, p)
        if prec == "fp64":
            check_moments(m["moments"], o["moments"])
            check_blocks(g["dFdH"], o["dFdH"])
        else:
            assert np.max(np.abs(m["moments"] - o["moments"]) / o["moments"][:, :1]) < bound
            assert np.max(np.abs(g["dFdH"] - o["dFdH"])) < bound * np.max(np.abs(o["dFdH"]))
    d = eng.fermi_moments(T, mu, p, moments=True, density=True)
    if prec == "fp64":
        check_moments(d["moments"], o["moments"])
        check_blocks(d["density"], o["density"])
    else:
        assert np.max(np.abs(d["density"] - o["density"])) < bound * np.max(np.abs(o["density"]))
