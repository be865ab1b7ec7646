"""The step kernel of 1x1 blocks on matrices that would otherwise run all their steps in one launch: setting
a key of its geometry selects it.  Lattices (rows of 7 entries) and graphs (uneven rows) in FP64 and FP32 at
probe counts of one, two and four probes per lane, with and without padding columns; every ending of the
three-term density accumulator; the geometry keys themselves, against the oracle.

Bounds as in the tests of the one-launch kernel, with b entries in a row: a moment of p terms is off by at most
4 p^2/2 (b + 5) u || |H_hat| ||_inf ||r||^2, and so is the density, in units of its largest entry.  FP64 moments:
the parity bar.
"""

import numpy as np
import pytest

from oracle import estimator as est
from tests.gpu_common import banner, check_moments, engine_or_skip
from workloads import rademacher, random_graph, simple_cubic

pytestmark = pytest.mark.gpu

T, MU = 0.2, 0.1


def problem(model, n, s, dense):
    H = simple_cubic(n, disorder=0.5, config_id=63) if model == "lattice" else random_graph(n, config_id=63)
    R = rademacher(H.n, s, config_id=64)
    if dense:
        R = R * (1.0 + 0.25 * np.cos(np.arange(H.n))[:, None])
    diag = H.block_rows() == H.col_idx
    hat = (2.0 * H.values.reshape(-1) - (H.e_max + H.e_min) * diag) / (H.e_max - H.e_min)
    norm = max(1.0, np.max(np.add.reduceat(np.abs(hat), H.row_ptr[:-1])))
    return H, R, (np.diff(H.row_ptr).max() + 5) * norm


def engine(H, R, prec):
    eng = engine_or_skip()
    eng.set_hamiltonian(H.row_ptr, H.col_idx, H.values, 1, H.e_min, H.e_max, prec)
    eng.set_probes(R)
    return eng


def compare(eng, o, p, prec, scale):
    bound = 2.0 * p ** 2 * scale * 2.0 ** (-53 if prec == "fp64" else -24)
    for doubling in (True, False):
        eng.set_moment_doubling(doubling)
        for density in (False, True):
            g = eng.fermi_moments(T, MU, p, moments=True, density=density)
            if prec == "fp64":
                check_moments(g["moments"], o["moments"])
            else:
                assert np.max(np.abs(g["moments"] - o["moments"]) / o["moments"][:, :1]) < bound
            if density:
                assert np.max(np.abs(g["density"] - o["density"])) < bound * np.max(np.abs(o["density"]))


CASES = [("lattice", 8, s, 40) for s in (1, 64, 100, 200, 256)] + [("graph", 700, s, 30) for s in (3, 130, 256)]
CASES += [("lattice", 5, 6, p) for p in (1, 2, 3, 4, 5, 6, 7, 8)]


@pytest.mark.parametrize("dense", [False, True])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("model,n,s,p", CASES)
def test_step1_forward(model, n, s, p, prec, dense):
    banner(f"step1 {model} n={n} s={s} p={p} {prec} dense={dense}")
    H, R, scale = problem(model, n, s, dense)
    eng = engine(H, R, prec)
    o = est.estimate(H, R, T, MU, p, density=True)
    eng.set_tuning("alt_sweep", 1)
    compare(eng, o, p, prec, scale)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("key,values", [("ppl", (1, 2, 4)), ("rpi", (1, 2, 7)), ("rows_per_wg", (4, 96)),
                                        ("grid", (8, 64)), ("alt_sweep", (0, 1))])
def test_step1_geometry_keys(key, values, prec):
    """A set key selects the step kernel with that geometry: two geometries add the moments in different orders
    (ppl and rpi may not), each call is bitwise repeatable, and -1 restores the default call."""
    banner(f"step1 keys {key} {prec}")
    H, R, scale = problem("lattice", 10, 256, False)
    eng = engine(H, R, prec)
    p = 60
    o = est.estimate(H, R, T, MU, p, density=True)
    default = eng.fermi_moments(T, MU, p, moments=True)["moments"]
    seen = []
    for v in values:
        eng.set_tuning(key, v)
        compare(eng, o, p, prec, scale)
        eng.set_moment_doubling(True)
        m = eng.fermi_moments(T, MU, p, moments=True)["moments"]
        assert np.array_equal(m, eng.fermi_moments(T, MU, p, moments=True)["moments"])
        assert not np.array_equal(m, default)
        seen.append(m)
    if key in ("rows_per_wg", "grid"):
        assert not np.array_equal(seen[0], seen[1])
    eng.set_tuning(key, -1)
    assert np.array_equal(default, eng.fermi_moments(T, MU, p, moments=True)["moments"])
