"""A last probe tile of 128 columns with at most 64 real ones as a batch of its own, at sizes that take it: 9x9
FP64 vectors of 128 MiB and more (7,300 block rows, 256 padded columns), and 1x1 matrices too large for the one
launch of all steps.  Moments, density and gradient, doubled and direct, sign-bit and dense probes with unequal weights,
against the oracle at the parity bar; the step count of each call shows that it ran as two batches, and the
moments are bitwise those of a call on each column range.  Smaller 9x9 vectors, and FP32 ones with density or gradient,
run whole.
"""

import numpy as np
import pytest

from oracle import estimator as est
from tests.gpu_common import banner, check_blocks, check_moments, engine_or_skip, load_hamiltonian
from workloads import cu_cluster, rademacher, simple_cubic

pytestmark = pytest.mark.gpu

T, MU, P = 0.3, 0.2, 5   # 2 and 4 steps: the sweep alternates, and an even count leaves it forward for the next batch
MODELS = {"cu7300": lambda: cu_cluster(7300, config_id=54).bsr(),
          "sc22": lambda: simple_cubic(22, disorder=0.5, config_id=54)}


def steps_of(eng, call):
    eng.set_timing(True)
    out = call()
    n = eng.step_timing()[1]
    eng.set_timing(False)
    return out, n


@pytest.mark.timeout(300)
@pytest.mark.parametrize("model,dense,s", [("cu7300", False, 160), ("cu7300", True, 150), ("sc22", False, 190),
                                           ("sc22", True, 129)])
def test_last_tile_batch(model, dense, s):
    banner(f"last-tile batch {model} s={s} dense={dense}")
    H = MODELS[model]()
    R = rademacher(H.n, s, config_id=904)
    if dense:
        R = R * (1.0 + 0.25 * np.cos(np.arange(H.n))[:, None])
    w = np.linspace(0.5, 1.5, s) / s
    o = est.estimate(H, R, T, MU, P, weights=w, density=True, gradient=True)
    eng = engine_or_skip()
    load_hamiltonian(eng, H)
    for doubling in (True, False):
        eng.set_moment_doubling(doubling)
        calls = {"moments": lambda: eng.fermi_moments(T, MU, P, moments=True),
                 "density": lambda: eng.fermi_moments(T, MU, P, moments=True, density=True),
                 "gradient": lambda: eng.energy_and_dEdH(T, MU, P)}
        part = {}
        for lo, hi in ((0, 128), (128, s)):
            eng.set_probes(R[:, lo:hi], w[lo:hi])
            part[lo] = {k: steps_of(eng, f) for k, f in calls.items()}
        eng.set_probes(R, w)
        for name, call in calls.items():
            g, n = steps_of(eng, call)
            t = eng.traces_at(T, MU)
            assert n == part[0][name][1] + part[128][name][1] == 2 * part[0][name][1], name
            for k in ("N", "E", "F"):
                assert abs(g[k] - o[k]) <= 1e-10 * max(1.0, abs(o[k])), (name, k)
                assert abs(t[k] - g[k]) <= 1e-13 * max(1.0, abs(g[k])), (name, k)
            if name != "gradient":
                check_moments(g["moments"], o["moments"], what=name)
                ranges = np.concatenate([part[lo][name][0]["moments"] for lo in (0, 128)])
                assert np.array_equal(g["moments"], ranges), name
            if name == "density":
                check_blocks(g["density"], o["density"], what=name)
            if name == "gradient":
                check_blocks(g["dFdH"], o["dFdH"], what=name)


@pytest.mark.parametrize("prec,atoms,calls", [("fp64", 1000, ("moments", "density", "gradient")),
                                              ("fp32", 1000, ("moments", "density", "gradient")),
                                              ("fp32", 14600, ("density", "gradient"))])
def test_runs_whole(prec, atoms, calls):
    banner(f"whole last tile {prec} atoms={atoms}")
    H = cu_cluster(atoms, config_id=55).bsr()
    R = rademacher(H.n, 150, config_id=905)
    eng = engine_or_skip()
    load_hamiltonian(eng, H, precision=prec)
    run = {"moments": lambda: eng.fermi_moments(T, MU, P, moments=True),
           "density": lambda: eng.fermi_moments(T, MU, P, moments=False, density=True),
           "gradient": lambda: eng.energy_and_dEdH(T, MU, P)}
    eng.set_probes(R[:, :64])
    one = {k: steps_of(eng, run[k])[1] for k in calls}
    eng.set_probes(R)
    assert {k: steps_of(eng, run[k])[1] for k in calls} == one
