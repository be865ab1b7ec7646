"""BF16 gradients from one build to the next: the reverse recurrence rounds its vectors to BF16 in every
step, so a last bit in the Chebyshev coefficients of its sources moves the forces by the path's whole
rounding error (1e-4 to 1e-3).  Recorded forces hold the coefficients' order of sums in place.

Bounds: with 64 probes nothing else has another order, so only the FP64 sums over the steps may move
(1e-12).  With 128 probes the FP32 sums of a contraction over the probes may be ordered differently: two
orders of K = 128 products are at most 2 K 2^-24 = 1.5e-5 apart, normwise.
"""

import json
import os

import numpy as np
import pytest

from tests.gpu_common import banner, engine_or_skip, load_hamiltonian, rel
from workloads import cu_cluster, rademacher

pytestmark = pytest.mark.gpu

GOLDEN = os.path.join(os.path.dirname(__file__), "golden", "bf16_forces.json")


@pytest.mark.parametrize("prec", ["bf16", "bf16x2"])
@pytest.mark.parametrize("s,bound", [(64, 1e-12), (128, 2 * 128 * 2.0 ** -24)])
def test_bf16_forces_are_the_recorded_ones(s, bound, prec):
    banner(f"recorded bf16 forces {prec} s={s}")
    with open(GOLDEN) as f:
        want = json.load(f)[f"{prec}_55_{s}_256"]
    cl = cu_cluster(55, config_id=71)
    H = cl.bsr()
    eng = engine_or_skip()
    load_hamiltonian(eng, H, precision=prec)
    eng.set_probes(rademacher(H.n, s, config_id=72))
    g = eng.energy_and_dEdH(0.2, 0.3, 256)
    assert abs(g["F"] - want["F"]) <= 1e-13 * abs(want["F"])
    e = rel(eng.hf_forces(cl.dH_dR()), np.array(want["forces"]))
    print(f"forces against the recorded ones: {e:.2e}")
    assert e <= bound
