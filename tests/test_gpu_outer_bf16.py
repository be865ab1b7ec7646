"""The BF16 segment gradient on the matrix cores at the edges of its probe chunks: one probe, 64 padded
columns (its own kernel), whole and partly masked chunks of 128, an odd last probe, against the
vector-unit contraction of the FP32 vectors of the same steps.  One rounding of either operand to BF16 is
at most 2^-8 relative, so a term of the gradient differs by at most 2^-7, and their sum normwise by
no more than the existing bound of 1e-2.
"""

import numpy as np
import pytest

from tests.gpu_common import banner, engine_or_skip, load_hamiltonian, rel
from workloads import cu_cluster, rademacher

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("s", [1, 63, 65, 127, 128, 129, 250, 385])
def test_outer_bf16(s):
    banner(f"outer bf16 s={s}")
    H = cu_cluster(79, config_id=28).bsr()
    eng = engine_or_skip()
    load_hamiltonian(eng, H, precision="bf16")
    eng.set_probes(rademacher(H.n, s, config_id=604))
    g = eng.energy_and_dEdH(0.3, 0.4, 50)
    eng.set_tuning("sddmm_mfma", 0)
    v = eng.energy_and_dEdH(0.3, 0.4, 50)
    assert g["F"] == v["F"]
    assert np.all(np.isfinite(g["dFdH"]))
    assert rel(g["dFdH"], v["dFdH"]) < 1e-2
