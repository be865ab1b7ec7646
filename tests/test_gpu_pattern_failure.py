"""A pattern whose upload fails for lack of device memory leaves none to keep: the call that asks for the kept
pattern is refused (it would otherwise read values by the new pattern's size, and run on buffers of which some hold the
old pattern and some the new), and the context works again with the next whole one.  Most of the device memory is
held by one allocation meanwhile.
"""

import numpy as np
import pytest

from oracle import estimator as est
from tests.gpu_common import banner, check_moments, engine_or_skip
from tests.test_gpu_run_rule import band
from workloads import rademacher

pytestmark = pytest.mark.gpu


def test_failed_pattern_cannot_be_kept():
    banner("pattern upload without memory")
    import paper_1812_05264_amd as pkg
    import torch
    n = 9700
    A, B = band(n, 5), band(n, 2001)
    R = rademacher(n, 3, config_id=68)
    eng = engine_or_skip()
    eng.set_hamiltonian(A.row_ptr, A.col_idx, A.values, 1, A.e_min, A.e_max, "fp64")
    torch.cuda.synchronize()
    # B's pattern takes 28 bytes an entry (0.54 GB); what the device reports as free leaves some out
    hold = [torch.empty(torch.cuda.mem_get_info()[0] - (400 << 20), dtype=torch.uint8, device="cuda")]
    try:
        for _ in range(64):
            hold.append(torch.empty(128 << 20, dtype=torch.uint8, device="cuda"))
    except torch.OutOfMemoryError:
        pass
    if len(hold) > 64:
        pytest.skip("the device gives more memory than it reports")
    del hold[-1]
    torch.cuda.empty_cache()
    with pytest.raises(pkg.RfoError, match="NOMEM|hipMalloc"):
        eng.set_hamiltonian(B.row_ptr, B.col_idx, B.values, 1, B.e_min, B.e_max, "fp64")
    del hold
    torch.cuda.empty_cache()
    with pytest.raises(pkg.RfoError, match="no previous pattern"):
        eng.set_hamiltonian(None, None, A.values, 1, A.e_min, A.e_max, "fp64")
    eng.set_hamiltonian(A.row_ptr, A.col_idx, A.values, 1, A.e_min, A.e_max, "fp64")
    eng.set_hamiltonian(None, None, A.values, 1, A.e_min, A.e_max, "fp64")
    eng.set_probes(R)
    o = est.estimate(A, R, 0.2, 0.1, 12)
    check_moments(eng.fermi_moments(0.2, 0.1, 12, moments=True)["moments"], o["moments"])
