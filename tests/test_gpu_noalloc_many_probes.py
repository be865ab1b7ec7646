"""The allocation-free moment call with many probes on few block rows, where the partials of 32 moments alone nearly
fill its work memory, and with so many terms that the moments and the coefficient tables do: the call is taken,
and its moments are bitwise those of rfo_fermi_moments.
"""

import numpy as np
import pytest

from oracle import estimator as est
from tests.gpu_common import banner, check_moments, engine_or_skip, load_hamiltonian
from workloads import cu_cluster, rademacher, simple_cubic

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,atoms,s,p", [("fp64", 55, 1024, 1000), ("fp32", 55, 1024, 1001), ("fp64", 13, 2048, 700)])
@pytest.mark.parametrize("doubling", [True, False])
def test_noalloc_many_probes(prec, atoms, s, p, doubling):
    banner(f"noalloc many probes {prec} atoms={atoms} s={s} doubling={doubling}")
    H = cu_cluster(atoms, config_id=57).bsr()
    R = rademacher(H.n, s, config_id=907)
    eng = engine_or_skip()
    load_hamiltonian(eng, H, precision=prec)
    eng.set_probes(R)
    eng.set_moment_doubling(doubling)
    a = eng.fermi_moments(0.2, 0.1, p, moments=True)
    b = eng.fermi_moments_noalloc(0.2, 0.1, p, moments=True)
    assert np.array_equal(a["moments"], b["moments"])
    assert all(a[k] == b[k] for k in ("N", "E", "F"))
    if prec == "fp64":
        o = est.estimate(H, R[:, ::64], 0.2, 0.1, p)
        check_moments(b["moments"][::64], o["moments"])


def test_noalloc_many_terms():
    """190,000 terms of one probe (64 columns): 672 bytes a term, 128 of them a full turn of the cosine table if it were
    kept, and then too many."""
    banner("noalloc many terms")
    H = simple_cubic(3, disorder=0.5, config_id=58)
    eng = engine_or_skip()
    load_hamiltonian(eng, H)
    eng.set_probes(rademacher(H.n, 1, config_id=908))
    a = eng.fermi_moments(0.2, 0.1, 190000, moments=True)
    b = eng.fermi_moments_noalloc(0.2, 0.1, 190000, moments=True)
    assert np.array_equal(a["moments"], b["moments"])
    assert all(a[k] == b[k] for k in ("N", "E", "F"))
