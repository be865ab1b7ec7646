"""The complex shifted product of 9x9 blocks and the solver's vector kernels: block rows of 1 to 19
blocks, one and two column tiles per wave, one and two tiles of a row per workgroup, with and without
an overlap, few and many rows and probes, against the oracle's sparse-LU solves at the parity bar.
"""

import numpy as np
import pytest

from oracle import rational as ra
from tests.gpu_common import TOL, banner, check_blocks, engine_or_skip
from tests.test_gpu_rational import fit_for, load
from tests.test_gpu_step9 import ragged
from workloads import rademacher
from workloads.bsr import BSR

pytestmark = pytest.mark.gpu

CASES = [(nb, s, ppl, rows) for nb, s in ((1, 3), (37, 5), (37, 130)) for ppl in (1, 2) for rows in (1, 2)]
CASES += [(2, 64, -1, -1), (37, 64, -1, -1), (300, 70, -1, -1), (260, 900, -1, -1)]  # the last: vectors over 16 MiB


@pytest.mark.parametrize("overlap", [False, True])
@pytest.mark.parametrize("nb,s,ppl,rows", CASES)
def test_cplx9(nb, s, ppl, rows, overlap):
    banner(f"cplx9 nb={nb} s={s} tiles={ppl} rows={rows} overlap={overlap}")
    G = ragged(nb)
    H = BSR(G.row_ptr, G.col_idx, G.values, 9, -1.2, 1.2, meta={})
    R = rademacher(H.n, s, config_id=79)
    if s % 2 == 1:
        R = R * (1.0 + 0.25 * np.cos(np.arange(H.n))[:, None])
    T, mu, nodes = 0.3, 0.1, 6
    fit = fit_for(H, nodes, T, mu)
    eng = engine_or_skip()
    eng.set_tuning("cplx_ppl", ppl)
    eng.set_tuning("cplx_rows", rows)
    load(eng, H, R)
    if overlap:
        # S = 1 + H / 20, so the pencil's spectrum is inside [-1 / 0.95, 1 / 0.95]
        vals = 0.05 * H.values
        rowi = np.repeat(np.arange(nb), np.diff(H.row_ptr))
        vals[rowi == H.col_idx] += np.eye(9)
        eng.set_overlap(vals, cg_tol=1e-14)
        g = eng.rational(mu, fit, tol=1e-13, max_iter=20000, density=True)
        o = ra.estimate_overlap(H, vals, R, fit, density=True)
        check_blocks(eng.density_q(), o["density_Q"])
    else:
        g = eng.rational(mu, fit, tol=1e-13, max_iter=20000, density=True, gradient=True)
        o = ra.estimate(H, R, fit, density=True, gradient=True)
        check_blocks(g["dFdH"], o["dFdH"])
    for k in ("N", "E", "F"):
        assert abs(g[k] - o[k]) <= TOL * max(1.0, abs(o[k])), (k, g[k], o[k])
    check_blocks(g["density"], o["density"])
