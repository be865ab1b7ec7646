"""Which 1x1 matrices run all their steps in one launch: those whose step is cheaper streamed by one workgroup per
probe column than spread over the chip.  Bands of 7 to 129 entries a row around the lines of the rule; a call
takes a launch per step exactly where it agrees bitwise with the same call with a step-kernel key set (the two
add a column's moments in different orders).  Results against the oracle, also for the long rows on the one-launch
path (bounds as in its own tests).
"""

import numpy as np
import pytest

from oracle import estimator as est
from tests.gpu_common import banner, check_moments, engine_or_skip
from workloads import BSR, rademacher

pytestmark = pytest.mark.gpu

T, MU, P = 0.2, 0.1, 24


def band(n, entries, seed=5):
    """Symmetric band of `entries` (odd) neighbouring columns, open ends."""
    rng = np.random.default_rng(seed)
    half = entries // 2
    upper = rng.uniform(-1.0, 1.0, (n, half + 1))          # (i, i + k), k = 0 .. half
    i = np.repeat(np.arange(n), entries)
    j = i + np.tile(np.arange(-half, half + 1), n)
    keep = (j >= 0) & (j < n)
    i, j = i[keep], j[keep]
    v = upper[np.minimum(i, j), np.abs(i - j)]
    ptr = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(np.bincount(i, minlength=n), out=ptr[1:])
    r = 1.01 * np.max(np.add.reduceat(np.abs(v), ptr[:-1]))
    return BSR(ptr, j.astype(np.int32), v.reshape(-1, 1, 1), 1, -r, r)


CASES = [(9600, 129, 4, "fp64", "steps"), (9600, 129, 64, "fp64", "steps"), (5000, 129, 1, "fp32", "steps"),
         (9600, 33, 128, "fp32", "steps"), (9600, 17, 64, "fp64", "steps"), (9600, 17, 256, "fp64", "one"),
         (9600, 7, 64, "fp64", "one"), (2000, 63, 64, "fp64", "one"), (1000, 129, 3, "fp32", "one"),
         (13000, 3, 130, "fp32", "one"), (19200, 9, 20, "fp32", "steps"), (3000, 7, 300, "fp32", "one")]


@pytest.mark.parametrize("n,entries,s,prec,path", CASES)
def test_path_by_cost(n, entries, s, prec, path):
    banner(f"run rule n={n} entries={entries} s={s} {prec}")
    H = band(n, entries)
    R = rademacher(n, s, config_id=65)
    eng = engine_or_skip()
    eng.set_hamiltonian(H.row_ptr, H.col_idx, H.values, 1, H.e_min, H.e_max, prec)
    eng.set_probes(R)
    o = est.estimate(H, R, T, MU, P, density=True)
    bound = 2.0 * P ** 2 * (entries + 5) * 2.0 ** (-53 if prec == "fp64" else -24)  # || |H_hat| ||_inf < 1
    for density in (False, True):
        eng.set_tuning("alt_sweep", -1)
        g = eng.fermi_moments(T, MU, P, moments=True, density=density)
        eng.set_tuning("alt_sweep", 1)
        b = eng.fermi_moments(T, MU, P, moments=True, density=density)
        for m in (g, b):
            if prec == "fp64":
                check_moments(m["moments"], o["moments"])
            else:
                assert np.max(np.abs(m["moments"] - o["moments"]) / o["moments"][:, :1]) < bound
            if density:
                assert np.max(np.abs(m["density"] - o["density"])) < bound * np.max(np.abs(o["density"]))
        if not (density and prec == "fp32"):  # FP64 sums of +-FP32 values: exact in either order
            assert np.array_equal(g["moments"], b["moments"]) == (path == "steps")


@pytest.mark.parametrize("dense", [False, True])
@pytest.mark.parametrize("n,prec,path", [(9600, "fp64", "one"), (9601, "fp64", "steps"), (19200, "fp32", "one"),
                                         (19201, "fp32", "steps")])
@pytest.mark.parametrize("s", [2, 130])
def test_largest_that_fit(s, n, prec, path, dense):
    """The most rows whose vectors fit the LDS (up to 19 slices of 64 rows a wave, none of them in registers) and
    one more: moments doubled and direct, density."""
    banner(f"largest one-launch n={n} s={s} {prec} dense={dense}")
    H = band(n, 3)
    R = rademacher(n, s, config_id=66)
    if dense:
        R = R * (1.0 + 0.25 * np.cos(np.arange(n))[:, None])
    p = 9
    eng = engine_or_skip()
    eng.set_hamiltonian(H.row_ptr, H.col_idx, H.values, 1, H.e_min, H.e_max, prec)
    eng.set_probes(R)
    o = est.estimate(H, R, T, MU, p, density=True)
    bound = 2.0 * p ** 2 * 8 * 2.0 ** (-53 if prec == "fp64" else -24)
    default = eng.fermi_moments(T, MU, p, moments=True)["moments"]
    eng.set_tuning("alt_sweep", 1)
    steps = eng.fermi_moments(T, MU, p, moments=True)["moments"]
    eng.set_tuning("alt_sweep", -1)
    assert np.array_equal(default, steps) == (path == "steps")
    eng.set_moment_doubling(False)
    direct = eng.fermi_moments(T, MU, p, moments=True)["moments"]
    d = eng.fermi_moments(T, MU, p, moments=True, density=True)
    for m in (default, direct, d["moments"]):
        if prec == "fp64":
            check_moments(m, o["moments"])
        else:
            assert np.max(np.abs(m - o["moments"]) / o["moments"][:, :1]) < bound
    assert np.max(np.abs(d["density"] - o["density"])) < bound * np.max(np.abs(o["density"]))


def test_slices_are_built_for_a_precision_that_runs_them():
    """FP64 keeps no second copy of a pattern whose vectors do not fit the one launch: the device memory of a
    Hamiltonian of 11.6M entries is its values twice (16 bytes an entry), columns, block rows, mirror and list
    positions (28), allocated in units of 2 MiB. The kept pattern set in FP32 builds the slices then, and back in FP64
    goes without them."""
    banner("slices by precision")
    import torch
    n, entries = 9700, 1201
    H = band(n, entries)
    eng = engine_or_skip()
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    eng.set_hamiltonian(H.row_ptr, H.col_idx, H.values, 1, H.e_min, H.e_max, "fp64")
    used = before - torch.cuda.mem_get_info()[0]
    print(f"{used / H.nnzb:.1f} bytes an entry")
    assert used < 44 * H.nnzb + 12 * (2 << 20)
    H = band(n, 5)
    R = rademacher(n, 3, config_id=67)
    o = est.estimate(H, R, T, MU, P, density=True)
    bound = 2.0 * P ** 2 * 10 * 2.0 ** -24
    eng.set_hamiltonian(H.row_ptr, H.col_idx, H.values, 1, H.e_min, H.e_max, "fp64")
    eng.set_probes(R)
    check_moments(eng.fermi_moments(T, MU, P, moments=True)["moments"], o["moments"])
    eng.set_hamiltonian(None, None, H.values, 1, H.e_min, H.e_max, "fp32")
    one = eng.fermi_moments(T, MU, P, moments=True)["moments"]
    eng.set_tuning("alt_sweep", 1)
    steps = eng.fermi_moments(T, MU, P, moments=True)["moments"]
    eng.set_tuning("alt_sweep", -1)
    assert not np.array_equal(one, steps)
    assert np.max(np.abs(one - o["moments"]) / o["moments"][:, :1]) < bound
    eng.set_hamiltonian(None, None, H.values, 1, H.e_min, H.e_max, "fp64")
    check_moments(eng.fermi_moments(T, MU, P, moments=True)["moments"], o["moments"])
