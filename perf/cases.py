"""Timed cases of the randomized Fermi-operator path, through the public Engine calls.

A case names a model (periodic simple-cubic lattice, Cu-like fcc cluster with 9x9 blocks, random
graph), its size, the arithmetic of the products, the probe block, the number of Chebyshev terms
and the call a program makes: moments, density blocks, energy with gradient and forces, a search
for the chemical potential on stored moments, the rational (pole) estimate, or moments with an
overlap.  prepare() builds the inputs from the seed and hands H and the probes to an Engine, as a
program does before the call; run() is the call.
"""

import functools
import math

import numpy as np
import torch

import paper_1812_05264_amd as rfo
from paper_1812_05264_amd.scan import find_mu

DEV = "cuda" if torch.cuda.is_available() else "cpu"
A_HALF = 0.5 * 3.61      # half the fcc lattice constant, Angstrom
DECAY = 1.5              # decay length of the hopping, Angstrom


def _case(name, call, model, size, precision, probes, s, p, T, mu):
    c = {"call": call, "model": model, "size": size, "precision": precision, "probes": probes,
         "s": s, "p": p, "T": T, "mu": mu}
    return c if name is None else {"name": name, **c}


def listed():
    return [
        # one small lattice, N/E/F and per-probe moments: the shortest call a program makes, as in
        # a loop over many disorder realisations
        _case("sc8_moments", "moments", "lattice", 8, "fp64", "sign", 64, 256, 0.1, 0.0),
        # energy and forces of a small cluster: one step of a molecular-dynamics or relaxation loop
        _case("cu55_forces", "forces", "cluster", 55, "fp64", "sign", 64, 256, 0.3, 1.165),
        # chemical potential for a wanted electron count on moments already computed
        _case("sc16_mu", "mu", "lattice", 16, "fp64", "sign", 64, 1024, 0.05, 0.3),
        # ordinary irregular sparse matrix, dense (Gaussian) probes, density blocks
        _case("graph_density", "density", "graph", 5003, "fp64", "dense", 50, 301, 0.2, 0.1),
        # an ordinary lattice in single precision with an odd number of probes
        _case("sc32_fp32_moments", "moments", "lattice", 32, "fp32", "sign", 100, 1001, 0.05, 0.3),
        # the largest lattice: density blocks over the full expansion
        _case("sc64_density", "density", "lattice", 64, "fp64", "sign", 256, 2048, 0.02, 0.3),
        # an ordinary cluster, moments only: N(mu), band energy and free energy
        _case("cu4k_moments", "moments", "cluster", 4000, "fp64", "sign", 128, 4000, 0.05, 1.165),
        # forces with multi-colour probes (32 colours, 288 columns) in single precision
        _case("cu4k_fp32_colored_forces", "forces", "cluster", 4000, "fp32", "colored", 288, 800, 0.1,
              1.165),
        # the largest cluster: energy, gradient and forces in FP64
        _case("cu16k_forces", "forces", "cluster", 16000, "fp64", "sign", 256, 500, 0.2, 1.165),
        # the same on the matrix cores in BF16
        _case("cu16k_bf16_forces", "forces", "cluster", 16000, "bf16", "sign", 256, 1000, 0.2, 1.165),
        # rational (pole) estimate with density blocks
        _case("cu250_rational", "rational", "cluster", 250, "fp64", "sign", 128, 24, 0.3, 1.165),
        # nonorthogonal basis: conjugate gradients with the overlap in every step, P and Q blocks
        _case("cu500_overlap", "overlap", "cluster", 500, "fp64", "sign", 128, 60, 0.3, 1.165),
    ]


def draw(rng):
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    T, mu = round(rng.uniform(0.05, 0.4), 3), round(rng.uniform(0.3, 1.5), 3)
    s = rng.choice([log(1, 256), 64, 128, 256])
    kind = rng.choice(["lattice", "lattice", "cluster", "cluster", "cluster", "graph", "mu", "rational", "overlap"])
    probes = rng.choice(["sign", "sign", "sign", "dense"])
    if kind in ("lattice", "graph"):
        n = log(8, 48) if kind == "lattice" else log(200, 60000)
        call = rng.choice(["moments", "density", "forces"])
        p = log(64, 800)
        return _case(None, call, kind, n, rng.choice(["fp64", "fp64", "fp32"]), probes, s, p, T, mu)
    if kind == "cluster":
        n, p = log(13, 6000), log(50, 600)
        prec = rng.choice(["fp64", "fp64", "fp32", "bf16", "bf16x2"])
        if rng.random() < 0.15:
            probes, s = "colored", 288
        call = rng.choice(["moments", "density", "forces", "forces"])
        return _case(None, call, kind, n, prec, probes, s, p, T, mu)
    if kind == "mu":
        return _case(None, "mu", "lattice", log(8, 24), "fp64", "sign", s, log(400, 3000), max(T, 0.1), mu)
    if kind == "rational":
        return _case(None, "rational", "cluster", log(13, 300), "fp64", "sign", s, rng.randint(16, 28), 0.3, mu)
    return _case(None, "overlap", "cluster", log(13, 600), "fp64", "sign", s, log(10, 60), T, mu)


# ---- geometry (a function of the sizes alone) ------------------------------------------------

def _morton(ijk):
    code = np.zeros(ijk.shape[0], dtype=np.int64)
    for b in range(10):
        for d in range(3):
            code |= ((ijk[:, d] >> b) & 1) << (3 * b + d)
    return code


def _csr(rows, cols, n):
    o = np.lexsort((cols, rows))
    rows, cols = rows[o], cols[o]
    ptr = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(np.bincount(rows, minlength=n), out=ptr[1:])
    key = rows * n + cols
    mirror = np.searchsorted(key, cols * n + rows)
    return ptr, rows, cols, mirror


@functools.lru_cache(maxsize=4)
def _lattice(L):
    i = np.arange(L ** 3)
    xyz = np.stack([i % L, i // L % L, i // (L * L)], axis=1)
    xyz = xyz[np.argsort(_morton(xyz), kind="stable")]
    index = np.empty(L ** 3, dtype=np.int64)
    index[xyz[:, 0] + L * (xyz[:, 1] + L * xyz[:, 2])] = i
    cols = [i]
    for d in range(3):
        for step in (1, -1):
            q = xyz.copy()
            q[:, d] = (q[:, d] + step) % L
            cols.append(index[q[:, 0] + L * (q[:, 1] + L * q[:, 2])])
    return _csr(np.tile(i, 7), np.concatenate(cols), L ** 3) + (None,)


@functools.lru_cache(maxsize=4)
def _cluster(n):
    R = int(math.ceil((3.0 * n / (2.0 * math.pi)) ** (1.0 / 3.0))) + 4
    g = np.arange(-R, R + 1)
    pts = np.stack(np.meshgrid(g, g, g, indexing="ij"), axis=-1).reshape(-1, 3)
    pts = pts[pts.sum(axis=1) % 2 == 0]
    ijk = pts[np.lexsort((pts[:, 2], pts[:, 1], pts[:, 0], (pts ** 2).sum(axis=1)))[:n]]
    ijk = ijk[np.argsort(_morton(ijk - ijk.min(axis=0)), kind="stable")]
    S = 2 * R + 7
    key = lambda q: ((q[:, 0] + R + 3) * S + q[:, 1] + R + 3) * S + q[:, 2] + R + 3  # noqa: E731
    where = np.full(S ** 3, -1, dtype=np.int64)
    where[key(ijk)] = np.arange(n)
    rows, cols = [np.arange(n)], [np.arange(n)]
    near = pts[np.isin((pts ** 2).sum(axis=1), (2, 4))]
    for off in near:
        J = where[key(ijk + off)]
        rows.append(np.nonzero(J >= 0)[0])
        cols.append(J[J >= 0])
    return _csr(np.concatenate(rows), np.concatenate(cols), n) + (ijk,)


@functools.lru_cache(maxsize=4)
def _graph(n):
    r = np.random.RandomState(n)
    i = np.repeat(np.arange(n), r.randint(0, 7, n))
    j = (i + r.randint(1, n, i.size)) % n
    near = r.rand(i.size) < 0.7
    j[near] = (i[near] + r.randint(1, 40, near.sum())) % n
    pairs = np.unique(np.minimum(i, j)[i != j] * n + np.maximum(i, j)[i != j])
    i, j = pairs // n, pairs % n
    d = np.arange(n)
    return _csr(np.concatenate([d, i, j]), np.concatenate([d, j, i]), n) + (None,)


GEOMETRY = {"lattice": _lattice, "cluster": _cluster, "graph": _graph}


# ---- inputs (from the seed) --------------------------------------------------------------------

def _normal(gen, *shape):
    return torch.randn(*shape, generator=gen, dtype=torch.float64, device=DEV)


def _symmetric(v, mirror):
    return 0.5 * (v + v[mirror].transpose(1, 2))


def _apply(vals, rows, cols, X, nb):
    """Y = H X for blocks [nnzb, bd, bd] and X [nb * bd, s], a chunk of blocks at a time."""
    bd, s = vals.shape[1], X.shape[1]
    Xb = X.view(nb, bd, s)
    Y = torch.zeros_like(Xb)
    step = max(1, (1 << 28) // (bd * s))
    for z in range(0, cols.numel(), step):
        g = Xb[cols[z:z + step]]
        Y.index_add_(0, rows[z:z + step], vals[z:z + step] * g if bd == 1 else torch.bmm(vals[z:z + step], g))
    return Y.view_as(X)


def _extremes(vals, rows, cols, nb, gen):
    """Extreme eigenvalues by 40 Lanczos steps, widened by 3% of the spread."""
    n = nb * vals.shape[1]
    v, w, b = _normal(gen, n, 1), torch.zeros(n, 1, dtype=torch.float64, device=DEV), 0.0
    v /= v.norm()
    al, be = [], []
    for _ in range(min(40, n)):
        u = _apply(vals, rows, cols, v, nb) - b * w
        a = (u * v).sum()
        u -= a * v
        b = u.norm()
        al.append(a)
        be.append(b)
        w, v = v, u / b
    al, be = torch.stack(al).cpu(), torch.stack(be).cpu()
    e = torch.linalg.eigvalsh(torch.diag(al) + torch.diag(be[:-1], 1) + torch.diag(be[:-1], -1))
    lo, hi = float(e[0]), float(e[-1])
    return lo - 0.03 * (hi - lo), hi + 0.03 * (hi - lo)


def _inputs(case, seed):
    gen = torch.Generator(device=DEV).manual_seed(1000003 * (seed + 1) + case["size"])
    ptr, rows, cols, mirror, ijk = GEOMETRY[case["model"]](case["size"])
    nb, nnzb = ptr.size - 1, cols.size
    r, c, m = (torch.from_numpy(a).to(DEV) for a in (rows, cols, mirror))
    x = {"ptr": ptr, "col": cols.astype(np.int32), "rows": r, "cols": c, "mirror": m, "nb": nb}
    if case["model"] == "lattice":
        v = torch.full((nnzb, 1, 1), -1.0, dtype=torch.float64, device=DEV)
        v[r == c] = torch.rand(nb, 1, 1, generator=gen, dtype=torch.float64, device=DEV) - 0.5
        x.update(values=v, bd=1, e_min=-1.01 * 6.5, e_max=1.01 * 6.5)
    elif case["model"] == "graph":
        v = _symmetric(_normal(gen, nnzb, 1, 1), m)
        rad = torch.zeros(nb, dtype=torch.float64, device=DEV).index_add_(0, r, v.abs().reshape(-1)).max()
        x.update(values=v, bd=1, e_min=-float(rad), e_max=float(rad))
    else:
        pos = torch.from_numpy(ijk * A_HALF).to(DEV)
        d = pos[r] - pos[c]
        dist = d.norm(dim=1)
        env = torch.exp(-dist / DECAY)[:, None, None]
        v = math.sqrt(2.0) * _symmetric(_normal(gen, nnzb, 9, 9), m) * env
        lo, hi = _extremes(v, r, c, nb, gen)
        v *= 20.0 / (hi - lo)
        v[r == c] -= 10.0 * (hi + lo) / (hi - lo) * torch.eye(9, dtype=torch.float64, device=DEV)
        x.update(values=v, bd=9, e_min=-10.0, e_max=10.0)
        if case["call"] == "forces":
            unit = torch.where((dist > 0)[:, None], d / dist.clamp(min=1e-300)[:, None], torch.zeros_like(d))
            x["dHdR"] = (-unit / DECAY)[:, :, None, None] * v[:, None]
        if case["call"] == "overlap":
            S = 0.16 * math.sqrt(2.0) * _symmetric(_normal(gen, nnzb, 9, 9), m) * env
            S[r == c] = torch.eye(9, dtype=torch.float64, device=DEV)
            edge = 10.0 / _extremes(S, r, c, nb, gen)[0]
            x.update(S=S, e_min=-edge, e_max=edge)
    if case["call"] == "forces" and "dHdR" not in x:
        a = _normal(gen, nnzb, 3, 1, 1)
        x["dHdR"] = a - a[m]
    n, s = nb * x["bd"], case["s"]
    if case["probes"] == "colored":
        cell = (ijk % 4) @ np.array([16, 4, 1])
        x["colours"] = np.unique(cell, return_inverse=True)[1].reshape(-1).astype(np.int32)
        x["signs"] = torch.randint(0, 2, (nb, 9), generator=gen, device=DEV).double().mul_(2).sub_(1)
    elif case["probes"] == "dense":
        x["R"] = _normal(gen, n, s)
    else:
        x["R"] = torch.randint(0, 2, (n, s), generator=gen, device=DEV).double().mul_(2).sub_(1)
    return x


def prepare(case, seed):
    x = _inputs(case, seed)
    eng = rfo.Engine(0)
    eng.set_hamiltonian(x["ptr"], x["col"], x["values"], x["bd"], x["e_min"], x["e_max"], case["precision"])
    if "S" in x:
        eng.set_overlap(x["S"])
    if "colours" in x:
        eng.set_colored_probes(x["colours"], 9, x["signs"].cpu().numpy())
    else:
        eng.set_probes(x["R"])
    st = {"case": case, "engine": eng, "dHdR": x.get("dHdR")}
    if case["call"] in ("density", "forces", "rational"):
        st["blocks"] = torch.empty_like(x["values"])
    if case["call"] == "mu":
        e = eng.fermi_moments(case["T"], case["mu"], case["p"], moments=False)
        st["wanted"] = e["N"]
    if case["call"] == "rational":
        st["fit"] = rfo.rational_fit(case["p"], case["T"], case["mu"], x["e_min"], x["e_max"])
    return st


# ---- the call ------------------------------------------------------------------------------------

def _as(case, v):
    """Results in the type whose digits the call's arithmetic carries."""
    if case["precision"] == "fp64":
        return v
    t = torch.as_tensor(v)
    return t.to(torch.float32 if case["precision"] == "fp32" else torch.bfloat16)


def run(state):
    case, eng = state["case"], state["engine"]
    T, mu, p = case["T"], case["mu"], case["p"]
    call = case["call"]
    if call == "moments":
        o = eng.fermi_moments(T, mu, p, moments=True)
        out = {"moments": o["moments"]}
    elif call == "density":
        o = eng.fermi_moments(T, mu, p, moments=False, density=True, density_out=state["blocks"])
        out = {"density": o["density"]}
    elif call == "forces":
        o = eng.energy_and_dEdH(T, mu, p, dFdH_out=state["blocks"])
        out = {"dFdH": o["dFdH"], "forces": eng.hf_forces(state["dHdR"])}
    elif call == "mu":
        found = find_mu(eng, state["wanted"], T, mu - 1.0, mu + 1.3, tol=1e-9)
        o = eng.traces_at(T, found)
        out = {"mu": found}
    elif call == "rational":
        o = eng.rational(mu, state["fit"], tol=1e-12, density=True, density_out=state["blocks"])
        out = {"density": o["density"]}
    else:
        o = eng.fermi_moments(T, mu, p, moments=True, density=True)
        out = {"moments": o["moments"], "density": o["density"], "Q": eng.density_q()}
    out.update({k: o[k] for k in ("N", "E", "F")})
    return {k: _as(case, v) for k, v in out.items()}


# ---- work and exact values -----------------------------------------------------------------------

def _sizes(case):
    g = GEOMETRY[case["model"]](case["size"])
    bd = 9 if case["model"] == "cluster" else 1
    return g[0].size - 1, g[2].size, bd


def work(case):
    """Products of the recurrence and, where a vector block exceeds what the caches of the card
    hold, one read of H and three passes over a vector block per product."""
    nb, nnzb, bd = _sizes(case)
    n, s, p, call = nb * bd, case["s"], case["p"], case["call"]
    hb = {"fp64": 8, "fp32": 4, "bf16": 2, "bf16x2": 4}[case["precision"]]
    vb = 8 if case["precision"] == "fp64" else 4
    nnz = nnzb * bd * bd
    h_bytes = nnz * hb + nnzb * 4 + nb * 8
    blocks = nnz * 8 if call in ("density", "forces", "rational", "overlap") else 0
    base = h_bytes + n * s / 8 + blocks
    if call == "mu":
        return {"bytes": s * p * 8.0, "flops": 2.0 * s * p}
    steps = {"moments": p // 2, "density": p - 1, "forces": 2 * (p // 2), "rational": 2 * 2 * p * 10,
             "overlap": p * 20}[call]
    width = 2 if call == "rational" else 1
    stream = n * s * vb * width
    per = (h_bytes + 3 * stream) if stream > (32 << 20) else 0
    flops = 2.0 * nnz * s * width * steps
    if call == "forces":
        flops += 2.0 * nnz * s * (p // 2)
        base += 3 * nnz * 8
    if call == "moments":
        base += s * p * 8
    return {"bytes": float(base + per * steps), "flops": float(flops)}


def _coefficients(case, a, b):
    """Chebyshev coefficients of f, x f and g on [a, b] from 4 p Chebyshev-Gauss nodes."""
    p, nq = case["p"], 4 * case["p"]
    e = 0.5 * (a + b) + 0.5 * (b - a) * np.cos(np.pi * (np.arange(nq) + 0.5) / nq)
    z = (e - case["mu"]) / case["T"]
    f = 1.0 - np.tanh(0.5 * z)
    g = -2.0 * case["T"] * (np.maximum(-z, 0.0) + np.log1p(np.exp(-np.abs(z))))
    out = []
    for h in (f, e * f, g):
        spec = np.fft.fft(np.concatenate([h, h[::-1]]))[:p]
        ck = (np.exp(-0.5j * np.pi * np.arange(p) / nq) * spec).real / nq
        ck[0] *= 0.5
        out.append(ck)
    return out


def _probe_block(case, x):
    if "R" in x:
        return x["R"], 1.0 / case["s"]
    nb = x["nb"]
    col = torch.from_numpy(x["colours"].astype(np.int64)).to(DEV)
    R = torch.zeros(nb, 9, 32, 9, dtype=torch.float64, device=DEV)
    o = torch.arange(9, device=DEV)
    R[torch.arange(nb, device=DEV)[:, None], o[None], col[:, None], o[None]] = x["signs"]
    return R.view(nb * 9, 288)[:, :9 * (int(col.max()) + 1)], 1.0


def _outer(x, X, Y, out, scale):
    """out[z] += scale X_I Y_J^T on the block pattern."""
    bd, s = x["bd"], X.shape[1]
    Xb, Yb = X.view(-1, bd, s), Y.view(-1, bd, s)
    step = max(1, (1 << 28) // (bd * s))
    for z in range(0, x["cols"].numel(), step):
        e = slice(z, z + step)
        yt = Yb[x["cols"][e]].transpose(1, 2).contiguous()
        out[e] += scale * torch.bmm(Xb[x["rows"][e]], yt)


def _dense(v, x):
    nb, bd = x["nb"], x["bd"]
    M = torch.zeros(nb, nb, bd, bd, dtype=torch.float64, device=DEV)
    M[x["rows"], x["cols"]] = v
    return M.permute(0, 2, 1, 3).reshape(nb * bd, nb * bd).contiguous()


def exact(case, seed):
    nb, nnzb, bd = _sizes(case)
    call, p = case["call"], case["p"]
    n, s = nb * bd, case["s"]
    moved = 48.0 * nnzb * bd * s * {"moments": p, "density": p, "forces": 3 * p, "mu": p}.get(call, 1)
    if moved > 6e13 or (call == "rational" and n > 3000) or (call == "overlap" and n > 6000):
        return None  # over about 20 seconds
    x = _inputs(case, seed)
    a, b = x["e_min"], x["e_max"]
    R, w = _probe_block(case, x)
    if call == "rational":
        # the fit's error is below 1e-11 of f and g: their exact values on the probe block
        e, U = torch.linalg.eigh(_dense(x["values"], x).cpu())
        z = (e - case["mu"]) / case["T"]
        f = 1.0 - torch.tanh(0.5 * z)
        g = -2.0 * case["T"] * (torch.clamp(-z, min=0.0) + torch.log1p(torch.exp(-z.abs())))
        U = U.to(DEV)
        C = U.T @ R
        q = w * (C * C).sum(1).cpu()
        D = torch.zeros_like(x["values"])
        _outer(x, U @ (f.to(DEV)[:, None] * C), R, D, w)
        return {"density": D, "N": float((q * f).sum()), "E": float((q * e * f).sum()),
                "F": float((q * g).sum())}
    if call == "overlap":
        Si = torch.linalg.inv(_dense(x["S"], x).cpu()).to(DEV)
        H = _dense(x["values"], x)
        Hh = (2.0 * H - (a + b) * _dense(x["S"], x)) / (b - a)
        step = lambda y: Hh @ (Si @ y)  # noqa: E731
    else:
        hv = x["values"] * (2.0 / (b - a))
        hv[x["rows"] == x["cols"]] -= (a + b) / (b - a) * torch.eye(bd, dtype=torch.float64, device=DEV)
        if bd == 1:
            M = torch.sparse_csr_tensor(torch.from_numpy(x["ptr"]).to(DEV), x["cols"], hv.reshape(-1), (n, n))
            step = lambda y: M @ y  # noqa: E731
        else:
            step = lambda y: _apply(hv, x["rows"], x["cols"], y, nb)  # noqa: E731
    cf, cef, cg = _coefficients(case, a, b)
    doubled = call in ("moments", "mu", "forces")
    last = p // 2 if doubled else p - 1
    y, prev, acc = R.clone(), None, cf[0] * R
    mom = torch.zeros(max(p, 2 * last + 1), R.shape[1], dtype=torch.float64, device=DEV)
    mom[0] = (R * R).sum(0)
    kept = [y]
    for k in range(1, last + 1):
        nxt = step(y) if k == 1 else 2.0 * step(y) - prev
        prev, y = y, nxt
        if doubled:
            mom[2 * k - 1] = (y * prev).sum(0) if k == 1 else 2.0 * (y * prev).sum(0) - mom[1]
            mom[2 * k] = 2.0 * (y * y).sum(0) - mom[0]
        else:
            mom[k] = (R * y).sum(0)
            acc += cf[k] * y
        if call == "forces":
            kept.append(y)
    mom = mom[:p].cpu().numpy()
    tr = w * mom.sum(1)
    out = {"N": float(cf @ tr), "E": float(cef @ tr), "F": float(cg @ tr)}
    if call == "mu":
        return {"mu": case["mu"], **out}
    if call in ("moments", "overlap"):
        out["moments"] = torch.from_numpy(mom.T.copy())
    if call == "density":
        out["density"] = torch.zeros_like(x["values"])
        _outer(x, acc, R, out["density"], w)
    if call == "overlap":
        P = Si @ acc
        out["density"], out["Q"] = torch.zeros_like(x["values"]), torch.zeros_like(x["values"])
        _outer(x, P, R, out["density"], w)
        _outer(x, Si @ (H @ P), R, out["Q"], w)
    if call == "forces":
        G = torch.zeros_like(x["values"])
        al, be = np.zeros(last + 2), np.zeros(last + 2)
        for j in range(1, last + 1):
            if 2 * j < p:
                al[j] = 2.0 * cg[2 * j]
            if j >= 2 and 2 * j - 1 < p:
                be[j] = 2.0 * cg[2 * j - 1]
        if last >= 1:
            be[1] = cg[1] - 0.5 * be[2:].sum()
        z1 = z2 = None  # z_{j+1}, z_{j+2}
        for j in range(last, 0, -1):
            z = 2.0 * al[j] * kept[j] + be[j] * kept[j - 1]
            if j < last:
                z += be[j + 1] * kept[j + 1] + 2.0 * step(z1)
            if j < last - 1:
                z -= z2
            z1, z2 = z, z1
            _outer(x, z, kept[j - 1], G, (1.0 if j == 1 else 2.0) * w * 2.0 / (b - a))
        G = _symmetric(G, x["mirror"])
        t = (G[:, None] * x["dHdR"]).sum((2, 3))
        F = torch.zeros(nb, 3, dtype=torch.float64, device=DEV)
        F.index_add_(0, x["rows"], -t)
        F.index_add_(0, x["cols"], t)
        out["dFdH"], out["forces"] = G, F.cpu()
    return out
