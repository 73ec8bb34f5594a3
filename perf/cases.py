"""The work that users have this framework do, as cases that can be timed.

The path is two-site ab initio DMRG at one window: build the renormalised
operators, apply the Davidson sigma step H_eff psi in one of its precisions,
solve, take the energy gradient; and the spin-adapted (SU(2)) sigma and
renormalisation step on caller-supplied reduced operators.  Each case is one
call (or the few calls that belong together) through the package's binding.

Inputs are seeded and synthetic: integrals h (diagonal -2 .. -0.2, N(0, 0.1)
off it) and (pq|rs) = sum_{L<24} B_L,pq B_L,rs with B_L symmetric N(0, 0.15);
an MPS whose sector dimensions follow a Gaussian in N and 2Sz around the
chain's average, with random canonical tensors; a random normalised window
vector; random reduced blocks for the spin-adapted operators.
"""
import math

import numpy as np
import torch

from paper_2603_28648_amd import Context

SITE_QN = ((0, 0), (1, 1), (1, -1), (2, 0))  # (N, 2Sz) of |0>, |up>, |dn>, |updn>


# ---- cases ------------------------------------------------------------------
def _window(name, kind, orb, elec, two_sz, bond, window, precision="fp64", graphs=False):
    return {"name": name, "kind": kind, "orb": orb, "elec": elec, "two_sz": two_sz, "bond": bond,
            "window": window, "precision": precision, "graphs": graphs}


def _su2(name, kind, orb, elec, two_s, dim, width, two_s_max, precision="fp64"):
    return {"name": name, "kind": kind, "orb": orb, "elec": elec, "two_s": two_s, "dim": dim, "width": width,
            "two_s_max": two_s_max, "precision": precision}


def listed():
    return [
        # the smallest production window: 8 orbitals, D = 64, replayed from a graph as in
        # an eigensolver loop; launches and latency are all of it
        _window("sigma fp64 8o D64", "sigma", 8, 8, 0, 64, 3, graphs=True),
        # an ordinary window (the gradient configuration): 16 orbitals, D = 512
        _window("sigma fp64 16o D512", "sigma", 16, 16, 0, 512, 7),
        # the CAS(22,22)-shaped middle bond, D = 1024: many operators on sectors of about 100
        _window("sigma fp64 22o D1024", "sigma", 22, 22, 0, 1024, 10, graphs=True),
        # large ragged sectors, fewer operators, an off-centre window of a high-spin state:
        # the block shapes of D = 4096 calculations
        _window("sigma fp64 15o D3001", "sigma", 15, 17, 3, 3001, 6),
        # the mixed-precision eigensolver's product, on the ordinary and the largest windows
        _window("sigma bf16x3 16o D512", "sigma", 16, 16, 0, 512, 7, "bf16x3", graphs=True),
        _window("sigma bf16x3 22o D1024", "sigma", 22, 22, 0, 1024, 10, "bf16x3", graphs=True),
        # FP64 emulated on INT8 with 47 bits
        _window("sigma ozaki 16o D512", "sigma", 16, 16, 0, 512, 7, "ozaki"),
        # a few eigensolver iterations at a window, as every step of a sweep runs them
        _window("davidson fp64 14o D256", "davidson", 14, 14, 0, 256, 6),
        # operators of a new window from new integrals, and the energy of its vector
        _window("operators 12o D256", "operators", 12, 12, 0, 256, 5),
        # the reverse direction: 1- and 2-RDM of a window vector for an orbital step
        _window("gradient fp64 10o D200", "gradient", 10, 10, 0, 200, 4),
        # spin-adapted sigma on the sectors of a 2048-multiplet middle bipartition (S = 5/2),
        # with the operator pairs of a 6-orbital Hamiltonian on each side
        _su2("su2 fp64 dim2048", "su2", 6, 89, 5, 2048, 2.0, 9),
        _su2("su2 bf16x3 dim2048", "su2", 6, 89, 5, 2048, 2.0, 9, "bf16x3"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["sigma"] * 6 + ["davidson", "operators", "gradient"] + ["su2"] * 3)
    if kind == "su2":
        elec = rng.randint(12, 95)
        return {"kind": kind, "orb": rng.randint(1, 6), "elec": elec, "two_s": elec % 2 + 2 * rng.randint(0, 2),
                "dim": _log_int(rng, 60, 2040), "width": round(rng.uniform(1.2, 2.4), 2),
                "two_s_max": rng.randint(5, 9), "precision": rng.choice(["fp64", "bf16x3"])}
    lo, hi, dmax = {"sigma": (6, 17, 1400), "davidson": (6, 13, 300), "operators": (5, 12, 250),
                    "gradient": (5, 10, 200)}[kind]
    orb = rng.randint(lo, hi)
    elec = rng.randint(orb // 2 + 1, orb + orb // 2)
    window = min(orb - 2, max(0, (orb - 2) // 2 + rng.randint(-2, 2)))
    precision = rng.choice(["fp64", "fp64", "bf16x3", "bf16", "ozaki"]) if kind == "sigma" else "fp64"
    return {"kind": kind, "orb": orb, "elec": elec, "two_sz": elec % 2 + 2 * rng.randint(0, 1),
            "bond": _log_int(rng, 100 if kind == "davidson" else 24, dmax), "window": window, "precision": precision,
            "graphs": rng.random() < 0.5}


# ---- inputs -----------------------------------------------------------------
def _integrals(K, rng):
    h = np.diag(np.linspace(-2.0, -0.2, K))
    iu = np.triu_indices(K, 1)
    h[iu] = rng.normal(0.0, 0.1, len(iu[0]))
    h = np.triu(h) + np.triu(h, 1).T
    b = rng.normal(0.0, 0.15, (24, K, K))
    b = np.triu(b) + np.triu(b, 1).transpose(0, 2, 1)
    m = b.reshape(24, K * K)
    return h, (m.T @ m).reshape(K, K, K, K)


def _fock_dim(K, n, tsz):
    if n < 0 or (n + tsz) % 2:
        return 0
    a, b = (n + tsz) // 2, (n - tsz) // 2
    return math.comb(K, a) * math.comb(K, b) if 0 <= a <= K and 0 <= b <= K else 0


def _add(q, n, sign=1):
    return (q[0] + sign * SITE_QN[n][0], q[1] + sign * SITE_QN[n][1])


def _bond_dims(K, N, tsz, D, b, cap):
    """{(N, 2Sz): dim} of one bond: Gaussian weights, bounded by cap and by the Fock space of either side."""
    out, w = {}, {}
    for q, c in cap.items():
        c = min(c, _fock_dim(b, *q), _fock_dim(K - b, N - q[0], tsz - q[1]))
        if c > 0:
            out[q] = c
            w[q] = math.exp(-(q[0] - N * b / K) ** 2 / 4.5 - (q[1] - tsz * b / K) ** 2 / 8.0)
    if sum(out.values()) <= D:
        return out
    total = sum(w.values())
    d = {q: min(c, int(round(D * w[q] / total))) for q, c in out.items()}
    best = max(w, key=lambda q: (w[q], q))
    d = {q: v for q, v in d.items() if v >= min(8, max(1, D // 32), out[q])} or {best: min(D, out[best])}
    rest = D - sum(d.values())
    order = sorted(d, key=lambda q: (-d[q], q))
    while rest > 0 and any(d[q] < out[q] for q in order):  # the remainder goes to sectors with room
        for q in order:
            if rest > 0 and d[q] < out[q]:
                d[q] += 1
                rest -= 1
    return d


def _reach(dims, sign):
    out = {}
    for q, d in dims.items():
        for n in range(4):
            x = _add(q, n, sign)
            out[x] = out.get(x, 0) + d
    return out


def _bonds(c):
    K, N, tsz, D, i = c["orb"], c["elec"], c["two_sz"], c["bond"], c["window"]
    dims = [None] * (K + 1)
    dims[0], dims[K] = {(0, 0): 1}, {(N, tsz): 1}
    for b in range(1, i + 1):
        dims[b] = _bond_dims(K, N, tsz, D, b, _reach(dims[b - 1], 1))
    for b in range(K - 1, i + 1, -1):
        dims[b] = _bond_dims(K, N, tsz, D, b, _reach(dims[b + 1], -1))
    left, right = _reach(dims[i], 1), _reach(dims[i + 2], -1)
    dims[i + 1] = _bond_dims(K, N, tsz, D, i + 1, {q: min(v, right.get(q, 0)) for q, v in left.items()})
    return [sorted((q[0], q[1], d) for q, d in x.items()) for x in dims]


def _isometry(rows, cols, rng):
    """rows x cols with orthonormal columns (Cholesky QR, twice)."""
    x = torch.from_numpy(rng.normal(size=(rows, cols)))
    for _ in range(3 if rows < 2 * cols else 2):
        chol = torch.linalg.cholesky(x.T @ x)
        x = torch.linalg.solve_triangular(chol.T, x, upper=True, left=False)
    return x.numpy()


def _site_blocks(bonds, b):
    """(l, n, r) of the blocks of site b in packed order."""
    index = {q[:2]: k for k, q in enumerate(bonds[b + 1])}
    return [(l, n, index[_add(q, n)]) for l, q in enumerate(bonds[b]) for n in range(4) if _add(q, n) in index]


def _sites(c, bonds, rng):
    """Canonical site tensors {(l, n): block}, None at the window's two sites."""
    out = [None] * c["orb"]
    for b in range(c["orb"]):
        if b in (c["window"], c["window"] + 1):
            continue
        lefts, rights, blocks, got = bonds[b], bonds[b + 1], _site_blocks(bonds, b), {}
        if b < c["window"]:
            for r, q in enumerate(rights):
                mine = [(l, n) for l, n, x in blocks if x == r]
                x, off = _isometry(sum(lefts[l][2] for l, _ in mine), q[2], rng), 0
                for l, n in mine:
                    got[l, n] = x[off:off + lefts[l][2]]
                    off += lefts[l][2]
        else:
            for l, q in enumerate(lefts):
                mine = [(n, r) for x, n, r in blocks if x == l]
                x, off = _isometry(sum(rights[r][2] for _, r in mine), q[2], rng).T, 0
                for n, r in mine:
                    got[l, n] = x[:, off:off + rights[r][2]]
                    off += rights[r][2]
        out[b] = got
    return out


def _mps_arrays(c, bonds, sites):
    flat = [s for x in bonds for s in x]
    data = [None if s is None else np.concatenate([s[l, n].ravel() for l, n, _ in _site_blocks(bonds, b)])
            for b, s in enumerate(sites)]
    return {"bond_offsets": np.cumsum([0] + [len(x) for x in bonds]).astype(np.int32),
            "sector_n": np.array([s[0] for s in flat], np.int32), "sector_2sz": np.array([s[1] for s in flat], np.int32),
            "sector_dim": np.array([s[2] for s in flat], np.int32), "sites": data}


def _psi_blocks(bonds, i):
    """(r, l, n1, n2) of the window vector's blocks in packed order."""
    index = {q[:2]: k for k, q in enumerate(bonds[i + 2])}
    got = [(index[_add(_add(q, n1), n2)], l, n1, n2) for l, q in enumerate(bonds[i])
           for n1 in range(4) for n2 in range(4) if _add(_add(q, n1), n2) in index]
    return sorted(got)


def _window_inputs(c, seed):
    rng = np.random.default_rng([seed, c["orb"], c["elec"], c["bond"], c["window"]])
    h, eri = _integrals(c["orb"], rng)
    bonds = _bonds(c)
    sites = _sites(c, bonds, rng)
    n = sum(bonds[c["window"]][l][2] * bonds[c["window"] + 2][r][2] for r, l, _, _ in _psi_blocks(bonds, c["window"]))
    psi = rng.normal(size=n)
    return h, eri, bonds, sites, psi / np.linalg.norm(psi)


def _triangle(a, b, c):
    return abs(a - b) <= c <= a + b and (a + b + c) % 2 == 0


def _multiplets(c, rng):
    """Sectors (N, 2S, dim) of one half: Gaussian in N, (2S + 1) exp(-S / 2) in the spin."""
    mid, width = c["elec"] / 2, c["width"]
    keys = [(n, s) for n in range(max(0, int(mid - 3 * width)), int(mid + 3 * width) + 2)
            for s in range(n % 2, min(c["two_s_max"], n) + 1, 2)]
    w = np.array([math.exp(-0.5 * ((n - mid) / width) ** 2) * (s + 1) * math.exp(-s / 4) for n, s in keys])
    w *= rng.uniform(0.7, 1.3, len(keys))
    d = np.maximum(1, np.round(c["dim"] * w / w.sum())).astype(int)
    return [(n, s, int(x)) for (n, s), x in zip(keys, d)]


def _pair_types(m):
    """(count, left dN, 2k, right parity) of the operator pairs of a Hamiltonian with m orbitals a side:
    block Hamiltonians, one-index and two-index pairs of ranks 0 and 1."""
    sym, anti = m * (m + 1) // 2, m * (m - 1) // 2
    return [(2, 0, 0, 0), (2 * m, 1, 1, 1), (2 * m, -1, 1, 1), (sym, 2, 0, 0), (sym, -2, 0, 0), (anti, 2, 2, 0),
            (anti, -2, 2, 0), (m * m, 0, 0, 0), (m * m, 0, 2, 0)]


def _operator_blocks(sectors, dn, tk):
    got, off = [], 0
    for o, (n2, s2, d2) in enumerate(sectors):
        for i, (n1, s1, d1) in enumerate(sectors):
            if n2 == n1 + dn and _triangle(s1, tk, s2):
                got.append((o, i, off))
                off += d2 * d1
    return got, off


def _coupled(c, lsec, rsec):
    """The coupled blocks (a, b) of the reduced window vector in packed order."""
    return [(a, b) for a, (na, sa, _) in enumerate(lsec) for b, (nb, sb, _) in enumerate(rsec)
            if na + nb == c["elec"] and _triangle(sa, sb, c["two_s"])]


def _su2_size(c, lsec, rsec):
    return sum(lsec[a][2] * rsec[b][2] for a, b in _coupled(c, lsec, rsec))


def _su2_inputs(c, seed):
    rng = np.random.default_rng([seed, c["orb"], c["elec"], c["dim"]])
    shape = np.random.default_rng([c["orb"], c["elec"], c["dim"]])  # sectors are the case's, values the seed's
    lsec, rsec = _multiplets(c, shape), _multiplets(c, shape)
    lay, pairs = ([], []), []
    for count, dn, tk, parity in _pair_types(c["orb"]):
        for _ in range(count):
            pairs.append((len(pairs), len(pairs), tk, parity, float(rng.normal())))
            lay[0].append(_operator_blocks(lsec, dn, tk))
            lay[1].append(_operator_blocks(rsec, -dn, tk))
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)

    def side(lst):
        base = np.concatenate([[0], np.cumsum([n for _, n in lst])])
        data = torch.randn(int(base[-1]) + 1, dtype=torch.float64, device="cuda", generator=gen)
        return [(blocks, data, int(base[k])) for k, (blocks, _) in enumerate(lst)]

    left, right = side(lay[0]), side(lay[1])
    psi = torch.randn(_su2_size(c, lsec, rsec), dtype=torch.float64, device="cuda", generator=gen)
    return lsec, rsec, left, right, pairs, psi / psi.norm()


# ---- the calls --------------------------------------------------------------
def prepare(case, seed):
    c = dict(case)
    if c["kind"] == "su2":
        lsec, rsec, left, right, pairs, psi = _su2_inputs(c, seed)
        ctx = Context(0)
        plan = ctx.su2_plan(lsec, rsec, c["elec"], c["two_s"], left, right, pairs, c["precision"])
        return {"case": c, "ctx": ctx, "plan": plan, "psi": psi, "out": torch.empty_like(psi), "keep": (left, right)}
    h, eri, bonds, sites, psi = _window_inputs(c, seed)
    ctx = Context(0)
    args = dict(site=c["window"], h=h, eri=eri, n_elec=c["elec"], two_sz=c["two_sz"],
                mps_arrays=_mps_arrays(c, bonds, sites))
    st = {"case": c, "ctx": ctx, "psi": torch.from_numpy(psi).cuda(), "args": args}
    st["out"] = torch.empty_like(st["psi"])
    ctx.build_ops(**args)
    if c["graphs"]:
        ctx.sigma_graphs(True)
    return st


def run(state):
    c, ctx = state["case"], state["ctx"]
    if c["kind"] == "su2":
        return state["plan"].sigma(state["psi"], state["out"])
    if c["kind"] == "sigma":
        return ctx.sigma(state["psi"], state["out"], c["precision"])
    if c["kind"] == "davidson":
        x = state["out"].copy_(state["psi"])
        r = ctx.davidson(x, tol=1e-12, max_iter=6)
        return {"energy": r["energy"], "psi": x}
    if c["kind"] == "operators":
        ctx.build_ops(**state["args"])
        e, norm = ctx.energy(state["psi"], sigma=state["out"])
        return {"energy": e, "norm": norm, "sigma": state["out"]}
    dh, deri = ctx.sigma_backward(state["psi"], precision=c["precision"])
    return {"dh": dh, "deri": deri}


# ---- what a pass cannot do without ------------------------------------------
def work(case):
    c = dict(case)
    if c["kind"] == "su2":
        return _su2_work(c)
    st = prepare(c, 0)
    info, n = st["ctx"].sigma_info("fp64"), st["psi"].numel()
    st["ctx"].close()
    flops = min(info["flops"], info["flops_terms"])  # the cheaper association order of every operator pair
    ops = info["operator_bytes"]
    if c["kind"] == "sigma":
        return {"bytes": ops + 16 * n, "flops": flops}
    if c["kind"] == "davidson":  # start, six corrections, final Rayleigh quotient
        return {"bytes": 8 * (ops + 16 * n), "flops": 8 * flops}
    integrals = 8 * (c["orb"] ** 2 + c["orb"] ** 4)
    # one sigma, and the operators written once (and read once by the sigma)
    if c["kind"] == "operators":
        return {"bytes": integrals + 2 * ops + 16 * n, "flops": flops}
    # adjoints of both sides of every product
    return {"bytes": integrals + 2 * ops + 16 * n, "flops": 2 * flops}


def _su2_work(c):
    shape = np.random.default_rng([c["orb"], c["elec"], c["dim"]])
    lsec, rsec = _multiplets(c, shape), _multiplets(c, shape)
    coupled = set(_coupled(c, lsec, rsec))
    flops = nbytes = 0.0
    for count, dn, tk, _ in _pair_types(c["orb"]):
        bl, nl = _operator_blocks(lsec, dn, tk)
        br, nr = _operator_blocks(rsec, -dn, tk)
        nbytes += 8.0 * count * (nl + nr)
        bras = {}
        for o, i, _ in bl:
            bras.setdefault(i, []).append(o)
        f = 0.0
        for o, i, _ in br:
            for a, (_, _, da) in enumerate(lsec):
                outs = [x for x in bras.get(a, []) if (x, o) in coupled] if (a, i) in coupled else []
                if outs:
                    f += 2.0 * da * rsec[i][2] * rsec[o][2]
                    f += sum(2.0 * lsec[x][2] * da * rsec[o][2] for x in outs)
        flops += count * f
    return {"bytes": nbytes + 16.0 * _su2_size(c, lsec, rsec), "flops": flops}


# ---- the same in 64 bits, plainly -------------------------------------------
def _parity(x):
    for s in (16, 8, 4, 2, 1):
        x = x ^ (x >> s)
    return 1 - 2 * (x & 1)


def _excite(v, K, p, q):
    """E_pq v = sum over spins of a+_p a_q v on the 4^K occupation amplitudes (site 0 slowest, digit up + 2 dn)."""
    idx = torch.arange(v.numel(), device=v.device)
    out = torch.zeros_like(v)
    for spin in (0, 1):
        def bit(site):
            return 1 << (2 * (K - 1 - site) + spin)

        def before(site):  # occupations of the spin-orbitals in front of (site, spin)
            m = (1 << 2 * K) - (1 << (2 * (K - site)))
            return m | (1 << (2 * (K - 1 - site)) if spin else 0)
        i = idx[(idx & bit(q)) != 0]
        j = i ^ bit(q)
        ok = (j & bit(p)) == 0
        i, j = i[ok], j[ok]
        sign = _parity(i & before(q)) * _parity(j & before(p))
        out[j | bit(p)] += sign * v[i]
    return out


class _Fock:
    """The window's states as occupation amplitudes."""

    def __init__(self, c, bonds, sites):
        self.c, self.K, self.i, self.bonds = c, c["orb"], c["window"], bonds
        t = [None if s is None else {k: torch.from_numpy(np.ascontiguousarray(x)).cuda() for k, x in s.items()}
             for s in sites]
        one = torch.ones(1, 1, dtype=torch.float64, device="cuda")
        self.left, self.right = [one], [one]
        for b in range(self.i):
            new = [torch.zeros(4 ** b, 4, s[2], dtype=torch.float64, device="cuda") for s in bonds[b + 1]]
            for l, n, r in _site_blocks(bonds, b):
                new[r][:, n] += self.left[l] @ t[b][l, n]
            self.left = [x.reshape(4 ** (b + 1), -1) for x in new]
        for b in range(self.K - 1, self.i + 1, -1):
            w = 4 ** (self.K - 1 - b)
            new = [torch.zeros(s[2], 4, w, dtype=torch.float64, device="cuda") for s in bonds[b]]
            for l, n, r in _site_blocks(bonds, b):
                new[l][:, n] += t[b][l, n] @ self.right[r]
            self.right = [x.reshape(-1, 4 * w) for x in new]

    def _walk(self):
        off = 0
        for r, l, n1, n2 in _psi_blocks(self.bonds, self.i):
            shape = (self.bonds[self.i][l][2], self.bonds[self.i + 2][r][2])
            yield r, l, n1, n2, off, shape
            off += shape[0] * shape[1]

    def expand(self, psi):
        v = torch.zeros(4 ** self.i, 4, 4, 4 ** (self.K - self.i - 2), dtype=torch.float64, device="cuda")
        for r, l, n1, n2, off, (a, b) in self._walk():
            v[:, n1, n2] += self.left[l] @ psi[off:off + a * b].reshape(a, b) @ self.right[r]
        return v.reshape(-1)

    def project(self, v, like):
        out, v = torch.empty_like(like), v.reshape(4 ** self.i, 4, 4, -1)
        for r, l, n1, n2, off, (a, b) in self._walk():
            out[off:off + a * b] = (self.left[l].T @ v[:, n1, n2] @ self.right[r].T).reshape(-1)
        return out

    def excitations(self, v):
        return torch.stack([_excite(v, self.K, p, q) for p in range(self.K) for q in range(self.K)])

    def hamiltonian(self, v, h, eri):
        K = self.K
        ex = self.excitations(v)
        # 1/2 sum (pq|rs) (E_pq E_rs - d_qr E_ps)
        one = torch.from_numpy(h - 0.5 * np.einsum("pqqs->ps", eri)).cuda().reshape(-1)
        out = one @ ex
        g = 0.5 * (torch.from_numpy(eri).cuda().reshape(K * K, K * K) @ ex)
        for p in range(K):
            for q in range(K):
                out += _excite(g[p * K + q], K, p, q)
        return out


def _six_j(a, b, c, d, e, f):
    """Racah's sum, doubled spins."""
    def fac(x):
        return math.factorial(x // 2)

    def delta(x, y, z):
        return fac(x + y - z) * fac(x - y + z) * fac(-x + y + z) / fac(x + y + z + 2)
    if not (_triangle(a, b, c) and _triangle(a, e, f) and _triangle(d, b, f) and _triangle(d, e, c)):
        return 0.0
    pre = math.sqrt(delta(a, b, c) * delta(a, e, f) * delta(d, b, f) * delta(d, e, c))
    s = 0.0
    for t in range(max(a + b + c, a + e + f, d + b + f, d + e + c), min(a + b + d + e, b + c + e + f, c + a + f + d) + 1, 2):
        s += (-1) ** (t // 2) * fac(t + 2) / (fac(t - a - b - c) * fac(t - a - e - f) * fac(t - d - b - f) *
                                              fac(t - d - e - c) * fac(a + b + d + e - t) *
                                              fac(b + c + e + f - t) * fac(c + a + f + d - t))
    return pre * s


def _su2_exact(c, seed):
    lsec, rsec, left, right, pairs, psi = _su2_inputs(c, seed)
    host = [x[0][1].cpu().numpy() for x in (left, right)]
    off, where = 0, {}
    for a, b in _coupled(c, lsec, rsec):
        where[a, b] = off
        off += lsec[a][2] * rsec[b][2]
    x = psi.cpu().numpy()
    y = np.zeros(off)
    vec = {k: x[o:o + lsec[k[0]][2] * rsec[k[1]][2]].reshape(lsec[k[0]][2], -1) for k, o in where.items()}
    out = {k: y[o:o + lsec[k[0]][2] * rsec[k[1]][2]].reshape(lsec[k[0]][2], -1) for k, o in where.items()}
    weight = {}
    for li, ri, tk, parity, coef in pairs:
        by_ket = {}
        for o, i, at in left[li][0]:
            at += left[li][2]
            by_ket.setdefault(i, []).append((o, host[0][at:at + lsec[o][2] * lsec[i][2]].reshape(lsec[o][2], -1)))
        for o, i, at in right[ri][0]:
            at += right[ri][2]
            m = host[1][at:at + rsec[o][2] * rsec[i][2]].reshape(rsec[o][2], -1).T
            for a in range(len(lsec)):
                if (a, i) not in where:
                    continue
                t = None
                for a2, block in by_ket.get(a, []):
                    if (a2, o) not in where:
                        continue
                    key = (lsec[a2][1], rsec[o][1], lsec[a][1], rsec[i][1], tk)
                    if key not in weight:
                        s2, t2, s1, t1, k = key
                        weight[key] = ((-1) ** ((s1 + t2 + c["two_s"] + k) // 2) * math.sqrt((s2 + 1) * (t2 + 1) / (k + 1))
                                       * _six_j(s1, t1, c["two_s"], t2, s2, k))
                    w = coef * weight[key] * (-1) ** (parity * lsec[a][0])
                    if w == 0.0:
                        continue
                    if t is None:
                        t = vec[a, i] @ m
                    out[a2, o] += w * (block @ t)
    return y


def exact(case, seed):
    c = dict(case)
    if c["kind"] == "su2":
        return _su2_exact(c, seed)
    if c["kind"] == "davidson" or c["orb"] > 10:
        return None
    h, eri, bonds, sites, psi = _window_inputs(c, seed)
    space, psi = _Fock(c, bonds, sites), torch.from_numpy(psi).cuda()
    v = space.expand(psi)
    if c["kind"] == "gradient":
        K = c["orb"]
        ex = space.excitations(v)
        gamma = (ex @ v).reshape(K, K)
        pair = (ex.reshape(K, K, -1).transpose(0, 1).reshape(K * K, -1) @ ex.T).reshape(K, K, K, K)
        for q in range(K):
            pair[:, q, q, :] -= gamma
        return {"dh": gamma, "deri": 0.5 * pair}
    s = space.project(space.hamiltonian(v, h, eri), psi)
    if c["kind"] == "operators":
        return {"energy": float(psi @ s), "norm": float(psi @ psi), "sigma": s}
    return s
