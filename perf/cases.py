"""Performance cases: the work that programs give this library, through its public entry points.

A case is one call of ``paper_2507_11424_amd.Handle`` on a seeded synthetic
tensor-network state (``peps_inputs``; the sizes are those of the named
workloads c1..c4 and hhx, of the benchmark and of the tests, or smaller ones
of the same kind).  ``op`` says which call:

    norm    boundary_contract: log Z of <psi|psi>
    env     environments: one-site density matrices, <ZZ>, two-site marginals
    sample  sample, given the state's boundary set (a program contracts a state
            once and then draws from it); uniforms are the caller's
    amp     amplitude: log p of given bitstrings by the separate contraction
    stats   sample_stats: KLD, effective sample size, importance-sampled <Z>
    bp      bp: messages, Z_BP and the loop BP error of every loop
    update  simple_update: one Heisenberg Trotter layer on a correlated state

Every case keeps one handle per state, as a program does.  A mode that stores
complex64 (fp32, bf16x3, bf16x6) hands its results on in single precision.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2507_11424_amd as tnb
from peps_inputs import build_lattice, heavy_hex_lattice, random_peps, rotated_square_lattice, site_dims
from peps_inputs.circuits import heisenberg_circuit

ROTSQ = {"rotsq21": (4, 10), "rotsq": (10, 20)}  # chip rows and largest column; 21 and 105 qubits


def listed():
    return [
        # sample quality of a finished run on the 144-qubit lattice: three reductions, all latency
        dict(name="stats_144q", op="stats", qubits=144, n=4096),
        # the smallest state (c1): launches and host time are everything
        dict(name="norm_4x4_D2", op="norm", lattice="square", rows=4, cols=4, D=2, chi=16, prec="fp64", dtype="c128"),
        # many samples of the smallest state, one wave of 1000
        dict(name="sample_4x4_D2", op="sample", lattice="square", rows=4, cols=4, D=2, chi=16, chi_x=16, n=1000,
             prec="fp64", dtype="c128"),
        # c2: an ordinary square lattice with truncating bonds
        dict(name="norm_8x8_D4", op="norm", lattice="square", rows=8, cols=8, D=4, chi=32, prec="fp64", dtype="c128"),
        # every local expectation value of a small lattice of odd sizes
        dict(name="env_5x7_D3", op="env", lattice="square", rows=5, cols=7, D=3, chi=27, prec="fp64", dtype="c128"),
        # c2 sampled: the per-sample environments of a full square lattice
        dict(name="sample_8x8_D4", op="sample", lattice="square", rows=8, cols=8, D=4, chi=32, chi_x=32, n=64,
             prec="fp64", dtype="c128"),
        # c3, the headline lattice (144 qubits): its norm in FP64 and in the split mode
        dict(name="norm_brick_D8", op="norm", lattice="brick", rows=12, cols=12, D=8, chi=64, prec="fp64",
             dtype="c64"),
        dict(name="norm_brick_D8_bf16x6", op="norm", lattice="brick", rows=12, cols=12, D=8, chi=64, prec="bf16x6",
             dtype="c64"),
        # the headline lattice sampled in the split mode
        dict(name="sample_brick_D8_bf16x6", op="sample", lattice="brick", rows=12, cols=12, D=8, chi=64, chi_x=32,
             n=8, prec="bf16x6", dtype="c64"),
        # verification of drawn samples on the 129-qubit heavy-hex lattice at twice the bond
        dict(name="amp_heavyhex_D8", op="amp", lattice="heavyhex", rows=7, cols=15, D=8, chi_x=16, n=32, prec="fp64",
             dtype="c64"),
        # BP and the loop error on the headline lattice
        dict(name="bp_brick_D8", op="bp", lattice="brick", rows=12, cols=12, D=8, dtype="c64"),
        # one Trotter layer on the heavy-hex lattice at the benchmark's bond
        dict(name="update_heavyhex_D16", op="update", lattice="heavyhex", rows=7, cols=15, D=16, dtype="c128"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo - 0.49), math.log(hi + 0.49)))))


_CAP = {}


def _caps():
    """Most work a drawn case of each call may have: the listed cases' own."""
    if not _CAP:
        for c in listed():
            _CAP[c["op"]] = max(_CAP.get(c["op"], 0.0), work(c)["flops"])
    return _CAP


def draw(rng):
    while True:
        op = rng.choice(["stats", "norm", "norm", "env", "sample", "sample", "amp", "bp", "update"])
        if op == "stats":
            return dict(op=op, qubits=rng.choice([16, 64, 105, 129, 144]) + rng.randrange(2), n=_log_int(rng, 8, 16384))
        kind = rng.choice(["square", "brick", "heavyhex", "rotsq21"] + (["rotsq"] if op in ("norm", "bp") else []))
        big = op in ("norm", "bp", "amp", "update") and kind in ("brick", "heavyhex")
        rows, cols = rng.randint(3, 12 if big else 8), rng.randint(3, 12 if big else 8)
        if kind == "heavyhex":
            rows, cols = rng.randint(2, 7 if big else 4), rng.randint(5, 15 if big else 11)
        elif kind.startswith("rotsq"):
            rows = cols = 0
        D = rng.choice([2, 3, 4, 5, 6, 8])
        c = dict(op=op, lattice=kind, rows=rows, cols=cols, D=D)
        if op == "update":
            c["D"] = rng.choice([2, 4, 6, 8, 12, 16]) if kind in ("brick", "heavyhex") else rng.choice([2, 3, 4, 6])
            c["dtype"] = rng.choice(["c128", "c128", "c64"])
        elif op == "bp":
            c["dtype"] = rng.choice(["c128", "c64"])
        else:
            c["prec"] = rng.choice(["fp64", "fp64", "fp32", "bf16x3", "bf16x6"])
            c["dtype"] = rng.choice(["c128", "c64"]) if c["prec"] == "fp64" else "c64"
            if op != "amp":
                c["chi"] = _log_int(rng, 4, 64)
            if op in ("sample", "amp"):
                c["chi_x"] = min(_log_int(rng, 4, 32), c.get("chi", 32))
                c["n"] = _log_int(rng, 1, 1000 if D <= 3 else 64)
        # launch counts and serial chains do not show in flops: the lattices above cap the sites
        if work(c)["flops"] <= 0.5 * _caps()[op]:
            return c


# ------------------------------------------------------------------ inputs

def _lattice(c):
    k = c["lattice"]
    if k in ROTSQ:
        return rotated_square_lattice(c["D"], *ROTSQ[k])
    if k == "heavyhex":
        return heavy_hex_lattice(c["rows"], c["cols"], c["D"])
    return build_lattice((k, c["rows"], c["cols"], c["D"]))


def _host_state(c, seed):
    """(lattice, host tensors): Haar product states plus 0.2 of Gaussian noise on
    the bonds, every tensor normalised -- the recipe of the named workloads."""
    lat = _lattice(c)
    T = random_peps(lat, "haar", 0.2, seed)
    if c["dtype"] == "c64":
        T = [[t.astype(np.complex64) for t in row] for row in T]
    return lat, T


def _bits_and_uniforms(n, q, seed):
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    return (torch.randint(0, 2, (n, q), generator=g, dtype=torch.uint8, device="cuda"),
            torch.rand((n, q), generator=g, dtype=torch.float64, device="cuda"))


def _log_weights(n, seed):
    g = torch.Generator(device="cuda").manual_seed(int(seed) + 1)
    z = torch.randn((2, n), generator=g, dtype=torch.float64, device="cuda")
    lq = -60.0 + 4.0 * z[0]
    return lq, lq + 0.3 * z[1] - 5.0


def prepare(c, seed):
    h = tnb.Handle(0)
    if c["op"] == "stats":
        bits, _ = _bits_and_uniforms(c["n"], c["qubits"], seed)
        lq, lp = _log_weights(c["n"], seed)
        return dict(c=c, h=h, bits=bits, lq=lq, lp=lp, log_Z=-5.0)
    lat, T = _host_state(c, seed)
    s = dict(c=c, h=h, lat=lat, peps=tnb.Peps.from_numpy(lat, T, dtype=c["dtype"]))
    if "prec" in c:
        s["opts"] = tnb.make_opts(chi=c.get("chi", 16), chi_x=c.get("chi_x"), prec=c["prec"])
    if c["op"] in ("sample", "amp"):
        s["bits"], s["uniforms"] = _bits_and_uniforms(c["n"], lat.n_qubits, seed)
    if c["op"] == "sample":
        s["log_Z"], _ = h.boundary_contract(s["peps"], s["opts"])
    if c["op"] == "update":
        s["gates"], s["G"] = heisenberg_circuit(lat, 1, 0.1)
        s["messages"] = h.message_buffer(s["peps"])
    return s


def _real(c, *t):
    """Results in the precision of the mode's storage."""
    return [x if c.get("prec", "fp64") == "fp64" else x.to(torch.float32) for x in t]


def _log_z(c, la, ar):
    return np.array([la, ar], dtype=np.float64 if c.get("prec", "fp64") == "fp64" else np.float32)


def run(s):
    c, h = s["c"], s["h"]
    if c["op"] == "stats":
        r = h.sample_stats(s["lq"], s["lp"], s["log_Z"], bits=s["bits"])
        return dict(scalars=np.array([r["log_norm_est"], r["kld"], r["ess"]]), z=r["z_is"])
    if c["op"] == "norm":
        return dict(log_z=_log_z(c, *h.boundary_contract(s["peps"], s["opts"])))
    if c["op"] == "env":
        r = h.environments(s["peps"], s["opts"])
        keys = ("rho1", "zz_h", "zz_v", "p2_h", "p2_v")
        return dict(zip(keys, (r["rho1"] if c["prec"] == "fp64" else r["rho1"].to(torch.complex64),
                               *_real(c, *(r[k] for k in keys[1:])))))
    if c["op"] == "sample":
        bits, lq, lp = h.sample(s["peps"], s["opts"], c["n"], uniforms=s["uniforms"])
        lq, lp = _real(c, lq, lp)
        return dict(bits=bits, log_q=lq, log_p=lp)
    if c["op"] == "amp":
        lp, arg = h.amplitude(s["peps"], s["opts"], s["bits"], want_arg=True)
        # log p and the phase of <x|psi> as a point on the circle
        lp, x, y = _real(c, lp, torch.cos(arg), torch.sin(arg))
        return dict(log_p=lp, cos=x, sin=y)
    if c["op"] == "bp":
        r = h.bp(s["peps"], want_messages=True)
        return dict(log_z=_log_z(c, r["log_abs_Z"], r["arg_Z"]), sweeps=r["sweeps"], eps=r["eps_loops"],
                    messages=r["messages"])
    out, eps, f = h.simple_update(s["peps"], s["gates"], s["G"], messages_out=s["messages"])
    # the new site tensors as one buffer, as a program stores a state
    return dict(sites=torch.cat([t.reshape(-1) for t in out.tensors]), eps=eps, fidelity=f, messages=s["messages"])


# ------------------------------------------------------------------ work

def _bonds(phys, bond_in, chi):
    """Target bonds of a one-site fit (the smaller of chi and the exact ones)."""
    L = len(phys)
    t = []
    for k in range(L - 1):
        left = math.prod(min(p, 1 << 20) for p in phys[:k + 1])
        right = math.prod(min(p, 1 << 20) for p in phys[k + 1:])
        t.append(min(chi, left, right, bond_in[k]))
    for k in range(L - 1):
        t[k] = min(t[k], (t[k - 1] if k else 1) * phys[k])
    for k in range(L - 2, -1, -1):
        t[k] = min(t[k], (t[k + 1] if k + 1 < L - 1 else 1) * phys[k + 1])
    return t


def _ends(b):
    return [1] + list(b), list(b) + [1]


def _set_flops(lat, chi, sweeps=2):
    """(multiply-adds of the boundaries below every row, their bonds per row)."""
    total, below = 0.0, {lat.rows - 1: [1] * (lat.cols - 1)}
    for r in range(lat.rows - 1, 0, -1):
        A = [site_dims(lat, r, k) for k in range(lat.cols)]
        b = below[r]
        t = _bonds([a[1] ** 2 for a in A], [b[k] * A[k][4] ** 2 for k in range(lat.cols - 1)], chi)
        (gl, gr), (yl, yr) = _ends(b), _ends(t)
        for k, (p, u, x, d, y) in enumerate(A):
            part = (yl[k] * gl[k] * x * x * d * d * gr[k] + yl[k] * x * d * gr[k] * x * d * p * u * y
                    + yl[k] * gr[k] * u * y * p * x * d * u * y)
            total += (2 * sweeps + 1) * (part + 2.0 * yl[k] * u * u * gr[k] * y * y * yr[k])
        below[r - 1] = t
    return total, below


def _amp_flops(lat, chi_x, sweeps=2):
    """(multiply-adds of one sample's amplitude boundaries, their bonds above every row)."""
    total, above = 0.0, {0: [1] * (lat.cols - 1)}
    for r in range(lat.rows - 1):
        A = [site_dims(lat, r, k) for k in range(lat.cols)]
        m = above[r]
        t = _bonds([a[3] for a in A], [m[k] * A[k][4] for k in range(lat.cols - 1)], chi_x)
        (al, ar), (yl, yr) = _ends(m), _ends(t)
        for k, (p, u, x, d, y) in enumerate(A):
            total += (2 * sweeps + 1) * (yl[k] * al[k] * x * u * ar[k] + yl[k] * x * u * ar[k] * d * y
                                         + 2.0 * yl[k] * ar[k] * d * y * yr[k])
        above[r + 1] = t
    return total, above


def _double_row_flops(lat, above, below):
    """One pass over every row between the boundaries above and below it."""
    total = 0.0
    for r in range(lat.rows):
        (a, A), (g, G) = _ends(above[r]), _ends(below[r])
        for k in range(lat.cols):
            p, u, x, d, y = site_dims(lat, r, k)
            total += (a[k] * x * x * g[k] * u * u * A[k] + g[k] * A[k] * x * u * u * x * p * d * y
                      + g[k] * A[k] * d * y * p * u * x * d * y + g[k] * A[k] * y * y * d * d * G[k])
    return total


def _sample_row_flops(lat, above, below):
    """One sample's environments over every row: the traced pass from the right,
    one and a half projected passes from the left, each site by the cheaper of
    site by site and (without an up bond) the column's transfer matrix."""
    total = 0.0
    for r in range(lat.rows):
        (a, A), (g, G) = _ends(above[r]), _ends(below[r])
        for k in range(lat.cols):
            p, u, x, d, y = site_dims(lat, r, k)
            for s, times in ((p, 1.0), (1, 1.5)):
                head = a[k] * a[k] * A[k] * g[k] * x * x * u
                one = (a[k] * A[k] * g[k] * x * u * x * s * d * y + a[k] * A[k] * x * s * y * d * g[k] * d * G[k]
                       + a[k] * A[k] * A[k] * x * s * d * G[k] * y * y)
                if u == 1:
                    one = min(one, a[k] * A[k] * (g[k] * x * x * G[k] * y * y + A[k] * G[k] * y * y))
                total += times * (head + one)
    return total


def work(c):
    if c["op"] == "stats":
        n, q = c["n"], c["qubits"]
        return dict(bytes=16.0 * n + n * q + 8 * q, flops=10.0 * n + n * q)
    lat = _lattice(c)
    dims = [site_dims(lat, r, k) for r in range(lat.rows) for k in range(lat.cols)]
    esz = 16 if c["dtype"] == "c128" else 8
    nbytes = float(sum(math.prod(d) for d in dims) * esz)
    N = lat.n_qubits
    if c["op"] == "norm":
        mac = _set_flops(lat, c["chi"])[0]
    elif c["op"] == "env":
        m, below = _set_flops(lat, c["chi"])
        above = {r: below[lat.rows - 1 - r] for r in range(lat.rows)}
        # left, right and four projections; six more per horizontal pair, D^2 wider ones per vertical pair
        mac = 2 * m + (12 + 6 * c["D"] ** 2) * _double_row_flops(lat, above, below)
    elif c["op"] == "sample":
        below = _set_flops(lat, c["chi"])[1]
        m, above = _amp_flops(lat, c["chi_x"])
        mac = c["n"] * (m + _sample_row_flops(lat, above, below))
        nbytes += c["n"] * (N * 9 + 16)
    elif c["op"] == "amp":
        mac = c["n"] * _amp_flops(lat, c["chi_x"])[0]
        nbytes += c["n"] * (N + 16)
    else:
        # a sweep is twelve products per site; some tens of sweeps to 1e-13, one solve per colour group
        sweep = sum(math.prod(d) * (8 * max(d[1:]) + sum(d[1:])) for d in dims)
        mac = 40.0 * sweep
        if c["op"] == "bp":
            mac += 16.0 * c["D"] ** 6 * N / 4
        else:
            mac = 3 * mac + sum(4.0 * (4 * c["D"]) ** 3 for _ in range(N))
            nbytes *= 2
    return dict(bytes=nbytes, flops=8.0 * mac)


# ------------------------------------------------------------------ the values in 64 bits

def _statevector(T):
    """psi[x_0, x_1, ..] over the qubits in row-major order, contracted site by site."""
    cols = len(T[0])
    psi = torch.ones((1,) * (cols + 1), dtype=torch.complex128)[None]  # [x][v_0 .. v_{cols-1}][l]
    for row in T:
        for k, t in enumerate(row):
            A = torch.from_numpy(np.asarray(t, dtype=np.complex128))     # [p][u][l][d][r]
            psi = psi.movedim(1 + k, -1)                                 # [x][others][l][u]
            rest = psi.shape[1:-2]
            p, u, x, d, y = A.shape
            m = psi.reshape(-1, x * u) @ A.permute(2, 1, 0, 3, 4).reshape(x * u, p * d * y)
            m = m.reshape(psi.shape[0], -1, p, d, y).permute(0, 2, 1, 3, 4)
            psi = m.reshape((psi.shape[0] * p,) + rest + (d, y)).movedim(-2, 1 + k)
    return psi.reshape(-1)


def _exact_sample(T, u):
    """Sequential draw with the given uniforms: bits, log q, log p."""
    psi = _statevector(T)
    nq = int(round(math.log2(psi.numel())))
    p = [(psi.abs() ** 2)]
    for _ in range(nq):
        p.append(p[-1].reshape(-1, 2).sum(1))  # marginals of the leading qubits
    p = p[::-1]
    idx = torch.zeros(u.shape[0], dtype=torch.int64)
    bits = torch.zeros(u.shape, dtype=torch.uint8)
    lq = torch.zeros(u.shape[0], dtype=torch.float64)
    for q in range(nq):
        p0, p1 = p[q + 1][2 * idx], p[q + 1][2 * idx + 1]
        b = (u[:, q] >= p0 / (p0 + p1)).to(torch.int64)
        lq += torch.log(torch.where(b == 0, p0, p1) / (p0 + p1))
        bits[:, q] = b.to(torch.uint8)
        idx = 2 * idx + b
    return bits, lq, torch.log(p[-1][idx])


def _is_exact(c, lat):
    """Whether no bond of the case is truncated: chi reaches every exact bond."""
    if lat.n_qubits > 16 or c["op"] in ("bp", "update"):
        return False
    full, below = _set_flops(lat, 1 << 30)
    return all(max(b, default=1) <= c.get("chi", 1 << 30) for b in below.values()) and \
        c.get("chi_x", 1 << 30) >= c["D"] ** min(lat.rows, lat.cols)


def _exact_bp(T):
    """(log|Z_BP|, arg, messages [site][leg][Dm][Dm]) by parallel sweeps to convergence."""
    rows, cols = len(T), len(T[0])
    step = {1: (-1, 0), 2: (0, -1), 3: (1, 0), 4: (0, 1)}
    opp = {1: 3, 2: 4, 3: 1, 4: 2}
    A = {(r, k): np.asarray(T[r][k], dtype=np.complex128) for r in range(rows) for k in range(cols)}
    msg = {}
    for v, a in A.items():
        for leg in step:
            D = a.shape[leg]
            msg[v, leg] = np.eye(D, dtype=np.complex128) / math.sqrt(D)

    def sent(v, leg):
        a = A[v]
        t = a
        for x in step:
            if x != leg:
                t = np.moveaxis(np.tensordot(t, msg[v, x], ([x], [0])), -1, x)
        axes = [x for x in range(5) if x != leg]
        return np.tensordot(t, a.conj(), (axes, axes))

    for _ in range(2000):
        new, change = dict(msg), 0.0
        for v, a in A.items():
            for leg, (dr, dk) in step.items():
                if a.shape[leg] == 1:
                    continue
                m = sent(v, leg)
                m = (m + m.conj().T) / 2
                m /= np.linalg.norm(m)
                w = (v[0] + dr, v[1] + dk)
                change = max(change, np.abs(m - msg[w, opp[leg]]).max())
                new[w, opp[leg]] = m
        msg = new
        if change < 1e-15:
            break
    la = ar = 0.0
    for v, a in A.items():
        z = np.sum(sent(v, 4) * msg[v, 4])
        for leg in (3, 4):
            if a.shape[leg] > 1:
                w = (v[0] + step[leg][0], v[1] + step[leg][1])
                z /= np.sum(msg[v, leg] * msg[w, opp[leg]])
        la += math.log(abs(z))
        ar += math.atan2(z.imag, z.real)
    dm = max(max(a.shape[1:]) for a in A.values())
    out = np.zeros((rows * cols, 4, dm, dm), dtype=np.complex128)
    for (v, leg), m in msg.items():
        out[v[0] * cols + v[1], leg - 1, :m.shape[0], :m.shape[1]] = m
    return la, math.remainder(ar, 2 * math.pi), out


def exact(c, seed):
    """The results in 64 bits where plain tensor algebra reaches them: the metrics,
    states of at most 16 qubits whose bonds are not truncated, and BP's fixed point.
    A truncated boundary is defined by its fit, so it has no other value."""
    if c["op"] == "stats":
        bits, _ = _bits_and_uniforms(c["n"], c["qubits"], seed)
        lq, lp = (x.cpu().numpy().astype(np.longdouble) for x in _log_weights(c["n"], seed))
        w = np.exp(lp - lq - (lp - lq).max())
        ln = (lp - lq).max() + np.log(w.mean())
        kld = (lq - lp).mean() + np.longdouble(-5.0)
        x = 1 - 2 * bits.cpu().numpy().astype(np.float64)
        z = (w[:, None] * x).sum(0) / w.sum()
        return dict(scalars=np.array([ln, kld, w.sum() ** 2 / (w * w).sum()], dtype=np.float64),
                    z=torch.from_numpy(z.astype(np.float64)))
    lat, T = _host_state(c, seed)
    if c["op"] == "bp":
        if lat.rows * lat.cols > 64 and c["lattice"] != "brick":
            return None
        la, ar, msg = _exact_bp(T)
        return dict(log_z=_log_z({}, la, ar), sweeps=None, eps=None, messages=torch.from_numpy(msg))
    if c["op"] not in ("norm", "sample", "amp") or not _is_exact(c, lat):
        return None
    if c["op"] == "norm":
        return dict(log_z=_log_z({}, math.log(float((_statevector(T).abs() ** 2).sum())), 0.0))
    bits, u = _bits_and_uniforms(c["n"], lat.n_qubits, seed)
    if c["op"] == "sample":
        b, lq, lp = _exact_sample(T, u.cpu())
        return dict(bits=b, log_q=lq, log_p=lp)
    a = _statevector(T)
    place = (1 << torch.arange(lat.n_qubits - 1, -1, -1)).to(torch.int64)
    a = a[(bits.cpu().to(torch.int64) * place).sum(1)]
    return dict(log_p=2 * torch.log(a.abs()), cos=a.real / a.abs(), sin=a.imag / a.abs())
