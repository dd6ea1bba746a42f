"""Timed cases of the reconstruction path through its public entry points.

``listed()`` names the cases, ``draw`` gives further ones of the same ranges,
``prepare`` makes what a program holds before the call (device inputs, output
and workspace buffers), ``run`` is one pass, ``work`` the bytes and operations
a pass cannot do without and ``exact`` its result in plain FP64 torch/numpy.

Cut maps are chains (subcircuit c measures the cuts of bond c and is
initialised by those of bond c - 1), as in the runtime study of the paper:
subcircuit outputs are random numbers, the identity row of every entry tensor
spread over many decades, the other rows that row times Uniform[-1, 1).
"""
import math

import numpy as np
import torch

import paper_2205_05836_amd as cq

DEV = "cuda:0"


def listed():
    return [
        # the smallest circuit that is cut: 8 qubits, one wire cut; a call is all latency
        {"name": "fd_8q_fp64", "kind": "fd", "bonds": "1", "outs": "4,4", "prec": "fp64", "perm": True},
        # the 20-qubit circuit cut in two by four wire cuts, in uncut-qubit order
        {"name": "fd_20q_fp32", "kind": "fd", "bonds": "4", "outs": "10,10", "prec": "fp32", "perm": True},
        # an ordinary uneven chain with scaled 16-bit operands
        {"name": "fd_25q_fp16_split", "kind": "fd", "bonds": "3,2", "outs": "9,7,9", "prec": "fp16_split",
         "perm": False},
        # the 30-qubit benchmark chain (two bonds of four cuts) in its headline, single and double forms
        {"name": "fd_30q_bf16_split", "kind": "fd", "bonds": "4,4", "outs": "10,10,10", "prec": "bf16_split",
         "perm": False},
        {"name": "fd_30q_fp32", "kind": "fd", "bonds": "4,4", "outs": "10,10,10", "prec": "fp32", "perm": False},
        {"name": "fd_30q_fp64", "kind": "fd", "bonds": "4,4", "outs": "10,10,10", "prec": "fp64", "perm": False},
        # one small dynamic-definition query, waited for by the program that reads its records
        {"name": "dd_1x3_fp64", "kind": "dd", "bonds": "2,2", "n_inst": 1, "n_out": 12, "active": 5, "R": 4,
         "prec": "fp64"},
        # the batched dynamic definition: 16 instances of four 20-output subcircuits, 2^32 bins a recursion
        {"name": "dd_16x4_fp32", "kind": "dd", "bonds": "2,1,2", "n_inst": 16, "n_out": 20, "active": 8, "R": 4,
         "prec": "fp32"},
        # attribution of the benchmark chain's middle subcircuit (four initialised, four measured cut ends)
        {"name": "attr_14w_4i4m", "kind": "attr", "width": 14, "r": 4, "o": 4, "spread": False},
        # every variant of a 22-slot subcircuit of the dynamic-definition size
        {"name": "variants_22w_2i2m", "kind": "variants", "width": 22, "r": 2, "o": 2, "layers": 8, "spread": False},
        # ground truth of an uncut circuit, the size of the benchmark chain
        {"name": "sim_30q", "kind": "sim", "n": 30, "layers": 8},
        # a QPU run of every variant of a 22-slot subcircuit with a few thousand shots, scored by Eq. 3
        {"name": "shots_144x4m", "kind": "shots", "rows": 144, "cols": 1 << 22, "shots": 8192},
    ]


def _ints(text):
    return [int(x) for x in text.split(",")]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["fd", "fd", "fd", "fd", "dd", "dd", "attr", "attr", "variants", "sim", "shots", "shots"])
    while True:
        c = _draw(rng, kind)
        if c is not None:
            return c


def _draw(rng, kind):
    if kind == "fd":
        ns = rng.choice([2, 3, 3, 4])
        n = rng.randint(6, 30)
        cutsp = sorted(rng.sample(range(1, n), ns - 1))
        outs = [b - a for a, b in zip([0] + cutsp, cutsp + [n])]
        bonds = [rng.randint(1, 4) for _ in range(ns - 1)]
        ks = _ks(bonds)
        # a subcircuit has at least as many outputs as arriving cuts, and entries of at most 1 GiB
        if any(b > o for b, o in zip(bonds, outs[1:])) or sum(bonds) > 8:
            return None
        if any(2 * k + o > 27 for k, o in zip(ks, outs)):
            return None
        case = {"kind": "fd", "bonds": ",".join(map(str, bonds)), "outs": ",".join(map(str, outs)),
                "prec": rng.choice(["fp64", "fp32", "bf16_split", "fp16_split", "bf16", "fp16"]),
                "perm": rng.random() < 0.4 and n <= 26}
        return case if work(case)["flops"] <= 7e11 else None
    if kind == "dd":
        ns = rng.randint(2, 4)
        bonds = [rng.randint(1, 2) for _ in range(ns - 1)]
        n_out = rng.randint(6, 20)
        active = rng.randint(2, min(8, n_out - 1))
        case = {"kind": "dd", "bonds": ",".join(map(str, bonds)), "n_inst": _log_int(rng, 1, 16), "n_out": n_out,
                "active": active, "R": rng.randint(2, 6), "prec": rng.choice(["fp64", "fp32", "fp32", "bf16_split"])}
        return case if work(case)["bytes"] <= 2e10 else None
    if kind in ("attr", "variants"):
        most = 4 if kind == "attr" else 3
        r, o, w = rng.randint(0, most), rng.randint(0, most), rng.randint(4, 22)
        if r + o == 0 or o + r > w:
            return None
        case = {"kind": kind, "width": w, "r": r, "o": o, "spread": rng.random() < 0.5}
        if kind == "variants":
            case["layers"] = rng.randint(2, 8)
        return case if work(case)["bytes"] <= 3.5e9 else None
    if kind == "sim":
        return {"kind": "sim", "n": rng.randint(4, 28), "layers": rng.randint(2, 10)}
    rows, cols = _log_int(rng, 1, 4096), _log_int(rng, 16, 1 << 22)
    shots = _log_int(rng, 100, 1000000)
    if rows * cols > 144 << 22 or rows * shots > 1 << 27:
        return None
    return {"kind": "shots", "rows": rows, "cols": cols, "shots": shots}


# -- cut maps, circuits and inputs ------------------------------------------

def _ks(bonds):
    return [(bonds[c - 1] if c else 0) + (bonds[c] if c < len(bonds) else 0) for c in range(len(bonds) + 1)]


def _chain(bonds, outs):
    """(width, init_cut, meas_cut) per subcircuit of a chain."""
    subs, first = [], [0]
    for b in bonds:
        first.append(first[-1] + b)
    for c, n in enumerate(outs):
        left, right = (bonds[c - 1] if c else 0), (bonds[c] if c < len(bonds) else 0)
        init, meas = [-1] * (n + right), [-1] * (n + right)
        for j in range(left):
            init[j] = first[c - 1] + j
        for j in range(right):
            meas[n + j] = first[c] + j
        subs.append((n + right, init, meas))
    return subs


def _sub(case):
    """One subcircuit with r initialised and o measured slots: at the two ends
    of the register, or spread over it."""
    w, r, o = case["width"], case["r"], case["o"]
    init, meas = [-1] * w, [-1] * w
    for t in range(r):
        init[t * w // r if case["spread"] else t] = t
    for u in range(o):
        meas[u * w // o + (w // o - 1) if case["spread"] else w - o + u] = r + u
    return w, init, meas


def _gen(*key):
    g = torch.Generator(device=DEV)
    x = 0x9E3779B97F4A7C15
    for k in key:
        x = ((x ^ int(k)) * 0xBF58476D1CE4E5B9 + 0x94D049BB133111EB) % (1 << 62)
    g.manual_seed(x)
    return g


def _rand(shape, gen):
    return torch.rand(shape, dtype=torch.float64, device=DEV, generator=gen)


def _entries(seed, inst, c, k, n):
    """(4^k, 2^n): the identity row like a sparse Dirichlet draw, the other
    rows that row times Uniform[-1, 1)."""
    g = _gen(seed, inst, c)
    row = -torch.log1p(-_rand((1 << n,), g)) * _rand((1 << n,), g) ** 10
    row /= row.sum()
    e = _rand((4 ** k, 1 << n), g).mul_(2.0).sub_(1.0)
    e[0] = 1.0
    return e.mul_(row)


def _haar(rng):
    z = rng.standard_normal((2, 2)) + 1j * rng.standard_normal((2, 2))
    q, r = np.linalg.qr(z)
    return q * (np.diagonal(r) / np.abs(np.diagonal(r)))


def _brickwork(n, layers, seed):
    """Layers of Haar-random one-qubit unitaries and CZs on alternating pairs."""
    rng = np.random.default_rng([seed, n, layers])
    ops = []
    for t in range(layers):
        ops += [("u", q, _haar(rng)) for q in range(n)]
        ops += [("cz", i, i + 1) for i in range(t % 2, n - 1, 2)]
    return ops


def _rows(shape, gen):
    """Rows of outcome probabilities of a random circuit (exponential, sum 1)."""
    p = torch.log1p(_rand(shape, gen).neg_()).neg_()
    return p.div_(p.sum(-1, keepdim=True))


def _perm(case, seed, n):
    return [int(q) for q in np.random.default_rng([seed, 77]).permutation(n)] if case["perm"] else None


def _empty(n, dtype=torch.uint8):
    return torch.empty(max(int(n), 1), dtype=dtype, device=DEV)


def _inputs(case, seed):
    kind = case["kind"]
    if kind == "fd":
        bonds, outs = _ints(case["bonds"]), _ints(case["outs"])
        return [_entries(seed, 0, c, k, n) for c, (k, n) in enumerate(zip(_ks(bonds), outs))]
    if kind == "dd":
        ks = _ks(_ints(case["bonds"]))
        return [[_entries(seed, i, c, k, case["n_out"]) for c, k in enumerate(ks)] for i in range(case["n_inst"])]
    if kind == "attr":
        return _rows((4 ** case["r"], 3 ** case["o"], 1 << case["width"]), _gen(seed, 1))
    if kind == "variants":
        return _brickwork(case["width"], case["layers"], seed)
    if kind == "sim":
        return _brickwork(case["n"], case["layers"], seed)
    return _rows((case["rows"], case["cols"]), _gen(seed, 2))


def prepare(case, seed):
    kind, x = case["kind"], _inputs(case, seed)
    s = {"case": case, "x": x}
    if kind == "fd":
        subs, prec = _chain(_ints(case["bonds"]), _ints(case["outs"])), case["prec"]
        n = sum(_ints(case["outs"]))
        perm = _perm(case, seed, n)
        s |= {"subs": subs, "perm": perm, "ws": _empty(cq.cq_fd_workspace_size(subs, prec, perm)),
              "out": _empty(2 ** n, torch.float64 if prec == "fp64" else torch.float32)}
    elif kind == "dd":
        bonds, n, a = _ints(case["bonds"]), case["n_out"], case["active"]
        subs = _chain(bonds, [n] * (len(bonds) + 1))
        ns = len(subs)
        s["inst"] = [dict(subs=subs, entries=e, active=[(1 << a) - 1] * ns,
                          merged=[((1 << n) - 1) ^ ((1 << a) - 1)] * ns, max_active=[a] * ns) for e in x]
        s["ws"] = _empty(cq.cq_dd_workspace_size(s["inst"], case["prec"], case["R"]))
    elif kind == "attr":
        sub = _sub(case)
        s |= {"sub": sub, "ws": _empty(cq.cq_attribute_workspace_size(sub)),
              "out": _empty(4 ** (case["r"] + case["o"]) << (case["width"] - case["o"]), torch.float64).view(
                  4 ** (case["r"] + case["o"]), -1)}
    elif kind == "variants":
        sub = _sub(case)
        shape = (4 ** case["r"], 3 ** case["o"], 1 << case["width"])
        s |= {"sub": sub, "ws": _empty(cq.cq_variants_workspace_size(sub)),
              "out": torch.empty(shape, dtype=torch.float64, device=DEV)}
    elif kind == "sim":
        s |= {"ws": _empty(cq.cq_simulate_workspace_size(case["n"])), "out": _empty(1 << case["n"], torch.float64)}
    else:
        s |= {"seed": seed, "out": torch.empty_like(x), "chi": _empty(1, torch.float64),
              "ws": _empty(cq.cq_sample_shots_workspace_size(case["rows"], case["cols"], case["shots"])),
              "cws": _empty(cq.cq_chi2_workspace_size())}
    return s


# -- one pass -----------------------------------------------------------------

def _dd_arrays(recs, R, ns):
    """The records of a batch as arrays (zeros where a run stopped early)."""
    m = len(recs)
    a = {"total": np.zeros((m, R)), "value": np.zeros((m, R, R)), "bin": np.zeros((m, R, R), np.int64),
         "rec": np.zeros((m, R, R), np.int64), "masks": np.zeros((m, R, 4, ns), np.int64)}
    for i, rows in enumerate(recs):
        for j, rc in enumerate(rows):
            a["total"][i, j] = rc["total"]
            for t, (v, r, b) in enumerate(rc["list"]):
                a["value"][i, j, t], a["rec"][i, j, t], a["bin"][i, j, t] = v, r, b
            a["masks"][i, j] = (rc["active"], rc["merged"], rc["fixed"], rc["fixed_vals"])
    return a


def run(s):
    c, kind = s["case"], s["case"]["kind"]
    if kind == "fd":
        return cq.cq_reconstruct_fd(s["subs"], s["x"], prec=c["prec"], out_perm=s["perm"], out=s["out"],
                                    workspace=s["ws"])
    if kind == "dd":
        recs, _ = cq.cq_reconstruct_dd(s["inst"], prec=c["prec"], R=c["R"], workspace=s["ws"])
        return _dd_arrays(recs, c["R"], len(s["inst"][0]["subs"]))
    if kind == "attr":
        return cq.cq_attribute(s["sub"], s["x"], entries=s["out"], workspace=s["ws"])
    if kind == "variants":
        return cq.cq_variant_probabilities(s["sub"], s["x"], out=s["out"], workspace=s["ws"])
    if kind == "sim":
        return cq.cq_simulate_probabilities(c["n"], s["x"], out=s["out"], workspace=s["ws"])
    f = cq.cq_sample_shots(s["x"], c["shots"], s["seed"], out=s["out"], workspace=s["ws"])
    return {"freq": f, "chi2": cq.cq_chi2(f, s["x"], out=s["chi"], workspace=s["cws"])}


# -- what a pass cannot do without ------------------------------------------

def _chain_flops(bonds, outs):
    """Fewest operations of a pairwise contraction of the chain."""
    n = len(outs)
    edge = [0] + list(bonds) + [0]
    best = {(i, i): 0.0 for i in range(n)}
    for size in range(2, n + 1):
        for i in range(n - size + 1):
            j = i + size - 1
            step = 2.0 * 4.0 ** (edge[i] + edge[j + 1]) * 2.0 ** sum(outs[i:j + 1])
            best[i, j] = min(best[i, m] + best[m + 1, j] + step * 4.0 ** edge[m + 1] for m in range(i, j))
    return best[0, n - 1]


def work(case):
    kind = case["kind"]
    if kind == "fd":
        bonds, outs = _ints(case["bonds"]), _ints(case["outs"])
        entries = sum(8.0 * 4 ** k * 2 ** n for k, n in zip(_ks(bonds), outs))
        return {"bytes": entries + 2.0 ** sum(outs) * (8 if case["prec"] == "fp64" else 4),
                "flops": _chain_flops(bonds, outs)}
    if kind == "dd":
        elems = case["n_inst"] * sum(4.0 ** k * 2 ** case["n_out"] for k in _ks(_ints(case["bonds"])))
        return {"bytes": 8.0 * elems, "flops": elems}
    if kind in ("attr", "variants"):
        r, o, w = case["r"], case["o"], case["width"]
        table = 8.0 * 4 ** r * 3 ** o * 2 ** w
        if kind == "attr":
            entries = 8.0 * 4 ** (r + o) * 2 ** (w - o)
            return {"bytes": table + entries, "flops": (table + entries) / 8}
        return {"bytes": table, "flops": 2.0 ** r * case["layers"] * w * 14.0 * 2 ** w}
    if kind == "sim":
        return {"bytes": 8.0 * 2 ** case["n"], "flops": case["layers"] * case["n"] * 14.0 * 2 ** case["n"]}
    return {"bytes": 32.0 * case["rows"] * case["cols"], "flops": 4.0 * case["rows"] * case["cols"]}


# -- the same in plain FP64 ---------------------------------------------------

def _contract(bonds, ents):
    """2^-K times the chain contraction of the entries, 2^n FP64 values."""
    t = ents[0].t()  # (outputs so far, labels of the open bond)
    for c, b in enumerate(bonds):
        e = ents[c + 1]
        nb = 4 ** bonds[c + 1] if c + 1 < len(bonds) else 1
        t = t @ e.reshape(4 ** b, -1)  # (outs, right labels x new outputs)
        t = t.reshape(t.shape[0], nb, -1).permute(0, 2, 1).reshape(-1, nb)
    return t.reshape(-1) * 2.0 ** -sum(bonds)


def _to_uncut_order(p, perm):
    n = len(perm)
    x = torch.arange(1 << n, dtype=torch.int64, device=DEV)
    src = torch.zeros_like(x)
    for i, q in enumerate(perm):
        src |= ((x >> (n - 1 - q)) & 1) << (n - 1 - i)
    return p[src]


def _apply_u(psi, n, q, u):
    x = psi.view(1 << q, 2, -1)
    new = torch.empty_like(x)
    for i in range(2):
        torch.mul(x[:, 0], complex(u[i][0]), out=new[:, i])
        new[:, i].add_(x[:, 1], alpha=complex(u[i][1]))
    return new.view(-1)


def _simulate(psi, n, ops):
    for op in ops:
        if op[0] == "u":
            psi = _apply_u(psi, n, op[1], op[2])
        else:
            a, b = sorted(op[1:3])
            psi.view(1 << a, 2, 1 << (b - a - 1), 2, -1)[:, 1, :, 1].neg_()
    return psi


_H = [[2.0 ** -0.5, 2.0 ** -0.5], [2.0 ** -0.5, -(2.0 ** -0.5)]]
_HSD = [[2.0 ** -0.5, -1j * 2.0 ** -0.5], [2.0 ** -0.5, 1j * 2.0 ** -0.5]]
_KETS = [(1, 0), (0, 1), (2.0 ** -0.5, 2.0 ** -0.5), (2.0 ** -0.5, 1j * 2.0 ** -0.5)]


def _exact_variants(case, ops):
    w, init, meas = _sub(case)
    islots, mslots = [q for q in range(w) if init[q] >= 0], [q for q in range(w) if meas[q] >= 0]
    out = torch.empty((4 ** case["r"], 3 ** case["o"], 1 << w), dtype=torch.float64, device=DEV)
    for j in range(4 ** case["r"]):
        psi = torch.ones(1, dtype=torch.complex128, device=DEV)
        for q in range(w):
            d = (j >> (2 * (len(islots) - 1 - islots.index(q)))) & 3 if q in islots else 0
            psi = (psi[:, None] * torch.tensor(_KETS[d], dtype=torch.complex128, device=DEV)).reshape(-1)
        psi = _simulate(psi, w, ops)
        for b in range(3 ** case["o"]):
            v = psi
            for u, q in enumerate(mslots):
                d = b // 3 ** (len(mslots) - 1 - u) % 3
                if d:
                    v = _apply_u(v, w, q, _H if d == 1 else _HSD)
            out[j, b] = v.real ** 2 + v.imag ** 2
    return out


def _exact_attr(case, v):
    w, _, meas = _sub(case)
    r, o = case["r"], case["o"]
    n = w - o
    mslots = [q for q in range(w) if meas[q] >= 0]
    order = [q for q in range(w) if meas[q] < 0] + mslots
    v = v.view([-1] + [2] * w).permute([0] + [1 + q for q in order]).reshape(4 ** r, 3 ** o, 1 << n, 1 << o)
    for u in range(o):  # measured slot u: basis digit and outcome bit -> label digit (I, X, Y, Z)
        rest = o - 1 - u
        v = v.reshape(-1, 3, 3 ** rest, 1 << n, 2, 1 << rest)
        s, d = v.sum(4), v[:, :, :, :, 0] - v[:, :, :, :, 1]
        v = torch.stack([s[:, 0], d[:, 1], d[:, 2], d[:, 0]], 1)
    for t in range(r):  # initialised slot t: prepared state -> label digit
        v = v.reshape(4 ** t, 4, -1)
        a, b, p, i = v[:, 0], v[:, 1], v[:, 2], v[:, 3]
        v = torch.stack([a + b, 2 * p - a - b, 2 * i - a - b, a - b], 1)
    return v.reshape(4 ** (r + o), 1 << n)


def _mul32(a, b):
    """Low and high 32 bits of the product of two 32-bit values (int64)."""
    al, ah, bl, bh = a & 0xffff, a >> 16, b & 0xffff, b >> 16
    mid = al * bh + ((al * bl) >> 16)
    low = (mid & 0xffff) + ah * bl
    return ((low & 0xffff) << 16) | ((al * bl) & 0xffff), ah * bh + (mid >> 16) + (low >> 16)


def _exact_shots(case, p, seed):
    """Counts of the integer sampling rule (Philox4x32-10, 2^52 quantisation)."""
    rows, cols, shots = case["rows"], case["cols"], case["shots"]
    out = torch.zeros_like(p)
    s = torch.arange(shots, dtype=torch.int64, device=DEV)
    for r in range(rows):
        c = (p[r].clamp(0, 1) * 2.0 ** 52).to(torch.int64).cumsum(0)
        w, k = [s, torch.zeros_like(s), torch.full_like(s, r), torch.zeros_like(s)], [seed & 0xffffffff, seed >> 32]
        for _ in range(10):
            (l0, h0), (l2, h2) = _mul32(w[0], 0xD2511F53), _mul32(w[2], 0xCD9E8D57)
            w = [h2 ^ w[1] ^ k[0], l2, h0 ^ w[3] ^ k[1], l0]
            k = [(k[0] + 0x9E3779B9) & 0xffffffff, (k[1] + 0xBB67AE85) & 0xffffffff]
        tot = c[-1]  # below 2^53: t = floor((w0 + 2^32 w1) tot / 2^64)
        t0, t1 = tot & 0xffffffff, tot >> 32
        (_, h00), (l01, h01), (l10, h10), (l11, h11) = (_mul32(w[0], t0), _mul32(w[0], t1), _mul32(w[1], t0),
                                                        _mul32(w[1], t1))
        t = ((h00 + l01 + l10) >> 32) + h01 + h10 + l11 + (h11 << 32)
        hit = torch.searchsorted(c, t, right=True)
        out[r] = torch.bincount(hit, minlength=cols).to(torch.float64) / shots
    return out


def _exact_dd(case, ents):
    """Algorithm 1 on one instance, every bin in FP64: totals and list values."""
    bonds, n, R, amax = _ints(case["bonds"]), case["n_out"], case["R"], case["active"]
    ns, full = len(bonds) + 1, (1 << n) - 1
    total, value = np.zeros(R), np.zeros((R, R))
    act, fixed, vals, todo = [(1 << amax) - 1] * ns, [0] * ns, [0] * ns, []
    for r in range(R):
        red, merged = [], [full ^ a ^ f for a, f in zip(act, fixed)]
        for c in range(ns):  # bit i of a mask is output i, output 0 the most significant axis
            e, ax = ents[c].view([-1] + [2] * n), 1
            for i in range(n):
                if fixed[c] >> i & 1:
                    e = e.select(ax, vals[c] >> i & 1)
                elif merged[c] >> i & 1:
                    e = e.sum(ax)
                else:
                    ax += 1
            red.append(e.reshape(ents[c].shape[0], -1))
        p = _contract(bonds, red)
        total[r] = float(p.sum())
        if any(merged):
            top = torch.topk(p, min(R, p.numel()))
            todo += [(float(v), r, int(b), list(act), list(fixed), list(vals)) for v, b in zip(*top)]
            todo = sorted(todo, key=lambda e: (-e[0], e[1], e[2]))[:R]
        for t, e in enumerate(todo):
            value[r, t] = e[0]
        if not todo:
            break
        _, _, b, act, fixed, vals = todo.pop(0)
        act, fixed, vals = list(act), list(fixed), list(vals)
        for c in reversed(range(ns)):
            for i in reversed(range(n)):
                if act[c] >> i & 1:
                    vals[c] |= (b & 1) << i
                    b >>= 1
            fixed[c] |= act[c]
            left = [i for i in range(n) if not fixed[c] >> i & 1][:amax]
            act[c] = sum(1 << i for i in left)
    return total, value


def exact(case, seed):
    kind = case["kind"]
    if kind == "dd":
        ns = len(_ints(case["bonds"])) + 1
        # the bins of a recursion have to fit; 16-bit bins choose their own candidates
        if case["active"] * ns > 24 or case["n_out"] > 20 or case["prec"] == "bf16_split":
            return None
        got = [_exact_dd(case, e) for e in _inputs(case, seed)]
        return {"total": np.stack([t for t, _ in got]), "value": np.stack([v for _, v in got]), "bin": None,
                "rec": None, "masks": None}
    x = _inputs(case, seed)
    if kind == "fd":
        p = _contract(_ints(case["bonds"]), x)
        perm = _perm(case, seed, sum(_ints(case["outs"])))
        return p if perm is None else _to_uncut_order(p, perm)
    if kind == "attr":
        return _exact_attr(case, x)
    if kind == "variants":
        return _exact_variants(case, x)
    if kind == "sim":
        psi = torch.zeros(1 << case["n"], dtype=torch.complex128, device=DEV)
        psi[0] = 1.0
        psi = _simulate(psi, case["n"], x)
        return torch.view_as_real(psi).square_().sum(-1)
    f = _exact_shots(case, x, seed)
    d, t = f - x, f + x
    return {"freq": f, "chi2": torch.where(t != 0, d * d / t, torch.zeros_like(t)).sum().reshape(1)}
