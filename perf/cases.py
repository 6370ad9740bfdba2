"""Performance cases of the channelwise Clebsch-Gordan convolution library.

Each case is one call sequence that a force-field or simulation program makes,
through the Python binding, on inputs made from a seed:

  conv     convolution forward and backward (a layer's training or force step);
           with "rebuild" the graph is built inside the pass, as in a simulation
           whose neighbour list has just changed
  conv64   the same in float64
  radial   forward and backward with the radial weights formed in the kernels
  bwd2     the double backward (training on forces)
  tp       the standalone weighted tensor product, forward and backward
  records  the tensor product with caller-supplied records and a second operand
           per channel, forward and backward
  linear   equivariant linear mixing, forward and backward

Graphs are periodic boxes of rigid water molecules at liquid density with a
cutoff near 5 A (about 52 neighbours), or small open clusters.
"""
from __future__ import annotations

import math
from fractions import Fraction
from functools import lru_cache

import numpy as np
import torch

from paper_2609_35099_amd import e3mi

MOL_PER_A3 = 0.033428    # liquid water
R_CUT = 5.0
CLUSTER_PER_A3 = 0.1     # open clusters: atoms per cubic Angstrom
CLUSTER_CUT = 4.0
K_BESSEL = 8


def listed():
    return [
        # the smallest call: a 64-atom molecule with few channels, where launches and latency count
        {"name": "conv_cluster64_c8", "op": "conv", "blocks": "0e+1o", "C": 8, "lsh": 2, "lout": 2,
         "natural": False, "atoms": 64, "mols": 0, "pad": 0.0, "rebuild": False},
        # one step of a small simulation: a 1,503-atom water box, 10% padding edges, new neighbour list
        {"name": "md_1503_c128", "op": "conv", "blocks": "0e+1o", "C": 128, "lsh": 3, "lout": 3,
         "natural": False, "atoms": 0, "mols": 501, "pad": 0.1, "rebuild": True},
        # a light model (32 channels, l <= 2) on a mid-sized box
        {"name": "conv_9999_c32", "op": "conv", "blocks": "0e+1o+2e", "C": 32, "lsh": 2, "lout": 2,
         "natural": False, "atoms": 0, "mols": 3333, "pad": 0.0, "rebuild": False},
        # a channel count that is no power of two, natural parities only
        {"name": "conv_5001_c96_natural", "op": "conv", "blocks": "0e+1o+2e+3o", "C": 96, "lsh": 3, "lout": 3,
         "natural": True, "atoms": 0, "mols": 1667, "pad": 0.0, "rebuild": False},
        # the largest: the 24,000-atom benchmark box
        {"name": "conv_24000_c128", "op": "conv", "blocks": "0e+1o+2e+3o", "C": 128, "lsh": 3, "lout": 3,
         "natural": False, "atoms": 0, "mols": 8000, "pad": 0.0, "rebuild": False},
        # a layout without kernels of its own (features of both parities), run block by block
        {"name": "conv_3000_c64_composed", "op": "conv", "blocks": "0e+0o+1o+1e+2e+2o", "C": 64, "lsh": 2, "lout": 2,
         "natural": False, "atoms": 0, "mols": 1000, "pad": 0.0, "rebuild": False},
        # double precision, as accuracy studies and some simulations use it
        {"name": "conv64_1503_c32", "op": "conv64", "blocks": "0e+1o+2e", "C": 32, "lsh": 3, "lout": 3,
         "natural": False, "atoms": 0, "mols": 501, "pad": 0.0, "rebuild": False},
        # radial weights formed in the kernels
        {"name": "radial_6000_c128", "op": "radial", "blocks": "0e+1o+2e+3o", "C": 128, "lsh": 3, "lout": 3,
         "natural": False, "atoms": 0, "mols": 2000, "pad": 0.0, "rebuild": False},
        # training on forces
        {"name": "bwd2_3000_c64", "op": "bwd2", "blocks": "0e+1o+2e", "C": 64, "lsh": 3, "lout": 3,
         "natural": False, "atoms": 0, "mols": 1000, "pad": 0.0, "rebuild": False},
        # the standalone tensor product at its benchmark size
        {"name": "tp_200k_c128", "op": "tp", "blocks": "0e+1o+2e", "C": 128, "lsh": 3, "lout": 3,
         "natural": False, "rows": 200000},
        # product of two feature tensors, all paths of a degree collapsed into one output block
        {"name": "records_30011_c100", "op": "records", "lx": 2, "ly": 2, "lz": 2, "C": 100, "rows": 30011},
        # mixing of the benchmark convolution's output
        {"name": "linear_24000_c128", "op": "linear", "blocks": "0e+1o+2e+3o", "lsh": 3, "lout": 3,
         "natural": False, "C": 128, "C_out": 128, "rows": 24000},
    ]


LAYOUTS = [
    ("0e+1o", 2, 2, False), ("0e+1o+2e", 2, 2, False), ("0e+1o", 3, 3, False), ("0e+1o+2e", 3, 3, False),
    ("0e+1o+2e+3o", 3, 3, False), ("0e+1o+2e", 3, 3, True), ("0e+1o+2e+3o", 3, 3, True),
    # without kernels of their own: a first layer's scalars, both parities, a mixed order
    ("0e", 3, 3, False), ("0e+0o+1o+1e", 2, 2, False), ("2e+0e+1o", 3, 2, True),
]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the ranges the listed ones stand for."""
    op = rng.choice(["conv"] * 8 + ["conv64", "radial", "radial", "bwd2", "bwd2", "tp", "tp", "tp", "records",
                                    "records", "linear", "linear", "linear"])
    if op == "records":
        return {"op": op, "lx": rng.randint(1, 3), "ly": rng.randint(1, 3), "lz": rng.randint(1, 3),
                "C": _log(rng, 4, 160), "rows": _log(rng, 200, 60000)}
    blocks, lsh, lout, natural = rng.choice(LAYOUTS)
    if op == "linear":
        return {"op": op, "blocks": blocks, "lsh": lsh, "lout": lout, "natural": natural,
                "C": 16 * _log(rng, 1, 12), "C_out": 16 * _log(rng, 1, 12), "rows": _log(rng, 64, 20000)}
    C = 4 * _log(rng, 1, 64)
    case = {"op": op, "blocks": blocks, "C": C, "lsh": lsh, "lout": lout, "natural": natural}
    if op == "tp":
        case["rows"] = min(_log(rng, 200, 150000), 150000 * 128 // C)
        return case
    case.update(atoms=0, mols=0, pad=rng.choice([0.0, 0.0, 0.1]), rebuild=op == "conv" and rng.random() < 0.25)
    if rng.random() < 0.2:
        case["atoms"] = _log(rng, 16, 400)
    else:
        case["mols"] = min(_log(rng, 64, 4000), (4000 if op == "conv" else 1200) * 128 // C)
        case["mols"] = max(64, case["mols"])
    return case


# ------------------------------------------------------------ layouts and couplings
def _cg(l1, m1, l2, m2, L, M):
    """<l1 m1 l2 m2 | L M>, Racah's formula."""
    f = math.factorial
    if M != m1 + m2:
        return 0.0
    pre = Fraction((2 * L + 1) * f(L + l1 - l2) * f(L - l1 + l2) * f(l1 + l2 - L), f(l1 + l2 + L + 1))
    pre *= f(L + M) * f(L - M) * f(l1 - m1) * f(l1 + m1) * f(l2 - m2) * f(l2 + m2)
    tot = Fraction(0)
    for k in range(l1 + l2 - L + 1):
        d = (k, l1 + l2 - L - k, l1 - m1 - k, l2 + m2 - k, L - l2 + m1 + k, L - l1 - m2 + k)
        if min(d) >= 0:
            tot += Fraction((-1) ** k, math.prod(f(v) for v in d))
    return math.copysign(math.sqrt(float(pre * tot * tot)), tot)


def _to_real(l):
    """Real harmonics (no Condon-Shortley sign) = U @ complex ones (with it)."""
    U = np.zeros((2 * l + 1, 2 * l + 1), complex)
    U[l, l] = 1
    for m in range(1, l + 1):
        c = (-1) ** m / math.sqrt(2)
        U[l + m, l + m], U[l + m, l - m] = c, 1 / math.sqrt(2)
        U[l - m, l + m], U[l - m, l - m] = -1j * c, 1j / math.sqrt(2)
    return U


@lru_cache(maxsize=None)
def _coupling(l1, l2, l3):
    """Real coupling block [2 l3 + 1, 2 l1 + 1, 2 l2 + 1], first non-zero entry positive."""
    c = np.zeros((2 * l3 + 1, 2 * l1 + 1, 2 * l2 + 1))
    for m1 in range(-l1, l1 + 1):
        for m2 in range(-l2, l2 + 1):
            if abs(m1 + m2) <= l3:
                c[m1 + m2 + l3, m1 + l1, m2 + l2] = _cg(l1, m1, l2, m2, l3, m1 + m2)
    r = np.einsum("MN,Nij,ai,bj->Mab", _to_real(l3), c, _to_real(l1).conj(), _to_real(l2).conj())
    r = r.imag if np.abs(r.imag).max() > np.abs(r.real).max() else r.real
    r = np.where(np.abs(r) < 1e-13, 0.0, r)
    return r * np.sign(r[r != 0][0])


class _Paths:
    """Paths of a layout: x block by x block, then l2, then l3, in output order."""

    def __init__(self, case):
        self.items, self.types, xo, oo = [], [], 0, 0
        for tok in case["blocks"].split("+"):
            l1, p1 = int(tok[0]), 1 if tok[1] == "e" else -1
            for l2 in range(case["lsh"] + 1):
                for l3 in range(abs(l1 - l2), min(l1 + l2, case["lout"]) + 1):
                    p3 = p1 * (-1) ** l2
                    if case["natural"] and p3 != (-1) ** l3:
                        continue
                    self.items.append((slice(xo, xo + 2 * l1 + 1), slice(l2 * l2, (l2 + 1) ** 2),
                                       slice(oo, oo + 2 * l3 + 1), _coupling(l1, l2, l3)))
                    self.types.append("%d%s" % (l3, "e" if p3 > 0 else "o"))
                    oo += 2 * l3 + 1
            xo += 2 * l1 + 1
        self.d_in, self.d_sh, self.d_out, self.n = xo, (case["lsh"] + 1) ** 2, oo, len(self.items)
        self.nnz = sum(int((c != 0).sum()) for *_, c in self.items)
        self.pairs = sum(int((c != 0).any(2).sum()) for *_, c in self.items)


def _irreps(blocks, C):
    return "+".join("%dx%s" % (C, t) for t in blocks.split("+"))


def _harmonics(lmax, v):
    """Component-normalised real harmonics of v / |v|, polar axis y (zeros past l = 0 for a zero vector)."""
    n = v.norm(dim=-1, keepdim=True)
    u = v / torch.where(n > 0, n, torch.ones_like(n))
    y, z, x = u[:, 0], u[:, 1], u[:, 2]
    q = math.sqrt
    rows = [torch.ones_like(x)]
    if lmax >= 1:
        rows += [q(3) * y, q(3) * z, q(3) * x]
    if lmax >= 2:
        rows += [q(15) * x * y, q(15) * y * z, q(5) / 2 * (2 * z * z - x * x - y * y), q(15) * x * z,
                 q(15) / 2 * (x * x - y * y)]
    if lmax >= 3:
        rows += [q(35 / 8) * y * (3 * x * x - y * y), q(105) * x * y * z, q(21 / 8) * y * (4 * z * z - x * x - y * y),
                 q(7) / 2 * z * (2 * z * z - 3 * x * x - 3 * y * y), q(21 / 8) * x * (4 * z * z - x * x - y * y),
                 q(105) / 2 * z * (x * x - y * y), q(35 / 8) * x * (x * x - 3 * y * y)]
    return torch.stack(rows, -1)


# ------------------------------------------------------------ inputs
def _positions(case, rng):
    """Atom positions and the box side (0: open)."""
    if case["atoms"]:
        side = (case["atoms"] / CLUSTER_PER_A3) ** (1 / 3)
        return rng.uniform(0, side, (case["atoms"], 3)), 0.0
    n = case["mols"]
    side, k = (n / MOL_PER_A3) ** (1 / 3), math.ceil(round(n ** (1 / 3), 9))
    site = np.sort(rng.permutation(k ** 3)[:n])
    o = (np.stack([site // (k * k), site // k % k, site % k], 1) + rng.uniform(0.35, 0.65, (n, 3))) * (side / k)
    a = rng.standard_normal((n, 3))
    b = np.cross(a, rng.standard_normal((n, 3)))
    a, b = (v / np.linalg.norm(v, axis=1, keepdims=True) for v in (a, b))
    t = math.radians(104.52)
    h1, h2 = o + 0.9572 * a, o + 0.9572 * (math.cos(t) * a + math.sin(t) * b)
    pos = np.stack([o, h1, h2], 1)[rng.permutation(n)].reshape(-1, 3)
    return pos % side, side


def _edges(case, seed):
    """(sender, receiver, vec, number of nodes, padding node or -1), edges in receiver order.

    The cutoff is set so that every seed's graph has the same number of edges:
    the closest pairs are taken."""
    p, side = _positions(case, np.random.default_rng(seed))
    pos, reach = torch.from_numpy(p).cuda().float(), 1.1 * R_CUT if side else math.inf
    snd, rcv, vec = [], [], []
    for r0 in range(0, len(pos), 2048):
        d = pos[r0:r0 + 2048, None] - pos[None]
        if side:
            d -= side * (d / side).round()
        r2 = (d * d).sum(-1)
        i, j = ((r2 < reach * reach) & (r2 > 0)).nonzero(as_tuple=True)
        rcv.append(i + r0), snd.append(j), vec.append(d[i, j])
    snd, rcv, vec, n, pad = torch.cat(snd).int(), torch.cat(rcv).int(), torch.cat(vec), len(pos), -1
    near = (vec * vec).sum(-1).sort(stable=True).indices[:_n_edges(case)].sort().values
    snd, rcv, vec = snd[near], rcv[near], vec[near]
    if case["pad"]:  # a static edge capacity: the unused edges point at a padding node
        extra = int(case["pad"] * len(snd))
        pad, n = n, n + 1
        fill = torch.full((extra,), pad, dtype=torch.int32, device="cuda")
        snd, rcv, vec = torch.cat([snd, fill]), torch.cat([rcv, fill]), torch.cat([vec, vec.new_ones(extra, 3)])
    return snd, rcv, vec.contiguous(), n, pad


def _inputs(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    dt = torch.float64 if case["op"] == "conv64" else torch.float32

    def normal(*shape):
        return torch.randn(shape, generator=g, device="cuda", dtype=dt)

    C, op = case["C"], case["op"]
    if op == "records":
        dx, dy, dz = ((case[k] + 1) ** 2 for k in ("lx", "ly", "lz"))
        R = case["rows"]
        return {"x": normal(R, dx, C), "y": normal(R, dy, C), "dz": normal(R, dz, C)}
    P = _Paths(case)
    if op == "linear":
        out = sorted(set(P.types))
        fan = {t: P.types.count(t) * C for t in out}
        W = torch.cat([(normal(fan[t] * case["C_out"]) / math.sqrt(fan[t])) for t in out])
        d = sum(2 * int(t[0]) + 1 for t in out)
        return {"x": normal(case["rows"], P.d_out, C), "W": W, "dout": normal(case["rows"], d, case["C_out"])}
    if op == "tp":
        R = case["rows"]
        y = _harmonics(case["lsh"], normal(R, 3).double()).float()
        return {"x": normal(R, P.d_in, C), "y": y, "w": normal(R, P.n, C), "dz": normal(R, P.d_out, C)}
    snd, rcv, vec, n, pad = _edges(case, seed)
    i = {"snd": snd, "rcv": rcv, "n": n, "pad": pad, "vec": vec.to(dt), "x": normal(n, P.d_in, C),
         "dm": normal(n, P.d_out, C)}
    # edge weights: a Bessel basis of the edge length times a linear layer
    r = vec.norm(dim=1, keepdim=True)
    cut = CLUSTER_CUT if case["atoms"] else R_CUT
    k = torch.arange(1, K_BESSEL + 1, device="cuda") * (math.pi / cut)
    h = (math.sqrt(2 / cut) * torch.sin(k * r) / r).to(dt).contiguous()
    W = normal(K_BESSEL, P.n, C) / math.sqrt(K_BESSEL)
    if op == "radial":
        i.update(h=h, W=W)
    else:
        i["s"] = (h @ W.reshape(K_BESSEL, -1)).reshape(-1, P.n, C)
    if op == "bwd2":
        E = len(snd)
        i["y"] = _harmonics(case["lsh"], vec.double()).float()
        i.update(ddx=normal(n, P.d_in, C), ddy=normal(E, P.d_sh), dds=normal(E, P.n, C))
    return i


def _records(case):
    """Every path between the three degree ranges, all of one output degree into one block."""
    i0, i1, i2, val = [], [], [], []
    for l1 in range(case["lx"] + 1):
        for l2 in range(case["ly"] + 1):
            for l3 in range(abs(l1 - l2), min(l1 + l2, case["lz"]) + 1):
                c = _coupling(l1, l2, l3)
                for M, a, b in zip(*np.nonzero(c)):
                    i0.append(l3 * l3 + M), i1.append(l1 * l1 + a), i2.append(l2 * l2 + b)
                    val.append(c[M, a, b] / math.sqrt(2 * l1 + 1))
    return np.array(i0), np.array(i1), np.array(i2), np.array(val)


def prepare(case, seed):
    i, op = _inputs(case, seed), case["op"]
    st = {"op": op, "in": i}
    if op == "records":
        st["tp"] = e3mi.RecordTP(*((case[k] + 1) ** 2 for k in ("lx", "ly", "lz")), *_records(case),
                                 y_per_channel=True)
        return st
    if op == "linear":
        P = _Paths(case)
        st["lin"] = e3mi.Linear(_irreps("+".join(P.types), case["C"]),
                                _irreps("+".join(sorted(set(P.types))), case["C_out"]))
        return st
    st["plan"] = e3mi.Plan(_irreps(case["blocks"], case["C"]), case["lsh"], case["lout"], natural=case["natural"])
    if op != "tp" and not case["rebuild"]:
        st["graph"] = e3mi.Graph(i["snd"], i["rcv"], i["n"], i["pad"])
    return st


def run(st):
    op, i = st["op"], st["in"]
    if op == "records":
        return st["tp"].forward(i["x"], i["y"]), st["tp"].backward(i["x"], i["y"], i["dz"])
    if op == "linear":
        return st["lin"].forward(i["x"], i["W"]), st["lin"].backward(i["x"], i["W"], i["dout"])
    plan = st["plan"]
    if op == "tp":
        return e3mi.tp_fwd(plan, i["x"], i["y"], i["w"]), e3mi.tp_bwd(plan, i["x"], i["y"], i["w"], i["dz"])
    graph = st["graph"] if "graph" in st else e3mi.Graph(i["snd"], i["rcv"], i["n"], i["pad"])
    if op == "bwd2":
        return e3mi.conv_bwd2(plan, graph, i["x"], i["y"], i["s"], i["dm"], i["ddx"], i["ddy"], i["dds"])
    if op == "radial":
        return (e3mi.conv_fwd_radial(plan, graph, i["x"], i["vec"], i["h"], i["W"]),
                e3mi.conv_bwd_radial(plan, graph, i["x"], i["vec"], i["h"], i["W"], i["dm"]))
    fwd, bwd = (e3mi.conv_fwd_f64, e3mi.conv_bwd_f64) if op == "conv64" else (e3mi.conv_fwd, e3mi.conv_bwd)
    return fwd(plan, graph, i["x"], i["vec"], i["s"]), bwd(plan, graph, i["x"], i["vec"], i["s"], i["dm"])


# ------------------------------------------------------------ cost and accuracy
def _n_edges(case):
    """Number of live edges."""
    if case["atoms"]:  # open cube: about half of the bulk's neighbours are inside, fewer in tiny clusters
        n, side = case["atoms"], (case["atoms"] / CLUSTER_PER_A3) ** (1 / 3)
        inside = max(0.3, 1 - 9 / 8 * CLUSTER_CUT / side * 2 / 3)
        return int(n * min(n - 1, CLUSTER_PER_A3 * 4 / 3 * math.pi * CLUSTER_CUT ** 3 * inside)) // 2 * 2
    return int(3 * case["mols"] * 3 * MOL_PER_A3 * 4 / 3 * math.pi * R_CUT ** 3) // 2 * 2


def work(case):
    """Each input read once, each output written once; the coupling's own
    multiply-adds (forward: one per (output row, x row) pair and output row;
    each cotangent contraction of the backward: one per pair or record)."""
    C, op = case["C"], case["op"]
    if op == "records":
        rows = sum((case[k] + 1) ** 2 for k in ("lx", "ly", "lz"))
        return {"bytes": 8 * case["rows"] * C * rows, "flops": 6 * len(_records(case)[0]) * case["rows"] * C}
    P = _Paths(case)
    if op == "linear":
        out = sorted(set(P.types))
        d = sum(2 * int(t[0]) + 1 for t in out)
        nw = P.n * C * case["C_out"]
        return {"bytes": 4 * (2 * case["rows"] * (P.d_out * C + d * case["C_out"]) + 2 * nw),
                "flops": 6 * case["rows"] * P.d_out * C * case["C_out"]}
    fwd, bwd = P.pairs + P.d_out, 2 * P.pairs + P.nnz
    if op == "tp":
        R = case["rows"]
        return {"bytes": 4 * R * (C * (2 * P.d_in + 2 * P.n + 2 * P.d_out) + 2 * P.d_sh),
                "flops": 2 * (fwd + bwd) * R * C}
    E = _n_edges(case)
    N = case["atoms"] or 3 * case["mols"]
    node = N * C * (2 * P.d_in + 2 * P.d_out)
    size = 8 if op == "conv64" else 4
    if op == "radial":
        return {"bytes": 4 * (node + E * (8 + 2 * K_BESSEL) + 2 * K_BESSEL * P.n * C),
                "flops": 2 * (fwd + bwd + 3 * K_BESSEL * P.n) * E * C}
    if op == "bwd2":
        return {"bytes": 4 * (N * C * (3 * P.d_in + 2 * P.d_out) + E * (3 * P.n * C + 3 * P.d_sh + 2)),
                "flops": 2 * (3 * fwd + 2 * bwd) * E * C}
    return {"bytes": size * (node + E * (2 * P.n * C + 8)), "flops": 2 * (fwd + bwd) * E * C}


def tolerance(case):
    """Other orders of the same sums, at the same precision: about four times the
    measured distance from 64 bits (float32: 0.5e-7 to 8e-7; float64, here
    against sums in another order: 5e-16 to 8e-16)."""
    if case["op"] == "conv64":
        return {"rel": 4e-15, "max": 1e-12}
    return {"rel": 2e-6, "max": 1e-4}


# ------------------------------------------------------------ the same in 64 bits
def _fwd_rows(P, x, y, s):
    """Messages [rows, d_out, C]."""
    out = []
    for k, (xs, ys, _, c) in enumerate(P.items):
        A = (y[:, ys] @ torch.from_numpy(c).to(y).reshape(-1, c.shape[2]).T).reshape(-1, *c.shape[:2])
        out.append(s[:, k, None] * (A @ x[:, xs]))
    return torch.cat(out, 1)


def _bwd_rows(P, x, y, s, dm):
    """Cotangents (dx, dy, ds) of every row."""
    dx, dy, ds = torch.zeros_like(x), torch.zeros_like(y), torch.empty_like(s)
    for k, (xs, ys, os, c) in enumerate(P.items):
        ct = torch.from_numpy(c).to(y).reshape(-1, c.shape[2])
        A = (y[:, ys] @ ct.T).reshape(-1, *c.shape[:2])
        d, xk = dm[:, os].contiguous(), x[:, xs].contiguous()
        ds[:, k] = (d * (A @ xk)).sum(1)
        u = s[:, k, None] * d
        dx[:, xs] += A.transpose(1, 2).contiguous() @ u
        dy[:, ys] += (u @ xk.transpose(1, 2).contiguous()).reshape(len(x), -1) @ ct
    return dx, dy, ds


def _chunks(n, width):
    step = max(256, (1 << 27) // max(1, width))
    return [slice(a, min(a + step, n)) for a in range(0, n, step)]


def exact(case, seed):
    """What run() returns, in float64, chunk by chunk."""
    i, op, C = _inputs(case, seed), case["op"], case["C"]
    D = {k: v.double() for k, v in i.items() if torch.is_tensor(v) and v.is_floating_point() and k not in
         ("s", "dds", "w", "dz")}
    if op == "records":
        x, y, dz = D["x"], D["y"], i["dz"].double()
        z, dx, dy = torch.zeros_like(dz), torch.zeros_like(x), torch.zeros_like(y)
        for a, b, c, v in zip(*_records(case)):
            z[:, a] += v * x[:, b] * y[:, c]
            dx[:, b] += v * dz[:, a] * y[:, c]
            dy[:, c] += v * dz[:, a] * x[:, b]
        return z, (dx, dy)
    P = _Paths(case)
    if op == "linear":
        x, W, dout, Co = D["x"], D["W"], D["dout"], case["C_out"]
        out, dx, dW, o, w0 = torch.zeros_like(dout), torch.zeros_like(x), torch.zeros_like(W), 0, 0
        for t in sorted(set(P.types)):
            d = 2 * int(t[0]) + 1
            for (_, _, rows, _), tt in zip(P.items, P.types):
                if tt == t:
                    w = W[w0:w0 + C * Co].view(C, Co)
                    xi, di = x[:, rows].reshape(-1, C), dout[:, o:o + d].reshape(-1, Co)
                    out[:, o:o + d] += (xi @ w).view(-1, d, Co)
                    dx[:, rows] = (di @ w.T.contiguous()).view(-1, d, C)
                    dW[w0:w0 + C * Co] = (xi.T.contiguous() @ di).reshape(-1)
                    w0 += C * Co
            o += d
        return out, (dx, dW)
    f64 = dict(dtype=torch.float64, device="cuda")
    if op == "tp":
        R = case["rows"]
        z = torch.empty(R, P.d_out, C, **f64)
        dx, dy, dw = torch.empty_like(D["x"]), torch.empty_like(D["y"]), torch.empty(R, P.n, C, **f64)
        for c in _chunks(R, P.d_out * C):
            x, y, w = D["x"][c], D["y"][c], i["w"][c].double()
            z[c] = _fwd_rows(P, x, y, w)
            dx[c], dy[c], dw[c] = _bwd_rows(P, x, y, w, i["dz"][c].double())
        return z, (dx, dy, dw)
    n, E = i["n"], len(i["snd"])
    live = int((i["snd"] != i["pad"]).sum())  # padding edges come last
    m, dx, ds = torch.zeros(n, P.d_out, C, **f64), torch.zeros(n, P.d_in, C, **f64), None
    if op == "radial":
        dh, dW = torch.zeros(E, K_BESSEL, **f64), torch.zeros_like(D["W"])
    else:
        ds = torch.zeros(E, P.n, C, **f64)
    dy = torch.zeros(E, P.d_sh if op == "bwd2" else 3, **f64)
    for c in _chunks(live, P.d_out * C):
        snd, rcv = i["snd"][c].long(), i["rcv"][c].long()
        x, dm = D["x"][snd], D["dm"][rcv]
        if op == "radial":
            s = (D["h"][c] @ D["W"].view(K_BESSEL, -1)).view(-1, P.n, C)
        else:
            s = i["s"][c].double()
        if op == "bwd2":
            y, ddx, ddy, dds = D["y"][c], D["ddx"][snd], D["ddy"][c], i["dds"][c].double()
            m.index_add_(0, rcv, _fwd_rows(P, ddx, y, s) + _fwd_rows(P, x, ddy, s) + _fwd_rows(P, x, y, dds))
            a, b, d = (_bwd_rows(P, ddx, y, s, dm), _bwd_rows(P, x, ddy, s, dm), _bwd_rows(P, x, y, dds, dm))
            dx.index_add_(0, snd, b[0] + d[0])
            dy[c], ds[c] = a[1] + d[1], a[2] + b[2]
            continue
        v = D["vec"][c].clone().requires_grad_(True)
        y = _harmonics(case["lsh"], v)
        m.index_add_(0, rcv, _fwd_rows(P, x, y.detach(), s))
        gx, gy, gs = _bwd_rows(P, x, y.detach(), s, dm)
        dx.index_add_(0, snd, gx)
        dy[c], = torch.autograd.grad(y, v, gy)
        if op == "radial":
            dh[c] = gs.reshape(len(gs), -1) @ D["W"].view(K_BESSEL, -1).T.contiguous()
            dW += (D["h"][c].T.contiguous() @ gs.reshape(len(gs), -1)).view_as(dW)
        else:
            ds[c] = gs
    if op == "bwd2":
        return dx, dy, ds, m
    return m, ((dx, dy, dh, dW) if op == "radial" else (dx, dy, ds))
