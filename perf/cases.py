"""Timed cases of the energy+force path: what programs built on this package
have it do, through its public Python entry points (``Potential.compute``,
``compute_noalloc``, ``md_run`` and the differentiable ``energy_forces``).

Workloads (the synthetic models of ``paper_2002_00054_amd/synth.py``):
  water   two elements, 6 A cutoff, 27/30 SFs, about 86 neighbours per atom;
  fcc     one element, 3.9 A cutoff, 14 SFs, about 18 neighbours;
  wide    the fcc model with its angular SFs as wide functions G9;
  three   three elements on the water lattice, 30 SFs per element over six
          element-pair classes (angular terms of other zeta and eta than the
          water model's).

Kinds of use:
  compute one structure, E, E_i and F (an energy+force server, a relaxation
          step, the benchmark);
  noalloc the same into caller-owned outputs with the static workspace;
  md      some velocity-Verlet steps from given positions and velocities;
  train   one training step on a batch of uneven boxes: energy and force
          loss, weight gradient.

``exact`` is a plain torch evaluation in float64 of the same formulas.
"""
import math

import numpy as np
import torch

from paper_2002_00054_amd import synth
from paper_2002_00054_amd.nnp import Potential, energy_forces

SPACING = synth.WATER_SPACING
MD_DT = 0.25  # fs
FORCE_WEIGHT = 0.1


def _case(name, kind, work, form, nx, ny, nz, spacing=None, n=0, layout="padded"):
    """n: MD steps or training boxes (the sides then bound the boxes' sides)."""
    if spacing is None:
        spacing = synth.NI_LATTICE if work in ("fcc", "wide") else SPACING
    return {"name": name, "kind": kind, "work": work, "form": form, "nx": nx, "ny": ny, "nz": nz,
            "spacing": spacing, "n": n, "layout": layout}


def listed():
    return [
        # the smallest call: one 192-atom structure at a time (data labelling, relaxation), all latency
        _case("water_192_fp32", "compute", "water", "fp32", 4, 4, 4),
        # a serving loop that may not allocate, an odd count of atoms, double precision
        _case("water_1029_fp64_noalloc", "noalloc", "water", "fp64", 7, 7, 7),
        # the usual structure of the parity and sweep runs
        _case("water_12288_fp32", "compute", "water", "fp32", 16, 16, 16),
        # a ragged box with three different edges, all-(q, n) kernels of a three-element model
        _case("three_15147_fp32", "compute", "three", "fp32", 17, 11, 27),
        # a middle size in the mixed-precision form
        _case("water_98304_bf16", "compute", "water", "bf16", 32, 32, 32),
        # one eighth of the large box (a spatial shard), double precision
        _case("water_255552_fp64", "compute", "water", "fp64", 44, 44, 44),
        # the benchmark
        _case("water_2044416_fp32", "compute", "water", "fp32", 88, 88, 88),
        # the second workload at its full size, short neighbour rows
        _case("fcc_1492992_fp32", "compute", "fcc", "fp32", 72, 72, 72),
        # wide angular functions on an uneven box, double precision
        _case("wide_34440_fp64", "compute", "wide", "fp64", 15, 14, 41),
        # one optimiser step of training in each precision: 32 boxes of 192 to 1536 atoms
        _case("train_32_fp32", "train", "water", "fp32", 4, 0, 8, n=32),
        _case("train_32_fp64", "train", "water", "fp64", 4, 0, 8, n=32),
        # molecular dynamics of a middle-size box, double precision (energy conservation runs)
        _case("md_12288_fp64", "md", "water", "fp64", 16, 16, 16, n=5),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    kind = rng.choice(("compute", "compute", "compute", "compute", "noalloc", "train", "md"))
    form = rng.choice(("fp32", "fp32", "fp64", "bf16"))
    spacing = SPACING if rng.random() < 0.5 else round(rng.uniform(3.0, 3.5), 3)
    if kind == "train":  # boxes of 192 to 1536 atoms
        lo = rng.randint(4, 6)
        return {k: v for k, v in _case("", "train", "water", rng.choice(("fp32", "fp64")), lo, 0,
                                       rng.randint(lo, 8), spacing, rng.randint(1, 40)).items() if k != "name"}
    work = rng.choice(("water", "water", "water", "fcc", "wide", "three")) if kind == "compute" else "water"
    lattice = work in ("fcc", "wide")
    least, most = (27, 370000) if lattice else (64, 680000)
    if work == "three":
        most = 100000
    if form != "fp32":
        most = min(most, 250000 if form == "fp64" else 600000)
    if not lattice and spacing < SPACING:  # denser: more neighbours and pairs of them
        most = int(most * (spacing / SPACING) ** 9)
    if work == "wide":
        most = min(most, 100000)
    if kind == "noalloc":
        most = 5200 if form == "fp32" else 4000
    if kind == "md":
        most = 20000
    side = _log(rng, least, most) ** (1.0 / 3.0)
    small = 3 if lattice else 4
    top = int(most ** (1.0 / 3.0))
    s = [max(small, min(top, round(side * rng.uniform(0.8, 1.25)))) for _ in range(3)]
    return {k: v for k, v in _case("", kind, work, form, *s, None if lattice else spacing,
                                   rng.randint(2, 6) if kind == "md" else 0,
                                   "index" if kind == "compute" and rng.random() < 0.1 else "padded").items()
            if k != "name"}


# ------------------------------------------------------------------ models
def _three_table():
    """Two angular eta, 6 radial and 6 classes x 4 angular SFs per centre; the
    scale is the size of the raw values on these boxes."""
    t = []
    for c in range(3):
        for nb in range(3):
            for eta in (0.004, 0.05):
                t.append(synth.SF(c, 2, (nb,), eta, shift=6.0 if eta < 0.01 else 3.0, scale=4.0))
        for e1 in range(3):
            for e2 in range(e1, 3):
                for eta, zeta, lam in ((0.002, 1.0, -1.0), (0.002, 4.0, 1.0), (0.03, 2.0, 1.0), (0.03, 16.0, -1.0)):
                    t.append(synth.SF(c, 3, (e1, e2), eta, 0.0, zeta, lam, shift=2.0, scale=8.0))
    return t


def _model(work):
    """(table, networks, elements) of a workload."""
    if work == "fcc":
        return synth.ni_table_scaled(), synth.ni_nets(), ("Ni",)
    if work == "wide":
        return synth.ni_table_scaled(wide=True), synth.ni_nets(), ("Ni",)
    if work == "three":
        t = _three_table()
        return t, synth.xavier_nets(synth.sf_counts(t, 3), 3), ("A", "B", "C")
    return synth.water_table_scaled(), synth.water_nets(), ("H", "O")


# ------------------------------------------------------------------ inputs
def _water(nx, ny, nz, spacing, g):
    """Jittered lattice of rigid, randomly rotated water molecules, wrapped."""
    dev = "cuda"
    box = torch.tensor([nx, ny, nz], dtype=torch.float64, device=dev) * spacing
    i = torch.cartesian_prod(*(torch.arange(n, dtype=torch.float64, device=dev) for n in (nx, ny, nz)))
    o = spacing * i + (torch.rand(len(i), 3, dtype=torch.float64, device=dev, generator=g) * 2 - 1) * synth.JITTER
    q = torch.randn(len(i), 4, dtype=torch.float64, device=dev, generator=g)
    w, x, y, z = (q / q.norm(dim=1, keepdim=True)).unbind(1)
    e1 = torch.stack((1 - 2 * (y * y + z * z), 2 * (x * y + z * w), 2 * (x * z - y * w)), 1)
    e2 = torch.stack((2 * (x * y - z * w), 1 - 2 * (x * x + z * z), 2 * (y * z + x * w)), 1)
    th = math.radians(synth.HOH_ANGLE_DEG)
    h1 = o + synth.OH_BOND * e1
    h2 = o + synth.OH_BOND * (math.cos(th) * e1 + math.sin(th) * e2)
    pos = torch.stack((o, h1, h2), 1).reshape(-1, 3) % box
    pos = torch.where(pos >= box, 0.0, pos)
    types = torch.tensor([synth.O, synth.H, synth.H], dtype=torch.int32, device=dev).repeat(len(i))
    return pos, types, box


def _fcc(nx, ny, nz, a, g):
    dev = "cuda"
    box = torch.tensor([nx, ny, nz], dtype=torch.float64, device=dev) * a
    i = torch.cartesian_prod(*(torch.arange(n, dtype=torch.float64, device=dev) for n in (nx, ny, nz)))
    basis = torch.tensor(synth.FCC_BASIS, dtype=torch.float64, device=dev)
    pos = ((i[:, None] + basis) * a).reshape(-1, 3)
    pos = (pos + (torch.rand(pos.shape, dtype=torch.float64, device=dev, generator=g) * 2 - 1) * synth.NI_JITTER) % box
    pos = torch.where(pos >= box, 0.0, pos)
    return pos, torch.zeros(len(pos), dtype=torch.int32, device=dev), box


def _sides(case):
    """Lattice sides of a training batch's boxes (the batch's make-up is part of the case)."""
    return [int(s) for s in np.random.default_rng(4).integers(case["nx"], case["nz"] + 1, size=case["n"])]


def _inputs(case, seed):
    """The structures of a case: positions and types (device), atom offsets and
    boxes (host), and what else the kind takes, as a dict."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    rd = torch.float64 if case["form"] == "fp64" else torch.float32
    d = {}
    if case["kind"] == "train":
        parts = [_water(s, s, s, case["spacing"], g) for s in _sides(case)]
    else:
        make = _fcc if case["work"] in ("fcc", "wide") else _water
        parts = [make(case["nx"], case["ny"], case["nz"], case["spacing"], g)]
    d["pos"] = torch.cat([p[0] for p in parts]).to(rd)
    d["types"] = torch.cat([p[1] for p in parts])
    n = len(d["types"])
    if case["work"] == "three":
        d["types"] = torch.randint(0, 3, (n,), dtype=torch.int32, device="cuda", generator=g)
    d["offs"] = np.cumsum([0] + [len(p[1]) for p in parts])
    d["boxes"] = np.stack([p[2].cpu().numpy() for p in parts])
    if case["kind"] == "md":
        m = torch.tensor(synth.WATER_MASSES, dtype=torch.float64, device="cuda")[d["types"].long()][:, None]
        v = torch.randn(n, 3, dtype=torch.float64, device="cuda", generator=g) * torch.sqrt(
            8.617333262e-5 * 300.0 / (m * 103.64269652680505))
        d["vel"] = (v - (m * v).sum(0) / m.sum()).to(rd)
    if case["kind"] == "train":
        flat = torch.tensor(synth.flat_params(synth.water_nets()), dtype=torch.float64, device="cuda")
        d["params"] = flat + 0.02 * torch.randn(len(flat), dtype=torch.float64, device="cuda", generator=g)
        d["counts"] = torch.tensor(np.diff(d["offs"]), dtype=torch.float64, device="cuda")
        d["E_ref"] = 0.1 * d["counts"] * torch.randn(case["n"], dtype=torch.float64, device="cuda", generator=g)
        d["F_ref"] = (0.3 * torch.randn(n, 3, dtype=torch.float64, device="cuda", generator=g)).to(rd)
    return d


def prepare(case, seed):
    d = _inputs(case, seed)
    table, nets, elements = _model(case["work"])
    pot = Potential(table, nets, precision=case["form"], elements=elements)
    if case["layout"] != "padded":
        pot.set_list_layout(case["layout"])
    d["case"], d["pot"] = case, pot
    if case["kind"] == "noalloc":
        d["ei"] = torch.empty(len(d["types"]), dtype=pot.dtype, device="cuda")
        d["f"] = torch.empty(len(d["types"]), 3, dtype=pot.dtype, device="cuda")
    if case["kind"] == "train":
        d["params"].requires_grad_(True)
    return d


def _loss(E, F, d):
    return torch.mean(((E - d["E_ref"]) / d["counts"]) ** 2) + FORCE_WEIGHT * torch.sum(
        (F - d["F_ref"]).double() ** 2) / (3 * len(F))


def run(state):
    kind, pot = state["case"]["kind"], state["pot"]
    pos, types = state["pos"], state["types"]
    if kind == "compute":
        e, ei, f = pot.compute(pos, types, state["boxes"][0])
        return {"E": e, "E_i": ei, "F": f}
    if kind == "noalloc":
        e = pot.compute_noalloc(pos, types, state["boxes"][0], state["ei"], state["f"])
        return {"E": e, "E_i": state["ei"], "F": state["f"]}
    if kind == "md":
        x, v = pos.clone(), state["vel"].clone()  # the run advances them in place
        f, ep, ek = pot.md_run(x, v, types, state["boxes"][0], synth.WATER_MASSES, MD_DT, state["case"]["n"])
        return {"x": x, "v": v, "F": f, "E_pot": ep, "E_kin": ek}
    E, F = energy_forces(state["params"], pos, pot, types, state["offs"], state["boxes"])
    loss = _loss(E, F, state)
    (grad,) = torch.autograd.grad(loss, state["params"])
    return {"loss": loss.detach(), "E": E.detach(), "F": F.detach(), "grad": grad}


# ------------------------------------------------------------------ work
def _atoms(case):
    if case["kind"] == "train":
        return 3 * sum(s ** 3 for s in _sides(case))
    return case["nx"] * case["ny"] * case["nz"] * (4 if case["work"] in ("fcc", "wide") else 3)


def work(case):
    """Each input read and each output written once; operations of the SF sums
    and of their gradients contracted into forces, from the mean number of
    neighbours and of neighbour pairs at the case's density (two random points
    of a sphere of radius rc are within rc of each other with probability
    15/32)."""
    table, nets, _ = _model(case["work"])
    n, rc, n_el = _atoms(case), table[0].rc, len(nets)
    per_site = 4 if case["work"] in ("fcc", "wide") else 3
    frac = {"water": (2 / 3, 1 / 3), "three": (1 / 3,) * 3}.get(case["work"], (1.0,))
    m = per_site / case["spacing"] ** 3 * 4.0 / 3.0 * math.pi * rc ** 3
    share = 1.0 if case["work"] == "wide" else 15.0 / 32.0
    sf = force = 0.0
    for e in range(n_el):
        rad = ang = 0.0
        classes = set()
        for s in table:
            if s.centre != e:
                continue
            if s.kind == 2:
                rad += frac[s.nbr[0]] * m
            else:
                a, b = sorted(s.nbr)
                ang += share * m * m * (frac[a] * frac[b] if a != b else frac[a] ** 2 / 2)
                classes.add((a, b))
        cand = sum(m * m * (frac[a] * frac[b] if a != b else frac[a] ** 2 / 2) for a, b in classes)
        sf += frac[e] * (20 * m + 6 * rad + 9 * cand + 30 * share * cand + 5 * ang)
        force += frac[e] * (34 * m + 10 * rad + 9 * cand + 108 * share * cand + 9 * ang)
    mlp = 4 * 25 * (len(table) / n_el + 26)
    real = 8 if case["form"] == "fp64" else 4
    if case["kind"] == "train":
        params = sum(x.size for net in nets for x in (*net.W, *net.b))
        return {"bytes": n * (3 * real + 4 + 6 * real) + 16 * params, "flops": n * (sf + 2 * force + 5 * mlp)}
    evaluations, extra = (case["n"] + 1, 9 * real) if case["kind"] == "md" else (1, real)
    return {"bytes": n * (6 * real + 4 + extra), "flops": n * evaluations * (sf + force + mlp)}


# ------------------------------------------------------------------ float64 reference
def _fc(s, rc):
    """Cosine cutoff from the squared distance; 0 beyond rc."""
    inside = s < rc * rc
    r = torch.sqrt(torch.where(inside, s, rc * rc))
    return torch.where(inside, 0.5 * (torch.cos(math.pi * r / rc) + 1.0), 0.0)


def _neighbours(pos, types, box, rc, lo, hi):
    """Rows of neighbour indices of atoms lo..hi, padded, and their mask."""
    d = pos[lo:hi, None, :] - pos[None, :, :]
    d -= box * torch.round(d / box)
    near = (d * d).sum(-1) < rc * rc
    near[torch.arange(hi - lo, device=pos.device), torch.arange(lo, hi, device=pos.device)] = False
    row, col = near.nonzero().unbind(1)
    count = near.sum(1)
    m = max(1, int(count.max()))
    slot = torch.arange(len(row), device=pos.device) - (count.cumsum(0) - count)[row]
    idx = torch.zeros(hi - lo, m, dtype=torch.int64, device=pos.device)
    idx[row, slot] = col
    return idx, torch.arange(m, device=pos.device) < count[:, None]


def _descriptors(D, mask, tj, tc, table, n_el):
    """Scaled SF rows [C, max n_sf] of C centres from their displacements D [C, m, 3]."""
    rc = table[0].rc
    s = torch.where(mask, (D * D).sum(-1), 1.0)
    r = torch.sqrt(s)
    fc = torch.where(mask, _fc(s, rc), 0.0)
    dot = D @ D.transpose(1, 2).contiguous()
    cos = dot / (r[:, :, None] * r[:, None, :])
    sjk = s[:, :, None] + s[:, None, :] - 2.0 * dot
    pair = mask[:, :, None] & mask[:, None, :] & ~torch.eye(D.shape[1], dtype=torch.bool, device=D.device)
    sjk = torch.where(pair, sjk, rc * rc)
    fcjk = _fc(sjk, rc)
    width = max(synth.sf_counts(table, n_el))
    rows = []
    el = [(tj == e) & mask for e in range(n_el)]
    radial, wide, pw, out = {}, {}, {}, torch.zeros(len(D), width, dtype=D.dtype, device=D.device)
    for e in range(n_el):
        cols = []
        for t in (t for t in table if t.centre == e):
            if t.kind == 2:
                key = (t.eta, t.rs)
                if key not in radial:
                    radial[key] = torch.exp(-t.eta * (r - t.rs) ** 2) * fc
                v = (radial[key] * el[t.nbr[0]]).sum(1)
            else:
                key = (t.kind, t.eta)
                if key not in wide:
                    g = torch.exp(-t.eta * s) * fc
                    wide[key] = g[:, :, None] * g[:, None, :] * pair
                    if t.kind == 3:
                        wide[key] = wide[key] * torch.exp(-t.eta * sjk) * fcjk
                if (t.zeta, t.lam) not in pw:
                    p = 1.0 + t.lam * cos
                    for _ in range(int(t.zeta).bit_length() - 1):
                        p = p * p
                    pw[(t.zeta, t.lam)] = p
                a, b = t.nbr[0], t.nbr[-1]
                # sum over ordered pairs (j of a, k of b); each unordered pair twice when a == b
                v = torch.matmul((wide[key] * pw[(t.zeta, t.lam)]), el[b].to(D.dtype)[:, :, None]).squeeze(-1)
                v = (v * el[a]).sum(1) * (2.0 ** (1.0 - t.zeta) * (0.5 if a == b else 1.0))
            cols.append((v - t.shift) / t.scale)
        row = torch.stack(cols, 1)
        row = torch.nn.functional.pad(row, (0, width - row.shape[1]))
        rows.append(torch.where((tc == e)[:, None], row, 0.0))
    for x in rows:
        out = out + x
    return out


def _split(flat, table, n_el):
    """Weights per element of a flat parameter vector."""
    nets, o = [], 0
    for ns in synth.sf_counts(table, n_el):
        sizes, net = [ns, *synth.HIDDEN, 1], []
        for i, k in zip(sizes[:-1], sizes[1:]):
            net.append((flat[o:o + i * k].reshape(k, i), flat[o + i * k:o + i * k + k]))
            o += i * k + k
        nets.append(net)
    return nets


def _energies(G, tc, nets):
    e = torch.zeros(len(G), dtype=G.dtype, device=G.device)
    for t, net in enumerate(nets):
        at = torch.nonzero(tc == t).squeeze(1)
        x = G[at][:, : net[0][0].shape[1]]
        for l, (W, b) in enumerate(net):
            x = torch.nn.functional.linear(x, W, b)
            if l < len(net) - 1:
                x = torch.tanh(x)
        e = e.index_add(0, at, x.squeeze(1))
    return e


def _reference(pos, types, box, table, nets, n_el, delta=None):
    """(E_i, F) in float64 and, with delta [n, 3], (G, v) too: the scaled SFs
    and their derivative along delta."""
    n, rc = len(pos), table[0].rc
    Ei, F = torch.zeros(n, dtype=torch.float64, device=pos.device), torch.zeros_like(pos)
    Gs, vs = [], []
    chunk = int(max(64, min(1024, 1.2e8 / max(n, 1))))
    for lo in range(0, n, chunk):
        hi = min(n, lo + chunk)
        idx, mask = _neighbours(pos, types, box, rc, lo, hi)
        D = pos[idx] - pos[lo:hi, None, :]
        D = D - box * torch.round(D / box)
        D = torch.where(mask[:, :, None], D, 1.0)
        tc, tj = types[lo:hi].long(), types[idx].long()
        D.requires_grad_(True)
        if delta is not None:
            dD = torch.where(mask[:, :, None], delta[idx] - delta[lo:hi, None, :], 0.0)
            G = _descriptors(D, mask, tj, tc, table, n_el)
            u = torch.ones_like(G, requires_grad=True)
            (gD,) = torch.autograd.grad(G, D, u, create_graph=True)
            (v,) = torch.autograd.grad((gD * dD).sum(), u)
            Gs.append(G.detach())
            vs.append(v)
            continue
        e = _energies(_descriptors(D, mask, tj, tc, table, n_el), tc, nets)
        (gD,) = torch.autograd.grad(e.sum(), D)
        gD = torch.where(mask[:, :, None], gD, 0.0)
        Ei[lo:hi] = e.detach()
        F[lo:hi] += gD.sum(1)
        F.index_add_(0, idx.reshape(-1), -gD.reshape(-1, 3))
    return (Ei, F) if delta is None else (torch.cat(Gs), torch.cat(vs))


def _exact_train(d, table, n_el):
    params = d["params"].detach()
    nets = _split(params, table, n_el)
    offs, E, F = d["offs"], [], []
    for b in range(len(offs) - 1):
        s = slice(int(offs[b]), int(offs[b + 1]))
        box = torch.tensor(d["boxes"][b], device="cuda")
        ei, f = _reference(d["pos"][s].double(), d["types"][s], box, table, nets, n_el)
        E.append(ei.sum())
        F.append(f)
    E, F = torch.stack(E).requires_grad_(True), torch.cat(F).requires_grad_(True)
    loss = _loss(E, F, {**d, "F_ref": d["F_ref"].double()})
    gE, gF = torch.autograd.grad(loss, (E, F))
    # dF/dtheta . gF = -d/dtheta sum_i dE_i/dG_i . v_i with v the derivative of G along gF
    flat = params.clone().requires_grad_(True)
    nets = _split(flat, table, n_el)
    total = torch.zeros((), dtype=torch.float64, device="cuda")
    for b in range(len(offs) - 1):
        s = slice(int(offs[b]), int(offs[b + 1]))
        box = torch.tensor(d["boxes"][b], device="cuda")
        G, v = _reference(d["pos"][s].double(), d["types"][s], box, table, None, n_el, gF[s])
        G.requires_grad_(True)
        e = _energies(G, d["types"][s].long(), nets)
        (c,) = torch.autograd.grad(e.sum(), G, create_graph=True)
        total = total + gE[b] * e.sum() - (c * v).sum()
    (grad,) = torch.autograd.grad(total, flat)
    return {"loss": loss.detach(), "E": E.detach(), "F": F.detach(), "grad": grad}


def _exact_md(d, case, table, nets, n_el):
    box = torch.tensor(d["boxes"][0], device="cuda")
    m = torch.tensor(synth.WATER_MASSES, dtype=torch.float64, device="cuda")[d["types"].long()][:, None]
    ev, amu = 1.602176634e-19, 1.66053906660e-27
    acc, kin = ev / 1e-10 / amu * 1e-30 / 1e-10, amu * 1e10 / ev
    x, v = d["pos"].double(), d["vel"].double()

    def wrap(p):
        p = p - box * torch.floor(p / box)
        return torch.where((p >= 0) & (p < box), p, 0.0)

    ep, ek = [], []
    for step in range(case["n"] + 1):
        if step:
            v = v + 0.5 * MD_DT * acc * F / m
            x = wrap(x + MD_DT * v)
        ei, F = _reference(x, d["types"], box, table, nets, n_el)
        if step:
            v = v + 0.5 * MD_DT * acc * F / m
        ep.append(float(ei.sum()))
        ek.append(float((0.5 * m * v * v).sum() * kin))
    return {"x": x, "v": v, "F": F, "E_pot": np.array(ep), "E_kin": np.array(ek)}


def exact(case, seed):
    if _atoms(case) > 300000:  # minutes in float64
        return None
    table, nets, _ = _model(case["work"])
    n_el = len(nets)
    d = _inputs(case, seed)
    if case["kind"] == "train":
        return _exact_train(d, table, n_el)
    nets = _split(torch.tensor(synth.flat_params(nets), dtype=torch.float64, device="cuda"), table, n_el)
    if case["kind"] == "md":
        return _exact_md(d, case, table, nets, n_el)
    box = torch.tensor(d["boxes"][0], device="cuda")
    ei, f = _reference(d["pos"].double(), d["types"], box, table, nets, n_el)
    return {"E": float(ei.sum()), "E_i": ei, "F": f}
