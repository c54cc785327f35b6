"""The work that users of this library have it do, as measurable cases.

Families (``kind``):

* ``force``: one bin + force call of a small periodic box or open block, in
  buffers the caller keeps (the latency of the smallest calls);
* ``step``: a time step of a differentiable simulation: bin, forces, position
  gradient (bins reused), in buffers the caller keeps;
* ``autograd``: the same through ``sr_force`` and ``backward``;
* ``batch``: many independent periodic subvolumes in one plan;
* ``blocks``: one open domain solved and differentiated in overlapping blocks;
* ``pk``: the on-the-fly power spectrum;
* ``centres``: the most bound particle of every halo of a catalogue.

Inputs are drawn on the GPU from the seed by the recipes of
``paper_1411_3396_amd/synth.py``: uniform matter, or a uniform background with
Plummer halos, one particle per unit cell on average, cutoff 3 cells.  The
float64 momentum check is left out: it sums to nearly zero, so its relative
change says nothing.
"""
import math

import numpy as np
import torch

from paper_1411_3396_amd import _sr, blocks, synth

R_S = 3.0
DEV = "cuda"


def listed():
    return [
        # one call on a handful of particles: what an interactive or adaptive code pays per call
        {"name": "force_1k", "kind": "force", "matter": "uniform", "n": 1000, "open": False, "eps": 0.05,
         "leaf_depth": 1, "random_mass": False},
        # the smallest named workload: 32^3 particles, a step of a unit-test sized simulation
        {"name": "step_uniform_32k", "kind": "step", "matter": "uniform", "n": 32768, "open": False, "eps": 0.05,
         "leaf_depth": 2, "random_mass": False},
        # an optimisation loop through autograd: an odd count, masses that differ, everything allocated per call
        {"name": "autograd_100k", "kind": "autograd", "matter": "clustered", "n": 100003, "open": False,
         "eps": 0.05, "leaf_depth": 1, "random_mass": True, "halo_frac": 0.4},
        # 128^3 particles at moderate clustering: the ordinary step
        {"name": "step_clustered_2m", "kind": "step", "matter": "clustered", "n": 2097152, "open": False,
         "eps": 0.05, "leaf_depth": 2, "random_mass": False, "halo_frac": 0.4},
        # the same box with a few very large halos: late-time clustering
        {"name": "step_extreme_2m", "kind": "step", "matter": "extreme", "n": 2097152, "open": False, "eps": 0.05,
         "leaf_depth": 2, "random_mass": False, "halo_frac": 0.4},
        # 256^3 particles at moderate clustering
        {"name": "step_clustered_16m", "kind": "step", "matter": "clustered", "n": 16777216, "open": False,
         "eps": 0.05, "leaf_depth": 2, "random_mass": False, "halo_frac": 0.4},
        # one node's share of the production run: 320^3 active cells and a 3-cell ghost shell
        {"name": "step_node_share", "kind": "step", "matter": "clustered", "n": 34645976, "open": True,
         "eps": 0.02, "leaf_depth": 2, "random_mass": False, "halo_frac": 0.75},
        # 96 uniform subvolumes of 1e4 to 1e6 particles as one graph replay
        {"name": "batch_96", "kind": "batch", "sub": 96, "n_lo": 10000, "n_hi": 1000000, "count_seed": 3},
        # a 128-cell domain with its ghosts in 2 x 2 overlapping blocks, forces and gradients
        {"name": "blocks_2m", "kind": "blocks", "n": 2406104, "nbx": 2, "nby": 2, "halo_frac": 0.75},
        # power spectrum of the 256^3 particles on the grid of the same side (bricks of 8 cells)
        {"name": "pk_256", "kind": "pk", "n": 16777216, "ng": 256, "halo_frac": 0.4},
        # a quick look on a grid whose side is no multiple of 8 (the deposit by cells)
        {"name": "pk_100", "kind": "pk", "n": 1000000, "ng": 100, "halo_frac": 0.4},
        # a late-time halo catalogue: many small halos, a few large ones
        {"name": "centres_2k", "kind": "centres", "halos": 2000, "n_min": 40, "n_max": 100000},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["force", "step", "step", "step", "autograd", "batch", "blocks", "pk", "pk", "centres"])
    if kind in ("force", "step", "autograd"):
        matter = rng.choice(["uniform", "clustered", "clustered"])
        lo, hi = {"force": (800, 60000), "step": (3000, 12000000), "autograd": (2000, 1500000)}[kind]
        c = {"kind": kind, "matter": matter, "n": _log(rng, lo, hi), "open": rng.random() < 0.4,
             "eps": rng.choice([0.05, 0.02, 0.01]), "leaf_depth": rng.choice([1, 2, 2, 3]),
             "random_mass": rng.random() < 0.3}
        if matter == "clustered":
            c["halo_frac"] = round(rng.uniform(0.3, 0.75), 3)
        return c
    if kind == "batch":
        lo = _log(rng, 1000, 30000)
        return {"kind": kind, "sub": rng.randint(3, 64), "n_lo": lo, "n_hi": lo * rng.randint(2, 20),
                "count_seed": rng.randint(0, 999)}
    if kind == "blocks":
        return {"kind": kind, "n": _log(rng, 50000, 3000000), "nbx": rng.randint(1, 4), "nby": rng.randint(1, 3),
                "halo_frac": round(rng.uniform(0.3, 0.75), 3)}
    if kind == "pk":
        ng = rng.choice([8 * rng.randint(4, 48), 2 * rng.randint(12, 80)])
        return {"kind": kind, "n": _log(rng, 10000, 12000000), "ng": ng, "halo_frac": round(rng.uniform(0.0, 0.6), 3)}
    return {"kind": "centres", "halos": _log(rng, 20, 4000), "n_min": 40, "n_max": _log(rng, 500, 60000)}


# ------------------------------------------------------------------- inputs


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _rand(g, *shape):
    return torch.rand(shape, generator=g, device=DEV, dtype=torch.float64)


def _plummer(g, scale):
    """Offsets of particles of Plummer spheres with these scale radii, truncated at ten of them."""
    n = scale.shape[0]
    u = (_rand(g, n) * (100.0 / 101.0) ** 1.5).clamp_min(1e-12)
    r = scale / torch.sqrt(u.pow(-2.0 / 3.0) - 1.0)
    cz = 2.0 * _rand(g, n) - 1.0
    ph = 2.0 * math.pi * _rand(g, n)
    sz = torch.sqrt((1.0 - cz * cz).clamp_min(0.0))
    return torch.stack([r * sz * torch.cos(ph), r * sz * torch.sin(ph), r * cz], dim=1)


def _to_box(x, lo, length):
    p = (torch.remainder(x - lo, length) + lo).float()
    hi = float(np.float32(lo + length))
    return torch.where(p >= hi, torch.full_like(p, lo), p).contiguous()


def _matter(case, g, seed, lo, length):
    """float32 positions [n, 3] in [lo, lo + length)^3, in random order."""
    n = case["n"]
    if case["matter"] == "uniform":
        return _to_box(lo + length * _rand(g, n, 3), lo, length)
    budget = int(round(case["halo_frac"] * n))
    if case["matter"] == "extreme":  # halo masses are absolute counts: few, very large halos
        rng = np.random.default_rng(seed)
        counts = []
        while sum(counts) < budget:
            counts.append(min(max(1, int(math.exp(rng.uniform(math.log(1e2), math.log(1e5))))), budget - sum(counts)))
        k = len(counts)
        hid = torch.repeat_interleave(torch.arange(k, device=DEV), torch.tensor(counts, device=DEV))
    else:  # halo masses are log-uniform weights of the halo share
        k = max(1, n // (1700 if case.get("open") else 1048))
        top = 1e6 if case.get("open") else 1e5
        w = torch.exp(math.log(1e2) + _rand(g, k) * (math.log(top) - math.log(1e2)))
        hid = torch.searchsorted(torch.cumsum(w / w.sum(), 0), _rand(g, budget)).clamp_max(k - 1)
    scale = torch.exp(math.log(0.5) + _rand(g, k) * (math.log(4.0) - math.log(0.5)))
    centre = lo + length * _rand(g, k, 3)
    x = torch.cat([lo + length * _rand(g, n - budget, 3), centre[hid] + _plummer(g, scale[hid])])
    return _to_box(x[torch.randperm(n, generator=g, device=DEV)], lo, length)


def _domain(case, seed):
    """Positions, masses, active count and problem of a force, step or autograd case."""
    g = _gen(seed)
    n = case["n"]
    depth = case.get("leaf_depth", 1)
    eps = case["eps"]
    poly = synth.filter_poly(R_S, eps)
    side = float(np.float32(n ** (1.0 / 3.0)))
    if case["open"]:  # an active cube in a shell of 3 cells of passive particles
        lo = -R_S
        pos = _matter(case, g, seed, lo, side)
        inner = side - 2.0 * R_S
        # the innermost share: the same count for every seed, the cube's faces move a little
        n_active = int(n * (inner / side) ** 3)
        act = torch.zeros(n, dtype=torch.bool, device=DEV)
        act[torch.argsort((pos - (lo + 0.5 * side)).abs().amax(dim=1))[:n_active]] = True
        pos = torch.cat([pos[act], pos[~act]]).contiguous()
        prob = synth.Problem.make((lo,) * 3, (side,) * 3, False, R_S, eps, poly, depth)
    else:
        side = max(side, 3.0 * R_S)
        pos = _matter(case, g, seed, 0.0, side)
        n_active = n
        prob = synth.Problem.make((0.0,) * 3, (side,) * 3, True, R_S, eps, poly, depth)
    mass = (0.5 + 1.5 * _rand(g, n)).float() if case["random_mass"] else torch.ones(n, device=DEV)
    cot = torch.randn((n_active, 3), generator=g, device=DEV)
    return pos, mass, n_active, prob, cot


def _batch_counts(case):
    rng = np.random.default_rng(case["count_seed"])
    return np.floor(np.exp(rng.uniform(math.log(case["n_lo"]), math.log(case["n_hi"]), case["sub"]))).astype(np.int64)


def _batch_inputs(case, seed):
    g = _gen(seed)
    counts = _batch_counts(case)
    poly = synth.filter_poly(R_S, 0.05)
    parts, probs = [], []
    for nb in counts:
        side = float(np.float32(max(float(nb) ** (1.0 / 3.0), 3.0 * R_S)))
        parts.append(_to_box(side * _rand(g, int(nb), 3), 0.0, side))
        probs.append(synth.Problem.make((0.0,) * 3, (side,) * 3, True, R_S, 0.05, poly))
    pos = torch.cat(parts).contiguous()
    return pos, torch.ones(pos.shape[0], device=DEV), counts, probs


def _blocks_case(case):
    return dict(case, matter="clustered", open=True, eps=0.02, random_mass=False, leaf_depth=1)


def _pk_inputs(case, seed):
    g = _gen(seed)
    box = float(np.float32(case["n"] ** (1.0 / 3.0)))
    pos = _matter(dict(case, matter="clustered", open=False), g, seed, 0.0, box)
    return pos, torch.ones(case["n"], device=DEV), box


def _halo_offsets(case):
    rng = np.random.default_rng(case["halos"] + 7 * case["n_max"])
    counts = synth.power_law_counts(rng, case["halos"], case["n_min"], case["n_max"], 1.9)
    return np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)


def _halo_inputs(case, seed):
    g = _gen(seed)
    off = _halo_offsets(case)
    counts = torch.tensor(np.diff(off), device=DEV)
    hid = torch.repeat_interleave(torch.arange(case["halos"], device=DEV), counts)
    a = (3.0 * counts.double() / (800.0 * math.pi)).pow(1.0 / 3.0) / 5.0
    centre = 320.0 * _rand(g, case["halos"], 3)
    pos = (centre[hid] + _plummer(g, a[hid])).float().contiguous()
    return pos, torch.ones(pos.shape[0], device=DEV), off


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("force", "step", "autograd"):
        pos, mass, n_active, prob, cot = _domain(case, seed)
        s = {"kind": kind, "pos": pos, "mass": mass, "n_active": n_active, "prob": prob, "cot": cot}
        if kind != "autograd":
            s["prob"] = _sr.as_problem(prob)
            s["ws"] = _sr.new_workspace(_sr.workspace_bytes(case["n"], prob), DEV)
            s["acc"] = torch.empty((n_active, 3), device=DEV)
            s["grad"] = torch.empty((case["n"], 3), device=DEV) if kind == "step" else None
        return s
    if kind == "batch":
        pos, mass, counts, probs = _batch_inputs(case, seed)
        plan = _sr.BatchPlan(np.concatenate([[0], np.cumsum(counts)]), counts, probs)
        ws = _sr.new_workspace(plan.ws_bytes, DEV)
        acc = torch.empty((plan.total_active, 3), device=DEV)
        plan.run(pos, mass, ws, acc)  # tunes the plan and captures its graph
        return {"kind": kind, "pos": pos, "mass": mass, "plan": plan, "ws": ws, "acc": acc}
    if kind == "blocks":
        pos, mass, n_active, prob, cot = _domain(_blocks_case(case), seed)
        ng = blocks.grid_units(prob)
        bf = blocks.BlockForce(prob, blocks.equal_blocks(ng, case["nbx"], case["nby"]), case["n"], n_active,
                               tune_cache="")
        bf.forward(pos, mass)  # tunes the batch of blocks and captures its graph
        return {"kind": kind, "pos": pos, "mass": mass, "bf": bf, "cot": cot}
    if kind == "pk":
        pos, mass, box = _pk_inputs(case, seed)
        plan = _sr.PkPlan(case["ng"], box, case["ng"] // 2, 1.0, case["n"])
        return {"kind": kind, "pos": pos, "mass": mass, "plan": plan, "ws": _sr.new_workspace(plan.ws_bytes, DEV)}
    pos, mass, off = _halo_inputs(case, seed)
    plan = _sr.CentresPlan(off)
    return {"kind": kind, "pos": pos, "mass": mass, "plan": plan, "ws": _sr.new_workspace(plan.ws_bytes, DEV)}


# ------------------------------------------------------------------- one pass


def run(s):
    kind = s["kind"]
    if kind == "force":
        return [_sr.force(s["pos"], s["mass"], s["prob"], s["n_active"], ws=s["ws"], out=s["acc"])]
    if kind == "step":
        a = (s["pos"], s["mass"], s["prob"])
        _sr.bin(*a, s["n_active"], ws=s["ws"])
        acc = _sr.force(*a, s["n_active"], ws=s["ws"], reuse_bins=True, out=s["acc"])
        grad = _sr.force_vjp(*a, s["cot"], s["n_active"], ws=s["ws"], reuse_bins=True, out=s["grad"])
        return [acc, grad]
    if kind == "autograd":
        pos = s["pos"].detach().requires_grad_(True)
        acc = _sr.sr_force(pos, s["mass"], s["prob"], s["n_active"])
        acc.backward(s["cot"])
        return [acc, pos.grad]
    if kind == "batch":
        s["plan"].run(s["pos"], s["mass"], s["ws"], s["acc"])
        return [s["acc"]]
    if kind == "blocks":
        acc = s["bf"].forward(s["pos"], s["mass"])
        return [acc, s["bf"].vjp(s["pos"], s["mass"], s["cot"], partition=False)]
    if kind == "pk":
        return list(s["plan"].run(s["pos"], s["mass"], s["ws"]))
    return list(s["plan"].run(s["pos"], s["mass"], 0.02, s["ws"]))


# ------------------------------------------------------------------- the work


def _pairs(pos, mass, prob, n_active, adjoint):
    n = int(pos.shape[0])
    ws = _sr.bin(pos, mass, prob, n_active)
    return float(_sr.count_pairs(ws, n, prob, n_active, adjoint=adjoint).item())


def work(case):
    """Bytes: positions and masses in, results (and cotangents) in and out, each once.  Flops: 30 per
    ordered pair within the cutoff for a force, 61 for a gradient, 12 for a potential, and of the power
    spectrum the transform's."""
    kind = case["kind"]
    if kind in ("force", "step", "autograd", "blocks"):
        pos, mass, n_active, prob, _ = _domain(_blocks_case(case) if kind == "blocks" else case, 0)
        b, f = 16.0 * case["n"] + 12.0 * n_active, 30.0 * _pairs(pos, mass, prob, n_active, False)
        if kind != "force":
            b += 12.0 * n_active + 12.0 * case["n"]
            f += 61.0 * _pairs(pos, mass, prob, n_active, True)
        return {"bytes": b, "flops": f}
    if kind == "batch":
        n = float(_batch_counts(case).sum())
        return {"bytes": 28.0 * n, "flops": 30.0 * n * 4.0 / 3.0 * math.pi * R_S ** 3}
    if kind == "pk":
        grid = float(case["ng"]) ** 3
        return {"bytes": 16.0 * case["n"] + 4.0 * grid, "flops": 2.5 * grid * math.log2(grid)}
    c = np.diff(_halo_offsets(case)).astype(np.float64)
    return {"bytes": 20.0 * float(c.sum()), "flops": 12.0 * float((c * (c - 1.0)).sum())}


# ------------------------------------------------------------------- in 64 bits

_MOST_PAIRS = 6.0e10  # candidate pairs of one exact sum: beyond, it would take too long
_CHUNK = 1 << 24


def _exact_pairs(pos, mass, n_active, prob, cot=None):
    """Forces [n_active, 3] (and with a cotangent the position gradient [n, 3]) by a float64 cell list."""
    n = int(pos.shape[0])
    x, m = pos.double(), mass.double()
    lo = torch.tensor(prob.lo, dtype=torch.float64, device=DEV)
    ln = torch.tensor(prob.len, dtype=torch.float64, device=DEV)
    nc = [max(1, int(v // prob.r_s)) for v in prob.len]
    ncd = torch.tensor(nc, device=DEV)
    ci = torch.floor((x - lo) / ln * ncd).long().clamp_min(0)
    ci = torch.minimum(ci, ncd - 1)
    cell = (ci[:, 0] * nc[1] + ci[:, 1]) * nc[2] + ci[:, 2]
    order = torch.argsort(cell)
    x, m, ci, cell = x[order], m[order], ci[order], cell[order]
    start = torch.searchsorted(cell, torch.arange(nc[0] * nc[1] * nc[2] + 1, device=DEV))
    active = order < n_active
    g = torch.zeros((n, 3), dtype=torch.float64, device=DEV)
    if cot is not None:
        g[active] = cot.double()[order[active]]
    acc, grad = torch.zeros_like(x), torch.zeros_like(x)
    rs2, e2 = float(prob.r_s) ** 2, float(prob.eps) ** 2
    nbs, total = [], 0.0
    for o in range(27):
        d = torch.tensor([o // 9 - 1, o // 3 % 3 - 1, o % 3 - 1], device=DEV)
        j = ci + d
        wrap = torch.div(j, ncd, rounding_mode="floor")
        j = j - wrap * ncd
        nb = (j[:, 0] * nc[1] + j[:, 1]) * nc[2] + j[:, 2]
        cnt = start[nb + 1] - start[nb]
        if not prob.periodic:
            cnt = torch.where((wrap != 0).any(dim=1), torch.zeros_like(cnt), cnt)
        total += float(cnt.sum())
        if total > _MOST_PAIRS:
            return None
        nbs.append((nb, cnt, wrap.double() * ln))
    for nb, cnt, shift in nbs:
        cum = torch.cumsum(cnt, 0)
        t0 = 0
        while t0 < n:
            before = int(cum[t0 - 1]) if t0 else 0
            t1 = max(t0 + 1, int(torch.searchsorted(cum, torch.tensor(before + _CHUNK, device=DEV), right=True)))
            c = cnt[t0:t1]
            i = torch.repeat_interleave(torch.arange(t0, t1, device=DEV), c)
            j = torch.arange(i.shape[0], device=DEV) - (cum[i] - cnt[i] - before) + start[nb[i]]
            d = x[j] + shift[i] - x[i]
            s = (d * d).sum(1)
            keep = (s < rs2) & (i != j)
            i, j, d, s = i[keep], j[keep], d[keep], s[keep]
            t = s + e2
            p, dp = torch.zeros_like(s), torch.zeros_like(s)
            for k in range(5, -1, -1):
                dp = dp * s + p
                p = p * s + prob.poly[k]
            f = t.pow(-1.5) - p
            lens = torch.bincount(i - t0, minlength=t1 - t0)
            acc[t0:t1] += torch.segment_reduce((m[j] * f)[:, None] * d, "sum", lengths=lens)
            if cot is not None:
                f1 = -1.5 * t.pow(-2.5) - dp
                u = m[i][:, None] * g[j] - m[j][:, None] * g[i]
                r = f[:, None] * u + (2.0 * f1 * (u * d).sum(1))[:, None] * d
                grad[t0:t1] += torch.segment_reduce(r, "sum", lengths=lens)
            t0 = t1
    out = torch.empty_like(acc)
    out[order] = acc
    if cot is None:
        return [out[:n_active]]
    og = torch.empty_like(grad)
    og[order] = grad
    return [out[:n_active], og]


def _exact_pk(case, seed):
    pos, mass, box = _pk_inputs(case, seed)
    ng, nb = case["ng"], case["ng"] // 2
    u = torch.remainder(pos.double() / (box / ng), ng)
    i0 = torch.floor(u).long() % ng
    f = u - torch.floor(u)
    rho = torch.zeros(ng ** 3, dtype=torch.float64, device=DEV)
    for c in range(8):
        w, at = mass.double(), 0
        for d in range(3):
            b = (c >> (2 - d)) & 1
            w = w * (f[:, d] if b else 1.0 - f[:, d])
            at = at * ng + (i0[:, d] + b) % ng
        rho.index_add_(0, at, w)
    dk = torch.fft.fftn(rho.view(ng, ng, ng) / rho.mean() - 1.0)
    n1 = torch.fft.fftfreq(ng, 1.0 / ng, dtype=torch.float64, device=DEV)
    w1 = torch.sinc(n1 / ng) ** 2
    win = w1[:, None, None] * w1[None, :, None] * w1[None, None, :]
    p = (dk.abs() / win) ** 2 * (box ** 3 / float(ng) ** 6)
    nn = torch.sqrt(n1[:, None, None] ** 2 + n1[None, :, None] ** 2 + n1[None, None, :] ** 2).reshape(-1)
    b = torch.floor(nn).long()
    sel = (b < nb) & (nn > 0)
    cnt = torch.bincount(b[sel], minlength=nb).clamp_min(1).double()
    pk = torch.bincount(b[sel], weights=p.reshape(-1)[sel], minlength=nb) / cnt
    km = torch.bincount(b[sel], weights=nn[sel] * (2.0 * math.pi / box), minlength=nb) / cnt
    return [pk, km, None]


def _exact_centres(case, seed):
    pos, mass, off = _halo_inputs(case, seed)
    c = np.diff(off).astype(np.float64)
    if float((c * c).sum()) > _MOST_PAIRS:
        return None
    x, m = pos.double(), mass.double()
    phi = torch.zeros(pos.shape[0], dtype=torch.float64, device=DEV)
    low = torch.zeros(case["halos"], dtype=torch.float64, device=DEV)
    e2 = float(np.float32(0.02)) ** 2
    for h in range(case["halos"]):
        a, b = int(off[h]), int(off[h + 1])
        rows = max(1, _CHUNK // max(1, b - a))
        for t0 in range(a, b, rows):
            t1 = min(b, t0 + rows)
            d2 = ((x[t0:t1, None, :] - x[None, a:b, :]) ** 2).sum(2) + e2
            phi[t0:t1] = m[t0:t1] / math.sqrt(e2) - (m[a:b] * d2.rsqrt()).sum(1)
        if b > a:
            low[h] = phi[a:b].min()
    return [phi, None, low]


def exact(case, seed):
    kind = case["kind"]
    if kind in ("force", "step", "autograd"):
        pos, mass, n_active, prob, cot = _domain(case, seed)
        return _exact_pairs(pos, mass, n_active, prob, None if kind == "force" else cot)
    if kind == "blocks":
        pos, mass, n_active, prob, cot = _domain(_blocks_case(case), seed)
        return _exact_pairs(pos, mass, n_active, prob, cot)
    if kind == "batch":
        if float(_batch_counts(case).sum()) > 3.0e7:
            return None
        pos, mass, counts, probs = _batch_inputs(case, seed)
        out, a = [], 0
        for nb, prob in zip(counts, probs):
            out += _exact_pairs(pos[a: a + int(nb)], mass[a: a + int(nb)], int(nb), prob)
            a += int(nb)
        return [torch.cat(out)]
    return _exact_pk(case, seed) if kind == "pk" else _exact_centres(case, seed)
