"""The work a user has the library do, as cases that can be timed and compared.

A case is a dict of plain values; ``prepare`` makes its inputs and whatever a
program keeps between calls (workspace, resident tree, mesh, batch), ``run``
is one pass through the public entry points, ``work`` says what the pass
cannot do without, and ``exact`` evaluates the same definition in 64 bits with
torch alone.

Kinds of case:
  * ``step``: build the tree and evaluate the short-range force on all
    particles, then free the tree: one time step of a program.  With
    ``mesh`` the long-range mesh force is accumulated onto it (full TreePM).
  * ``targets``: the force on a list of targets of a resident tree.
  * ``active``: the force on the active time-step levels of a resident tree.
  * ``batch``: many independent boxes, built and walked by one graph replay.
  * ``mesh``: the long-range force of caller-order particles.

Inputs: ``mixture`` (half uniform, half Plummer spheres, periodic unit box),
``zeldovich`` (a displaced grid, periodic), ``isolated`` (one Plummer sphere
in open space, Newtonian).  Parameters are scale-free in the particle number:
eps = 1/(40 N^(1/3)), r_s = 1.25/(2 N^(1/3)), r_cut = 4.5 r_s.
"""
import math

import torch

from paper_2609_17658_amd import og

DEV = "cuda"


def listed():
    step = {"kind": "step", "input": "mixture", "theta": 0.5, "precision": "mixed", "softening": "plummer",
            "criterion": "bh", "curve": "morton", "lists": "target", "lengths": False, "leaf_max": 8,
            "workspace": True, "mesh": 0}
    return [
        # a single small box, called as the README calls it (no workspace):
        # launches and host work count
        dict(step, name="step_1k", n=1000, workspace=False),
        # the parity box of the tests in full double precision
        dict(step, name="step_32k_fp64", n=32768, precision="fp64"),
        # a TreePM step of a small simulation: 64^3 particles, 128^3 mesh
        dict(step, name="treepm_64", n=262144, input="zeldovich", mesh=128),
        # a production setting (spline softening, relative criterion against
        # the previous accelerations, Peano-Hilbert order) at an odd size
        dict(step, name="step_487k_variants", n=486717, softening="spline", criterion="relative", curve="hilbert"),
        # the benchmark's headline box in both precisions
        dict(step, name="step_2m", n=2097152),
        dict(step, name="step_2m_fp64", n=2097152, precision="fp64"),
        # the largest box: 256^3 particles of a smooth early universe
        dict(step, name="step_16m", n=16777216, input="zeldovich"),
        # an isolated system in open space (no cutoff, bounding-cube root)
        dict(step, name="isolated_100k", n=100000, input="isolated"),
        # a few thousand targets of a resident tree
        dict(step, name="targets_5k", kind="targets", n=2097152, m=5000),
        # the active tenth of a resident tree (individual time steps)
        dict(step, name="active_1m", kind="active", n=1000000, share=0.1),
        # uneven independent boxes, replayed as a graph
        dict(step, name="batch_32", kind="batch", n=200000, boxes=32),
        # long-range force of caller-order particles on the headline's mesh
        dict(step, name="mesh_256", kind="mesh", n=2097152, mesh=256),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ranges: sizes over their logarithm, and
    the options in the mix a program meets."""
    kind = rng.choice(["step", "step", "step", "step", "targets", "active", "batch", "mesh"])
    c = {"kind": kind, "input": "mixture", "theta": rng.choice([0.4, 0.5, 0.5, 0.6, 0.7]), "precision": "mixed",
         "softening": rng.choice(["plummer", "plummer", "spline"]), "criterion": "bh",
         "curve": rng.choice(["morton", "hilbert"]), "lists": "target", "lengths": False,
         "leaf_max": rng.choice([8, 8, 8, 4, 16]), "workspace": rng.random() < 0.7, "mesh": 0}
    if kind == "step":
        c["input"] = rng.choice(["mixture", "mixture", "zeldovich", "isolated"])
        c["precision"] = rng.choice(["mixed", "mixed", "fp64"])
        if c["input"] == "isolated":
            c["n"] = _log_uniform(rng, 1000, 100000)
        elif c["input"] == "zeldovich":
            c["n"] = _log_uniform(rng, 10, 140 if c["precision"] == "mixed" else 100) ** 3
            if rng.random() < 0.5:
                c["mesh"] = 1 << max(4, math.ceil(math.log2(1.5 * c["n"] ** (1.0 / 3.0))))
        else:
            c["n"] = _log_uniform(rng, 1000, 2000000 if c["precision"] == "mixed" else 700000)
            if rng.random() < 0.25:
                c["criterion"] = "relative"
            elif rng.random() < 0.2:
                c["lengths"] = True
            elif rng.random() < 0.15:
                c["lists"] = "group"
    elif kind == "targets":
        c["n"] = _log_uniform(rng, 20000, 3000000)
        c["m"] = min(c["n"], _log_uniform(rng, 1, 100000))
    elif kind == "active":
        c["n"] = _log_uniform(rng, 20000, 2000000)
        c["share"] = round(math.exp(rng.uniform(math.log(0.002), 0.0)), 4)
    elif kind == "batch":
        c["n"] = _log_uniform(rng, 2000, 200000)  # largest box
        c["boxes"] = _log_uniform(rng, 2, 32)
        c["precision"] = rng.choice(["mixed", "mixed", "fp64"])
    else:
        c["mesh"] = 1 << rng.randint(4, 8)
        c["n"] = _log_uniform(rng, 1000, 2500000)
    return c


# ---------------------------------------------------------------- inputs --

def _generator(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _rand(shape, g):
    return torch.rand(shape, generator=g, dtype=torch.float64, device=DEV)


def _wrap(x):
    x = torch.remainder(x, 1.0)
    return torch.where(x >= 1.0, torch.zeros_like(x), x).contiguous()


def _plummer(n, a, g):
    """n offsets from a Plummer sphere of scale length a."""
    x = _rand(n, g).clamp_min(1e-12)
    r = a / torch.sqrt(x.pow(-2.0 / 3.0) - 1.0)
    mu = 2.0 * _rand(n, g) - 1.0
    phi = 2.0 * math.pi * _rand(n, g)
    s = torch.sqrt((1.0 - mu * mu).clamp_min(0.0))
    return torch.stack([r * s * torch.cos(phi), r * s * torch.sin(phi), r * mu], dim=1)


def _mixture(n, g):
    spheres, a = (8, 0.01) if n <= 300000 else (64, 0.005)
    half = n // 2
    centres = _rand((spheres, 3), g)
    which = torch.arange(n - half, device=DEV) % spheres
    cloud = centres[which] + _plummer(n - half, a, g)
    return _wrap(torch.cat([_rand((half, 3), g), cloud]))


def _zeldovich(n, g):
    """A side^3 grid displaced by the gradient of a Gaussian field with
    P(k) ~ k^-2 cut at the Nyquist wavenumber, rms displacement 0.3 cells."""
    side = round(n ** (1.0 / 3.0))
    white = torch.randn((side, side, side), generator=g, dtype=torch.float64, device=DEV)
    dk = torch.fft.rfftn(white)
    k1 = 2.0 * math.pi * torch.fft.fftfreq(side, d=1.0 / side, dtype=torch.float64, device=DEV)
    kz = 2.0 * math.pi * torch.fft.rfftfreq(side, d=1.0 / side, dtype=torch.float64, device=DEV)
    ks = [k1[:, None, None], k1[None, :, None], kz[None, None, :]]
    k2 = ks[0] * ks[0] + ks[1] * ks[1] + ks[2] * ks[2]
    keep = (k2 > 0) & (k2 <= (math.pi * side) ** 2)
    dk = torch.where(keep, dk / k2.clamp_min(1.0).pow(1.5), torch.zeros_like(dk))
    psi = torch.stack([torch.fft.irfftn(1j * k * dk, s=(side, side, side)) for k in ks], dim=-1)
    psi = psi * (0.3 / side / torch.sqrt((psi * psi).sum(-1).mean()).clamp_min(1e-300))
    q = (torch.arange(side, dtype=torch.float64, device=DEV) + 0.5) / side
    grid = torch.stack(torch.meshgrid(q, q, q, indexing="ij"), dim=-1)
    return _wrap((grid + psi).reshape(-1, 3))


def _inputs(case, seed):
    g = _generator(seed)
    n = case["n"]
    if case["input"] == "isolated":
        pos = (0.5 + _plummer(n, 0.05, g)).contiguous()
    elif case["input"] == "zeldovich":
        pos = _zeldovich(n, g)
    else:
        pos = _mixture(n, g)
    mass = ((0.5 + _rand(n, g)) / n).contiguous()
    return pos, mass, g


def _box_sizes(case):
    """Particle numbers of a batch's boxes: n, and others spread over the
    logarithm of [1000, n] (golden-ratio steps)."""
    lo, hi = math.log(1000.0), math.log(case["n"])
    return [case["n"]] + [int(round(math.exp(lo + (hi - lo) * (0.6180339887498949 * b % 1.0))))
                          for b in range(1, case["boxes"])]


def _lengths(n, eps, g):
    """Per-particle softening: 30 % at 5 eps, the rest at eps, scattered."""
    return eps * torch.where(_rand(n, g) < 0.3, 5.0, 1.0) * (0.8 + 0.4 * _rand(n, g))


def _params(case, n=None):
    side = (n or case["n"]) ** (1.0 / 3.0)
    p = {"G": 1.0, "eps": 1.0 / (40.0 * side), "r_s": 1.25 / (2.0 * side), "theta": case["theta"], "periodic": 1,
         "leaf_max": case["leaf_max"], "precision": case["precision"], "softening": case["softening"],
         "criterion": case["criterion"], "curve": case["curve"], "lists": case["lists"]}
    if case["mesh"]:
        p["r_s"] = 1.25 / case["mesh"]
    p["r_cut"] = 4.5 * p["r_s"]
    if case["criterion"] == "relative":
        p["alpha"] = 0.0025
    if case["input"] == "isolated":
        p.update(r_s=0.0, r_cut=0.0, periodic=0)
    return p


def _previous(acc):
    """Previous accelerations as a snapshot keeps them (single precision)."""
    return acc.float().double().contiguous()


# ------------------------------------------------------------------ runs --

def prepare(case, seed):
    stream = torch.cuda.current_stream()
    if case["kind"] == "batch":
        items = []
        for b, n in enumerate(_box_sizes(case)):
            pos, mass, _ = _inputs(dict(case, n=n), 1000 * seed + b)
            p = _params(case, n)
            p.pop("precision")
            items.append((pos, mass, 1.0, p))
        return {"case": case, "items": items,
                "batch": og.Batch(items, stream=stream, precision=case["precision"])}
    pos, mass, g = _inputs(case, seed)
    n = pos.shape[0]
    s = {"case": case, "pos": pos, "mass": mass, "params": _params(case), "stream": stream, "a_old": None,
         "workspace": None}
    if case["kind"] == "mesh":
        s["mesh"] = og.PM(case["mesh"], 1.0, 1.0, 1.25 / case["mesh"], stream=stream)
        return s
    if case["lengths"]:
        s["params"]["eps_particle"] = _lengths(n, s["params"]["eps"], g)
    if case["criterion"] == "relative":
        first = dict(s["params"], criterion="bh")
        tree = og.Tree(pos, mass, 1.0, first, stream=stream)
        s["a_old"] = _previous(tree.force(precision="fp64", with_pot=False)[0])
        tree.close()
    if case["kind"] == "step":
        if case["workspace"]:
            need = og.og_tree_workspace_bound(n, og.make_params(s["params"]))
            s["workspace"] = torch.empty(need, dtype=torch.uint8, device=DEV)
        if case["mesh"]:
            s["mesh"] = og.PM(case["mesh"], 1.0, 1.0, s["params"]["r_s"], stream=stream)
        return s
    s["tree"] = og.Tree(pos, mass, 1.0, s["params"], stream=stream)
    if case["kind"] == "targets":
        s["targets"] = torch.randperm(n, generator=g, device=DEV)[:case["m"]].contiguous()
    else:
        s["bin"] = _levels(case, pos, g)
        s["acc"] = torch.zeros((n, 3), dtype=torch.float64, device=DEV)
        s["pot"] = torch.zeros(n, dtype=torch.float64, device=DEV)
        s["count"] = torch.zeros(1, dtype=torch.int64, device=DEV)
    return s


def _levels(case, pos, g):
    """Time-step levels: `share` of the particles on levels 0 to 2, more of
    them in the second half of the list (the spheres), the rest above."""
    n = pos.shape[0]
    dense = (torch.arange(n, device=DEV) >= n // 2).double()
    on = _rand(n, g) < case["share"] * (0.5 + dense)
    low = torch.randint(0, 3, (n,), generator=g, device=DEV)
    return torch.where(on, low, low + 3).to(torch.int8)


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "batch":
        return [list(o) for o in s["batch"].replay()]
    if kind == "mesh":
        return s["mesh"].force(s["pos"], s["mass"])
    if kind == "targets":
        return s["tree"].force(targets=s["targets"])
    if kind == "active":
        s["tree"].force_active(s["bin"], 2, s["acc"], s["pot"], n_active=s["count"])
        return s["acc"], s["pot"], s["count"]
    tree = og.Tree(s["pos"], s["mass"], 1.0, s["params"], stream=s["stream"], workspace=s["workspace"])
    acc, pot = tree.force(a_old=s["a_old"])
    if case["mesh"]:
        s["mesh"].force_tree(tree, acc, pot, accumulate=True)
    tree.close()
    return acc, pot


# ------------------------------------------------------------------ work --

def _partners(case):
    """Partners per target of one walk, as measured on such boxes."""
    if case["input"] == "isolated":
        return 900.0 * (0.5 / case["theta"]) ** 2
    return (85.0 if case["input"] == "zeldovich" else 430.0) * (0.5 / case["theta"]) ** 2.1


def _mesh_work(case, n):
    cells = float(case["mesh"]) ** 3
    return 64.0 * n + 2 * 8.0 * cells, 250.0 * n + 5 * 5.0 * cells * math.log2(cells)


def work(case):
    """Bytes: positions and masses read, accelerations and potentials
    written (a mesh field once each way).  Operations: 42 per partner."""
    kind, n = case["kind"], float(case["n"])
    if kind == "mesh":
        b, f = _mesh_work(case, n)
        return {"bytes": b, "flops": f}
    if kind == "batch":
        n = float(sum(_box_sizes(case)))
    m = {"targets": float(case.get("m", 0)), "active": n * case.get("share", 1.0)}.get(kind, n)
    b = (32.0 * n if kind in ("step", "batch") else 32.0 * m) + 32.0 * m
    f = 42.0 * _partners(case) * m
    if kind == "step" and case["mesh"]:
        mb, mf = _mesh_work(case, n)
        b, f = b + mb, f + mf
    return {"bytes": b, "flops": f}


# ----------------------------------------------------------------- exact --
# The definition evaluated with torch in 64 bits: the octree of the level-21
# cells, the per-target walk rules, the softened short-range pair term, and
# the mesh force.

def _cells(x, lo, side):
    return ((x - lo) * (2097152.0 / side)).clamp(0.0, 2097151.0).to(torch.int64)


def _interleave(c):
    key = torch.zeros_like(c[:, 0])
    for b in range(21):
        for k in range(3):
            key |= ((c[:, k] >> b) & 1) << (3 * b + 2 - k)
    return key


def _octree(pos, mass, lo, side, leaf_max, eps):
    """Sorted particles and, per level, the nodes: first particle, count,
    cube centre, mass, centre of mass, length range, first child and number
    of children (0 for a leaf)."""
    key = _interleave(_cells(pos, lo, side))
    key, perm = torch.sort(key, stable=True)
    x, m = pos[perm], mass[perm]
    e = eps[perm] if eps is not None else None
    levels, inside = [], torch.ones(len(key), dtype=torch.bool, device=DEV)
    for level in range(22):
        at = torch.nonzero(inside).reshape(-1)
        if not len(at):
            break
        prefix, count = torch.unique_consecutive(key[at] >> (3 * (21 - level)), return_counts=True)
        first = at[torch.cumsum(count, 0) - count]
        drop, h = 21 - level, side * 2.0 ** -21
        corner = (_cells(x[first], lo, side) >> drop) << drop
        centre = lo + (corner.double() + 2.0 ** (20 - level)) * h
        node = torch.repeat_interleave(torch.arange(len(first), device=DEV), count)
        zero = torch.zeros(len(first), dtype=torch.float64, device=DEV)
        total = zero.index_add(0, node, m[at])
        moment = torch.zeros((len(first), 3), dtype=torch.float64, device=DEV)
        moment.index_add_(0, node, m[at, None] * (x[at] - centre[node]))
        t = {"first": first, "count": count, "centre": centre, "side": side * 2.0 ** -level, "m": total,
             "com": centre + moment / total[:, None]}
        if e is not None:
            t["emax"] = zero.scatter_reduce(0, node, e[at], "amax", include_self=False)
            t["emin"] = zero.scatter_reduce(0, node, e[at], "amin", include_self=False)
        internal = (count > leaf_max) & (level < 21)
        if level:
            up = levels[-1]
            parent = torch.searchsorted(up["prefix"], prefix >> 3)
            kids = torch.bincount(parent, minlength=len(up["first"]))
            up["kids"], up["kid0"] = kids, torch.cumsum(kids, 0) - kids
        t["prefix"] = prefix
        t["kids"] = t["kid0"] = torch.zeros_like(first)
        levels.append(t)
        inside = torch.zeros_like(inside)
        inside[at] = internal[node]
    return perm, x, m, e, levels


def _spline(r, h):
    u = r / h
    u2, u3 = u * u, u * u * u
    g0 = (32.0 / 3.0 - 192.0 / 5.0 * u2 + 32.0 * u3) / h ** 3
    w0 = (14.0 / 5.0 - 16.0 / 3.0 * u2 + 48.0 / 5.0 * u2 * u2 - 32.0 / 5.0 * u2 * u3) / h
    v = u.clamp_min(0.25)
    g1 = (64.0 / 3.0 - 48.0 * u + 192.0 / 5.0 * u2 - 32.0 / 3.0 * u3 - 1.0 / (15.0 * v ** 3)) / h ** 3
    w1 = (16.0 / 5.0 - 1.0 / (15.0 * v) - 32.0 / 3.0 * u2 + 16.0 * u3 - 48.0 / 5.0 * u2 * u2
          + 32.0 / 15.0 * u2 * u3) / h
    far = r.clamp_min(1e-300)
    g = torch.where(u < 0.5, g0, torch.where(u < 1.0, g1, far ** -3))
    w = torch.where(u < 0.5, w0, torch.where(u < 1.0, w1, 1.0 / far))
    return g, w


def _add_pairs(out, target, d, m, eps, p):
    """Adds the pair terms of partners of mass m at offsets d."""
    r2 = (d * d).sum(1)
    cut = p["r_s"] > 0
    if cut:
        keep = r2 < p["r_cut"] ** 2
        target, d, m, r2 = target[keep], d[keep], m[keep], r2[keep]
        eps = eps[keep] if isinstance(eps, torch.Tensor) else eps
    r = torch.sqrt(r2)
    if p["softening"] == "spline":
        g, w = _spline(r, 2.8 * eps)
    else:
        w = torch.rsqrt(r2 + eps * eps)
        g = w * w * w
    if cut:
        u = r / (2.0 * p["r_s"])
        tail = torch.erfc(u)
        g = g * (tail + 2.0 / math.sqrt(math.pi) * u * torch.exp(-u * u))
        w = w * tail
    out.index_add_(0, target, torch.cat([(m * g)[:, None] * d, -(m * w)[:, None]], dim=1))


def _image(d, p):
    return d - torch.round(d) if p["periodic"] else d


def _walk(pos, mass, p, targets=None, a_old=None):
    """Accelerations and potentials [M, 4] of the walk at the targets (caller
    indices; None: all)."""
    n = pos.shape[0]
    lo, side = torch.zeros(3, dtype=torch.float64, device=DEV), 1.0
    if not p["periodic"]:
        lo = pos.min(0).values
        side = float((pos.max(0).values - lo).max())
    perm, x, m, e, levels = _octree(pos, mass, lo, side, p["leaf_max"], p.get("eps_particle"))
    place = torch.empty_like(perm)
    place[perm] = torch.arange(n, device=DEV)
    want = torch.arange(n, device=DEV) if targets is None else targets
    out = torch.zeros((len(want), 4), dtype=torch.float64, device=DEV)
    order = torch.argsort(place[want])  # neighbours together: even chunks
    chunk = 1 << 16
    for c in range(0, len(want), chunk):
        row = order[c:c + chunk]
        me = place[want[row]]
        xt = x[me]
        et = e[me] if e is not None else None
        at = torch.linalg.norm(a_old[want[row]], dim=1) if a_old is not None else None
        got = torch.zeros((len(row), 4), dtype=torch.float64, device=DEV)
        tg = torch.arange(len(row), device=DEV)
        nd = torch.zeros_like(tg)
        for t in levels:
            if not len(tg):
                break
            s = t["side"]
            dc = _image(t["centre"][nd] - xt[tg], p).abs().amax(1)
            if p["r_s"] > 0:
                keep = dc <= p["r_cut"] + 0.5 * s
                tg, nd, dc = tg[keep], nd[keep], dc[keep]
            d = _image(t["com"][nd] - xt[tg], p)
            r2 = (d * d).sum(1)
            if p["criterion"] == "relative":
                opened = t["m"][nd] * s * s > p["alpha"] * at[tg] * r2 * r2
            else:
                opened = s * s > p["theta"] ** 2 * r2
            opened |= dc < 0.6 * s
            eps = p["eps"]
            if e is not None:
                hi = t["emax"][nd]
                opened |= (t["emin"][nd] < hi) & (hi > et[tg]) & (r2 < (2.8 * hi) ** 2)
                eps = torch.maximum(et[tg], hi)[~opened]
            far = ~opened
            _add_pairs(got, tg[far], d[far], t["m"][nd[far]], eps, p)
            tg, nd = tg[opened], nd[opened]
            kids = t["kids"][nd]
            leaf = kids == 0
            ltg, lnd = tg[leaf], nd[leaf]
            cnt = t["count"][lnd]
            at0 = torch.repeat_interleave(t["first"][lnd] - (torch.cumsum(cnt, 0) - cnt), cnt)
            j = at0 + torch.arange(len(at0), device=DEV)
            jt = torch.repeat_interleave(ltg, cnt)
            other = j != me[jt]
            j, jt = j[other], jt[other]
            eps = torch.maximum(et[jt], e[j]) if e is not None else p["eps"]
            _add_pairs(got, jt, _image(x[j] - xt[jt], p), m[j], eps, p)
            first = torch.repeat_interleave(t["kid0"][nd] - (torch.cumsum(kids, 0) - kids), kids)
            tg = torch.repeat_interleave(tg, kids)
            nd = first + torch.arange(len(first), device=DEV)
        out[row] = got
    return out


def _mesh(pos, mass, n, r_s):
    """Long-range acceleration and potential [N, 4] on an n^3 mesh."""
    u = pos * n
    i0 = torch.floor(u)
    f = u - i0
    i0 = i0.to(torch.int64) % n
    corners = []
    for c in range(8):
        b = torch.tensor([c >> 2 & 1, c >> 1 & 1, c & 1], device=DEV)
        i = (i0 + b) % n
        corners.append(((i[:, 0] * n + i[:, 1]) * n + i[:, 2], torch.where(b > 0, f, 1.0 - f).prod(1)))
    rho = torch.zeros(n ** 3, dtype=torch.float64, device=DEV)
    for i, w in corners:
        rho.index_add_(0, i, mass * w)
    rho_k = torch.fft.fftn((rho * float(n) ** 3).reshape(n, n, n))
    idx = torch.fft.fftfreq(n, d=1.0 / n, dtype=torch.float64, device=DEV)
    k = 2.0 * math.pi * idx
    kd = torch.where(idx == -(n // 2), torch.zeros_like(k), k)  # no derivative at the Nyquist wavenumber
    window = torch.sinc(idx / n) ** 4
    shape = [(n, 1, 1), (1, n, 1), (1, 1, n)]
    k2 = sum((k * k).reshape(s) for s in shape)
    w2 = window.reshape(shape[0]) * window.reshape(shape[1]) * window.reshape(shape[2])
    green = -4.0 * math.pi * torch.exp(-k2 * r_s * r_s) / k2.clamp_min(1.0) / w2
    green[0, 0, 0] = 0.0
    phi_k = green * rho_k
    out = torch.zeros((len(mass), 4), dtype=torch.float64, device=DEV)
    for col in range(4):
        field_k = phi_k if col == 3 else -1j * kd.reshape(shape[col]) * phi_k
        field = torch.fft.ifftn(field_k).real.reshape(-1)
        for i, w in corners:
            out[:, col] += w * field[i]
    out[:, 3] += mass / (math.sqrt(math.pi) * r_s)  # without the particle's own term
    return out


def exact(case, seed):
    kind = case["kind"]
    if case["lists"] == "group":
        return None  # the rules of a group's shared walk depend on the grouping
    if kind == "batch":
        both = []
        for b, n in enumerate(_box_sizes(case)):
            pos, mass, _ = _inputs(dict(case, n=n), 1000 * seed + b)
            o = _walk(pos, mass, _params(case, n))
            both.append([o[:, :3].contiguous(), o[:, 3].contiguous()])
        return both
    pos, mass, g = _inputs(case, seed)
    if kind == "mesh":
        o = _mesh(pos, mass, case["mesh"], 1.25 / case["mesh"])
        return o[:, :3].contiguous(), o[:, 3].contiguous()
    p = _params(case)
    n = pos.shape[0]
    if case["lengths"]:
        p["eps_particle"] = _lengths(n, p["eps"], g)
    a_old = targets = None
    if case["criterion"] == "relative":
        a_old = _previous(_walk(pos, mass, dict(p, criterion="bh"))[:, :3])
    if kind == "targets":
        targets = torch.randperm(n, generator=g, device=DEV)[:case["m"]]
    if kind == "active":
        on = torch.nonzero(_levels(case, pos, g) <= 2).reshape(-1)
        o = torch.zeros((n, 4), dtype=torch.float64, device=DEV)
        if len(on):
            o[on] = _walk(pos, mass, p, on)
        return o[:, :3].contiguous(), o[:, 3].contiguous(), None
    o = _walk(pos, mass, p, targets, a_old)
    if kind == "step" and case["mesh"]:
        o += _mesh(pos, mass, case["mesh"], p["r_s"])
    return o[:, :3].contiguous(), o[:, 3].contiguous()
