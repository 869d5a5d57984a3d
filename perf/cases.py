"""The work whose speed is measured: relaxation calls over the range of sizes, regions and options a user runs.

``listed()`` names twelve cases and ``draw()`` gives more of the same ranges; ``prepare()`` makes a case's inputs
and context, ``run()`` is one pass through the public binding, ``work()`` the bytes and operations a pass cannot do
without, and ``exact()`` the same pass in 64 bits with plain torch.

A pass loads a particle set, relaxes it by a few steps and fetches the result, with the metrics a program logs at
that interval; or it is one gradient evaluation of the relaxation loss.  Passes are short because trajectories are
chaotic: after many steps two correct builds no longer agree in their last digits.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1906_07925_amd import mpsph as M

KAPPA, TAU, SIGMA0, NU, C_ACC, C_VEL, C_VISC = 2.0, 1.3, 3.0, 0.1, 0.25, 1.0 / 40.0, 0.125
METRICS = ("residual_l2", "kinetic", "dt1", "dt2", "elr_mean")   # what a program logs of a run
N_RBF, RBF_WIDTH, MESH = 32, 0.15, 48


# ------------------------------------------------------------------------------------------
# Cases
# ------------------------------------------------------------------------------------------

def _case(name, region, n, colours, init, steps, **kw):
    c = {"name": name, "region": region, "n": n, "colours": colours, "init": init, "steps": steps,
         "graph": False, "metrics": False, "cell_log2": 0, "lanes": 0}
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call: one eager step of a thousand 2D particles (an interactive preview, a unit test)
        _case("square_1k", "square", 1024, 4, "lattice", 1, metrics=True),
        # the paper's small square in its inner loop: ten steps as one graph, then the log line
        _case("square_4k_graph", "square", 4096, 4, "lattice", 10, graph=True, metrics=True),
        # a small region whose boundary carries its own particles (types, mirror rule), odd count
        _case("ball_seeded_20k", "ball", 20011, 8, "seeded", 4, metrics=True),
        # a periodic box, odd lattice side (37^3): the minimum-image kernels
        _case("periodic_50k", "periodic", 50653, 8, "lattice", 4, graph=True),
        # an ordinary graded 3D mesh near its target density, prime count
        _case("cube_100k", "cube", 100003, 16, "graded", 4, metrics=True),
        # the graded annulus from a random start, as the configurations have it
        _case("annulus_262k", "annulus", 262144, 16, "random", 2, metrics=True),
        # a region and size field given only on a background mesh
        _case("levelset_262k", "levelset", 262144, 16, "random", 2),
        # several sub-domains of uneven size advanced together, 2D and 3D mixed, replayed as a graph
        _case("batch_12", "batch", 360000, 8, "random", 5, graph=True, metrics=True),
        # a gradient evaluation of an optimisation loop, small: launches and host work count
        _case("grad_8k", "rbf_cube", 8192, 16, "lattice", 4, ckpt=2),
        # the same at a quarter of the benchmark's size
        _case("grad_262k", "rbf_cube", 262144, 16, "lattice", 4, ckpt=2),
        # a large mesh in the late part of a run (particles distributed by the target density), library defaults
        _case("cube_1m_relaxed", "cube", 1000003, 64, "graded", 2),
        # the benchmark's cube at the configuration its autotuner picks, from the jittered lattice
        _case("cube_2m", "cube", 2097152, 64, "lattice", 2, cell_log2=6, lanes=8, metrics=True),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["square", "square", "annulus", "periodic", "cube", "cube", "ball", "levelset", "batch",
                       "rbf_cube"])
    colours = rng.choice([2, 4, 8, 16, 32, 64])
    graph = rng.random() < 0.5
    metrics = rng.random() < 0.5
    if kind == "square":
        side = _logint(rng, 24, 400)
        return _draw("square", side * side, colours, "lattice", 1 if side > 100 else rng.randint(1, 8), graph, metrics)
    if kind == "annulus":
        return _draw("annulus", _logint(rng, 2000, 262144), colours, "random", rng.randint(1, 2), graph, metrics)
    if kind == "periodic":
        side = _logint(rng, 10, 64)
        return _draw("periodic", side ** 3, colours, "lattice", rng.randint(1, 4), graph, metrics)
    if kind == "cube":
        n = _logint(rng, 4000, 1000003)
        lanes = rng.choice([0, 0, 8])
        return _draw("cube", n, colours, "graded", rng.randint(1, 2), graph, metrics, lanes=lanes)
    if kind == "ball":
        return _draw("ball", _logint(rng, 2000, 200000), colours, "seeded", rng.randint(1, 3), graph, metrics)
    if kind == "levelset":
        return _draw("levelset", _logint(rng, 8000, 262144), colours, "random", rng.randint(1, 2), graph, metrics)
    if kind == "batch":
        return _draw("batch", _logint(rng, 20000, 360000), colours, "random", rng.randint(1, 4), graph, metrics)
    return _draw("rbf_cube", _logint(rng, 2000, 262144), colours, "lattice", rng.randint(1, 3), False, False,
                 ckpt=rng.randint(1, 3))


def _draw(region, n, colours, init, steps, graph, metrics, **kw):
    c = _case("", region, n, colours, init, steps, graph=graph, metrics=metrics, **kw)
    del c["name"]
    return c


# ------------------------------------------------------------------------------------------
# Regions and size fields
# ------------------------------------------------------------------------------------------

def _spec(region, n):
    """The region with its size field at unit scale (s0 = 1), as the binding takes it."""
    if region == "square":
        return dict(dim=2, geometry="box", lo=(0.0,) * 2, hi=(1.0,) * 2, field="uniform", n=n)
    if region == "annulus":   # spacing grows 1:4 from the inner to the outer circle
        return dict(dim=2, geometry="annulus", lo=(-1.0,) * 2, hi=(1.0,) * 2, centre=(0.0,) * 2, r_in=0.2, r_out=1.0,
                    field="radial_linear", fcentre=(0.0,) * 2, fa=3.0 / 0.8, fb=0.2, n=n)
    if region == "periodic":
        return dict(dim=3, geometry="periodic", lo=(0.0,) * 3, hi=(1.0,) * 3, field="uniform", n=n)
    if region == "cube":      # spacing graded 1:4 with the distance to an embedded sphere
        return dict(dim=3, geometry="box", lo=(0.0,) * 3, hi=(1.0,) * 3, field="sphere_distance", fcentre=(0.5,) * 3,
                    fa=3.0 / (math.sqrt(3.0) / 2.0 - 0.25), fb=0.25, n=n)
    if region == "plain_cube":
        return dict(dim=3, geometry="box", lo=(0.0,) * 3, hi=(1.0,) * 3, field="uniform", n=n)
    if region in ("ball", "plain_ball"):
        return dict(dim=3, geometry="ball", lo=(0.0,) * 3, hi=(1.0,) * 3, centre=(0.5,) * 3, r_out=0.5,
                    field="uniform", seeded=region == "ball", n=n)
    if region == "levelset":  # a ball of radius 0.4 graded 1:3 from its centre, sampled on a background mesh
        ax = np.linspace(0.0, 1.0, MESH) - 0.5
        r = np.sqrt(ax[:, None, None] ** 2 + ax[None, :, None] ** 2 + ax[None, None, :] ** 2).reshape(-1)
        return dict(dim=3, geometry="levelset", lo=(0.0,) * 3, hi=(1.0,) * 3, field="grid", grid_n=(MESH,) * 3,
                    grid_phi=0.4 - r, grid_s=1.0 + 2.0 * np.minimum(r / 0.4, 1.5), n=n)
    if region == "rbf_cube":
        return dict(dim=3, geometry="box", lo=(0.0,) * 3, hi=(1.0,) * 3, field="rbf_exp", n_rbf=N_RBF,
                    rbf_width=RBF_WIDTH, rbf_coeff=np.zeros(N_RBF), n=n)
    raise KeyError(region)


def _relative_spacing(spec, x, coeff=None):
    """s(x) / s0 at the rows of x (float64)."""
    f = spec["field"]
    if f == "uniform":
        return torch.ones(x.shape[0], dtype=x.dtype, device=x.device)
    if f in ("radial_linear", "sphere_distance"):
        t = (x - x.new_tensor(spec["fcentre"])).norm(dim=1) - spec["fb"]
        return 1.0 + spec["fa"] * (t.abs() if f == "sphere_distance" else t)
    if f == "grid":
        return _mesh(spec, "grid_s", x)[0]
    mu = x.new_tensor(np.asarray(spec["rbf_centre"]))
    g = torch.exp(-((x[:, None, :] - mu) ** 2).sum(-1) / (2.0 * spec["rbf_width"] ** 2))
    return torch.exp(g @ coeff)


def _mesh(spec, key, x):
    """Multilinear interpolant of the background mesh's node values and its gradient."""
    m, d = MESH, x.shape[1]
    v = x.new_tensor(np.asarray(spec[key]))
    u = x * (m - 1)
    b = u.detach().floor().clamp(0, m - 2)
    f = u - b
    b = b.long()
    val, grad = 0.0, [0.0] * d
    for cn in range(1 << d):
        bits = [(cn >> a) & 1 for a in range(d)]
        idx = sum((b[:, a] + bits[a]) * m ** a for a in range(d))
        w = [f[:, a] if bits[a] else 1.0 - f[:, a] for a in range(d)]
        val = val + math.prod(w) * v[idx]
        for a in range(d):
            rest = math.prod([w[c] for c in range(d) if c != a])
            grad[a] = grad[a] + (1.0 if bits[a] else -1.0) * (m - 1) * rest * v[idx]
    return val, torch.stack(grad, dim=1)


def _inside(spec, x):
    g = spec["geometry"]
    if g == "levelset":
        return (x - 0.5).norm(dim=1) < 0.4
    if g in ("box", "periodic"):
        return torch.ones(x.shape[0], dtype=torch.bool, device=x.device)
    r = (x - x.new_tensor(spec["centre"])).norm(dim=1)
    return (r <= spec["r_out"]) & (r >= spec.get("r_in", 0.0))


def _lattice_points(spec, m):
    """Midpoints of an m^dim grid over the bounding box that lie in the region, and their cell volume."""
    lo, hi = spec["lo"], spec["hi"]
    ax = [torch.linspace(0.0, 1.0, 2 * m + 1, dtype=torch.float64)[1::2] * (hi[a] - lo[a]) + lo[a]
          for a in range(spec["dim"])]
    x = torch.stack(torch.meshgrid(*ax, indexing="ij"), dim=-1).reshape(-1, spec["dim"])
    vol = math.prod((hi[a] - lo[a]) / m for a in range(spec["dim"]))
    return x[_inside(spec, x)], vol


_SCALE: dict = {}


def _scale(region, n):
    """Field scale for which the target density integrates to n over the region."""
    if region == "rbf_cube":
        return n ** (-1.0 / 3.0)
    if region not in _SCALE:
        spec = _spec(region, n)
        x, vol = _lattice_points(spec, 400 if spec["dim"] == 2 else 64)
        _SCALE[region] = float((_relative_spacing(spec, x) ** -spec["dim"]).sum() * vol)
    return (_SCALE[region] / n) ** (1.0 / _spec(region, n)["dim"])


# ------------------------------------------------------------------------------------------
# Inputs (made from the seed, on the GPU)
# ------------------------------------------------------------------------------------------

def _uniform(spec, m, gen, accept=None):
    """m points uniform in the region, thinned by accept(x) (a probability) where given."""
    lo = torch.tensor(spec["lo"], dtype=torch.float64, device="cuda")
    hi = torch.tensor(spec["hi"], dtype=torch.float64, device="cuda")
    out, have = [], 0
    while have < m:
        x = torch.rand((max(2 * (m - have), 4096), spec["dim"]), generator=gen, device="cuda", dtype=torch.float64)
        x = lo + (hi - lo) * x
        x = x[_inside(spec, x)]
        if accept is not None:
            x = x[torch.rand(x.shape[0], generator=gen, device="cuda", dtype=torch.float64) < accept(x)]
        out.append(x)
        have += x.shape[0]
    return torch.cat(out)[:m]


def _points(case, spec, n, gen):
    """Initial positions (float64) and types."""
    d, init = spec["dim"], case["init"]
    types = torch.zeros(n, dtype=torch.int32, device="cuda")
    if init == "lattice":     # cell-centred lattice, jittered by a quarter spacing; surplus sites dropped at random
        side = int(math.ceil(n ** (1.0 / d) - 1e-9))
        g = torch.stack(torch.meshgrid(*[torch.arange(side, device="cuda")] * d, indexing="ij"), dim=-1).reshape(-1, d)
        x = (g + 0.5 + 0.5 * (torch.rand(g.shape, generator=gen, device="cuda", dtype=torch.float64) - 0.5)) / side
        keep = torch.randperm(x.shape[0], generator=gen, device="cuda")[:n].sort().values
        lo, hi = x.new_tensor(spec["lo"]), x.new_tensor(spec["hi"])
        return lo + (hi - lo) * x[keep], types
    if init == "graded":      # distributed by the target density, as late in a run
        return _uniform(spec, n, gen, lambda x: _relative_spacing(spec, x) ** -d), types
    if init == "seeded":      # a random interior and a boundary sphere (Fibonacci spiral) with its share of the particles
        ns = int(round(4.0 * math.pi * 0.25 / _scale(case["region"], n) ** 2))
        k = torch.arange(ns, device="cuda", dtype=torch.float64) + 0.5
        z = 1.0 - 2.0 * k / ns
        ph = k * (math.pi * (3.0 - math.sqrt(5.0))) + 2.0 * math.pi * torch.rand((), generator=gen, device="cuda")
        r = torch.sqrt(1.0 - z * z)
        surf = 0.5 + 0.5 * (1.0 - 1e-6) * torch.stack([r * torch.cos(ph), r * torch.sin(ph), z], dim=1)
        x = torch.cat([_uniform(spec, n - ns, gen), surf])
        types[n - ns:] = 1
        mix = torch.randperm(n, generator=gen, device="cuda")
        return x[mix], types[mix]
    return _uniform(spec, n, gen), types


def _domain(case, region, n, gen):
    """One domain: spec with its field scale, float32 positions, colours, types."""
    spec = _spec(region, n)
    spec["s0"] = _scale(region, n)
    if region == "rbf_cube":
        spec["rbf_centre"] = torch.rand((N_RBF, 3), generator=gen, device="cuda", dtype=torch.float64).cpu().numpy()
    x, types = _points(case, spec, n, gen)
    seeds = _uniform(spec, case["colours"], gen)
    colour = torch.cat([torch.cdist(c, seeds).argmin(dim=1) for c in x.split(1 << 18)]).to(torch.int32)
    return spec, x.to(torch.float32), colour, types


def _inputs(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    if case["region"] != "batch":
        return [_domain(case, case["region"], case["n"], gen)], gen
    # twelve domains of four kinds, counts spread by a factor of about fifty
    share = [math.exp(4.0 * ((k * 5) % 12) / 11.0) for k in range(12)]
    kinds = ("square", "annulus", "plain_cube", "plain_ball")
    return [_domain(case, kinds[k % 4], max(64, int(case["n"] * share[k] / sum(share))), gen) for k in range(12)], gen


def prepare(case, seed):
    doms, gen = _inputs(case, seed)
    specs, xs, cols, types = zip(*doms)
    one = len(doms) == 1
    R = M.Relaxer(specs[0] if one else list(specs), n=specs[0]["n"] if one else [s["n"] for s in specs],
                  s0=specs[0]["s0"] if one else [s["s0"] for s in specs])
    if case["cell_log2"] or case["lanes"]:
        R.configure(case["cell_log2"] or -1, case["lanes"] or 4)
    state = {"case": case, "relaxer": R, "x": xs[0] if one else torch.cat([x.reshape(-1) for x in xs]),
             "colour": torch.cat(cols), "type": torch.cat(types) if case["init"] == "seeded" else None}
    if "ckpt" in case:
        state["coeff"] = _coefficients(gen).requires_grad_()
        state["x"].requires_grad_()
        state["loss"] = M.relax_loss_function()
    return state


def _coefficients(gen):
    """RBF coefficients of the size field as an optimiser holds them (float32, host)."""
    return (0.1 * torch.randn(N_RBF, generator=gen, device="cuda", dtype=torch.float32)).cpu()


# ------------------------------------------------------------------------------------------
# One pass
# ------------------------------------------------------------------------------------------

def run(state):
    case, R = state["case"], state["relaxer"]
    if "ckpt" in case:
        coeff, x = state["coeff"], state["x"]
        coeff.grad = x.grad = None
        loss = state["loss"].apply(coeff, x, R, state["colour"], state["type"], case["steps"], case["ckpt"], 1.0)
        loss.backward()
        return {"loss": loss.item(), "grad_coeff": coeff.grad, "grad_x": x.grad}
    R.load(state["x"], state["colour"], state["type"])
    if case["graph"]:
        R.step_graph(case["steps"])
    else:
        R.step(case["steps"])
    x, types = R.store()
    out = {"x": x, "type": types}
    if case["metrics"]:
        out["metrics"] = [[m[k] for k in METRICS] for m in R.domain_metrics()]
    return out


# ------------------------------------------------------------------------------------------
# What a pass cannot do without
# ------------------------------------------------------------------------------------------

def _pairs_per_particle(case, region):
    """Mean number of neighbours within the cut-off for the case's initial distribution."""
    spec = _spec(region, case["n"])
    d = spec["dim"]
    ball = math.pi if d == 2 else 4.0 * math.pi / 3.0
    if case["init"] == "graded" or spec["field"] in ("uniform", "rbf_exp"):
        return ball * (KAPPA * TAU) ** d
    x, vol = _lattice_points(spec, 64 if d == 2 else 24)
    s = _relative_spacing(spec, x)
    # uniform density n / V against the target s^-d
    return ball * (KAPPA * TAU) ** d * float((s ** d).mean() * (s ** -d).mean())


def work(case):
    """Bytes: positions, colours and types in, positions and types out.  Operations: per step, the 38 + 34 of the
    two pair sums for each ordered pair (2D: 29 + 27); a gradient adds the loss, its reverse and the reverse of every
    step, counted at twice the forward's operations."""
    kinds = ("square", "annulus", "plain_cube", "plain_ball") if case["region"] == "batch" else (case["region"],)
    flops = nbytes = 0.0
    for kind in kinds:
        n, d = case["n"] / len(kinds), _spec(kind, case["n"])["dim"]
        pairs = n * _pairs_per_particle(case, kind)
        per = 72.0 if d == 3 else 56.0
        flops += pairs * per * (3.0 * case["steps"] + 1.0 if "ckpt" in case else case["steps"])
        nbytes += n * (4 * d + 4 + 4 * d + (0 if "ckpt" in case else 4) + (4 if case["init"] == "seeded" else 0))
    return {"bytes": nbytes, "flops": flops}


# ------------------------------------------------------------------------------------------
# The same pass in 64 bits (Eq. 16-32 of the paper, plain torch)
# ------------------------------------------------------------------------------------------

def _neighbours(spec, x, reach):
    """Ordered pairs i != j with |x_i - x_j| < max(reach_i, reach_j), by bins no smaller than the largest reach."""
    d = x.shape[1]
    lo, hi = x.new_tensor(spec["lo"]), x.new_tensor(spec["hi"])
    length = float((hi - lo).max())
    periodic = spec["geometry"] == "periodic"
    nb = max(1, min(int(length / float(reach.max())), 12 if d == 3 else 40))
    b = ((x - lo) * (nb / length)).long().clamp(0, nb - 1)
    flat = sum(b[:, a] * nb ** a for a in range(d))
    order = flat.argsort()
    start = torch.searchsorted(flat[order], torch.arange(nb ** d + 1, device=x.device)).tolist()
    xo, ro = x[order], reach[order]
    out_i, out_j = [], []
    for cell in range(nb ** d):
        i0, i1 = start[cell], start[cell + 1]
        if i0 == i1:
            continue
        c = [cell // nb ** a % nb for a in range(d)]
        near = [sorted({(c[a] + o) % nb for o in (-1, 0, 1)} if periodic else
                       {k for k in (c[a] - 1, c[a], c[a] + 1) if 0 <= k < nb}) for a in range(d)]
        cells = [0]
        for a in reversed(range(d)):
            cells = [q * nb + k for q in cells for k in near[a]]
        cand = torch.cat([torch.arange(start[q], start[q + 1], device=x.device) for q in cells])
        for s in range(i0, i1, max(1, (1 << 26) // max(1, cand.numel()))):
            e = min(i1, s + max(1, (1 << 26) // max(1, cand.numel())))
            r2 = 0.0
            for a in range(d):
                u = xo[s:e, a, None] - xo[cand, a]
                if periodic:
                    u = u - length * torch.round(u / length)
                r2 = r2 + u * u
            i, j = torch.nonzero(r2 < torch.maximum(ro[s:e, None], ro[cand]) ** 2, as_tuple=True)
            i, j = i + s, cand[j]
            keep = i != j
            out_i.append(order[i[keep]])
            out_j.append(order[j[keep]])
    return torch.cat(out_i), torch.cat(out_j)


def _separation(spec, x, i, j):
    u = x[i] - x[j]
    if spec["geometry"] == "periodic":
        length = spec["hi"][0] - spec["lo"][0]
        u = u - length * torch.round(u.detach() / length)
    return u


def _safe_norm(v):
    n2 = (v * v).sum(-1)
    ok = n2 > 0
    return torch.where(ok, torch.sqrt(torch.where(ok, n2, 1.0)), 0.0)


def _normals(spec, x):
    """Unit normal of the region's level set at the rows of x (round and mesh regions)."""
    g = _mesh(spec, "grid_phi", x)[1] if spec["geometry"] == "levelset" else x - x.new_tensor(spec["centre"])
    return g / g.norm(dim=1, keepdim=True)


def _map_force(spec, x, t, f):
    """Force mapping of feature particles (Eq. 30-31)."""
    g = spec["geometry"]
    f = torch.where((t == 3)[:, None], torch.zeros_like(f), f)
    if g == "box":
        xd = x.detach()
        on = (xd == x.new_tensor(spec["lo"])) | (xd == x.new_tensor(spec["hi"]))
        return torch.where(on & (t > 0)[:, None], torch.zeros_like(f), f)
    if g == "periodic":
        return f
    nrm = _normals(spec, x)
    return torch.where((t > 0)[:, None], f - (f * nrm).sum(-1, keepdim=True) * nrm, f)


def _map_position(spec, x, t):
    """Closest-point projection and re-tagging, or the mirror rule of seeded features (Eq. 32)."""
    g, d = spec["geometry"], x.shape[1]
    lo, hi = x.new_tensor(spec["lo"]), x.new_tensor(spec["hi"])
    if g == "periodic":
        return torch.remainder(x - lo, hi - lo) + lo, t
    if g == "box":
        x = torch.maximum(torch.minimum(x, hi), lo)
        xd = x.detach()
        nf = ((xd == lo) | (xd == hi)).sum(-1)
        tag = torch.tensor([0, 1, 2 if d == 3 else 3, 3], device=x.device, dtype=t.dtype)[nf]
        return x, torch.where(t == 3, t, torch.maximum(t, tag))
    if g == "levelset":
        phi, grad = _mesh(spec, "grid_phi", x)
        out = (t > 0) | (phi < 0)
        return torch.where(out[:, None], x - phi[:, None] * grad / grad.norm(dim=1, keepdim=True), x), \
            torch.where(out & (t == 0), torch.ones_like(t), t)
    c = x.new_tensor(spec["centre"])
    r = (x - c).norm(dim=1)
    r_in, r_out = spec.get("r_in", 0.0), spec["r_out"]
    inner = r - r_in < r_out - r if g == "annulus" else torch.zeros_like(t, dtype=torch.bool)
    phi = torch.minimum(r - r_in, r_out - r) if g == "annulus" else r_out - r
    out = (t > 0) | (phi < 0)
    rb = torch.where(inner, torch.full_like(r, r_in), torch.full_like(r, r_out))
    if spec.get("seeded"):
        rb = torch.where(t == 0, torch.where(r > r_out, 2 * r_out - r, 2 * r_in - r), rb)
    x = torch.where(out[:, None], c + (rb / r)[:, None] * (x - c), x)
    return x, t if spec.get("seeded") else torch.where(out & (t == 0), torch.ones_like(t), t)


def _step(spec, x, colour, t, coeff=None):
    """One relaxation step; returns positions, types and the logged metrics."""
    n, d = x.shape
    alpha = 7.0 / (4.0 * math.pi) if d == 2 else 21.0 / (16.0 * math.pi)
    s = spec["s0"] * _relative_spacing(spec, x, coeff)
    h = TAU * s
    rho_t = s ** -d
    i, j = _neighbours(spec, x.detach(), KAPPA * h.detach())
    u = _separation(spec, x, i, j)
    r = _safe_norm(u)
    hij = 0.5 * (h[i] + h[j])
    near = r < KAPPA * hij
    act = (near & (t[j] >= t[i]) & (r > 0)).to(x.dtype)
    rs = torch.where(r > 0, r, 1.0)
    q = r / hij
    slope = alpha * hij ** (-d - 1) * (-5.0 * q) * (1.0 - 0.5 * q).clamp(min=0.0) ** 3 / rs * act
    inv2 = s[i] ** (2 * d) + s[j] ** (2 * d)
    beta = SIGMA0 * (colour[i] != colour[j])
    a = torch.zeros_like(x).index_add(0, i, (-(1.0 + beta) * inv2 * slope)[:, None] * u)
    a = _map_force(spec, x, t, a)
    am = _safe_norm(a)
    free = (t != 3) & (am > 0)
    rc = KAPPA * h
    dt1 = (C_ACC * torch.sqrt(rc / torch.where(free, am, 1.0)))[free].min()
    vt = 0.5 * dt1 * a * (t != 3)[:, None]
    vm = _safe_norm(vt)
    eta = rho_t * NU * rc * vm
    es = eta[i] + eta[j]
    harm = torch.where(es > 0, 2.0 * eta[i] * eta[j] / torch.where(es > 0, es, 1.0), 0.0)
    at = torch.zeros_like(x).index_add(0, i, (harm * inv2 * slope)[:, None] * (vt[i] - vt[j]))
    at = _map_force(spec, x, t, at)
    vs = torch.where(free, vm, 1.0)
    dt2 = torch.stack([dt1, (C_VEL * rc / vs)[free].min(), (C_VISC * rc / (NU * vs))[free].min()]).min()
    v = (vt + 0.5 * dt2 * at) * (t != 3)[:, None]
    metrics = None
    if not x.requires_grad:
        w = (1.0 - 0.5 * r / h[i]).clamp(min=0.0) ** 4 * (1.0 + 2.0 * r / h[i])
        rho = alpha * h ** -d * (1.0 + torch.zeros_like(h).index_add(0, i, w))
        normal = t == 0
        res = torch.sqrt((((rho / rho_t - 1.0) ** 2)[normal]).mean())
        nn = torch.full_like(h, math.inf).scatter_reduce(0, i[near], r[near], "amin")
        ok = normal & torch.isfinite(nn)
        metrics = [float(res), float(0.5 * (v * v).sum()), float(dt1), float(dt2), float((nn / s)[ok].mean())]
    x, t = _map_position(spec, x + dt2 * v, t)
    return x, t, metrics


def _loss(spec, x, colour, coeff):
    n, d = x.shape
    alpha = 21.0 / (16.0 * math.pi)
    h = TAU * spec["s0"] * _relative_spacing(spec, x, coeff)
    i, j = _neighbours(spec, x.detach(), KAPPA * h.detach())
    r = _safe_norm(_separation(spec, x, i, j))

    def w(q):
        return (1.0 - 0.5 * q).clamp(min=0.0) ** 4 * (1.0 + 2.0 * q)

    e = alpha * TAU ** -d * (1.0 + torch.zeros_like(h).index_add(0, i, w(r / h[i]))) - 1.0
    ifc = (w(r / (0.5 * (h[i] + h[j]))) * (colour[i] != colour[j])).sum() * 0.5
    return ((e * e).sum() + ifc) / n


def exact(case, seed):
    doms, gen = _inputs(case, seed)
    if "ckpt" in case:
        spec, x, colour, t = doms[0]
        coeff = _coefficients(gen).double().cuda().requires_grad_()
        x0 = x.double().requires_grad_()
        # each step is recomputed in the reverse pass from its stored start, so that one step's pairs are held at a time
        xs, ts = [x0.detach()], [t]
        with torch.no_grad():
            for _ in range(case["steps"]):
                y, u, _ = _step(spec, xs[-1], colour, ts[-1], coeff.detach())
                xs.append(y)
                ts.append(u)
        y = xs[-1].clone().requires_grad_()
        loss = _loss(spec, y, colour, coeff)
        gx, gc = torch.autograd.grad(loss, (y, coeff))
        for k in reversed(range(case["steps"])):
            y = xs[k].clone().requires_grad_()
            z, _, _ = _step(spec, y, colour, ts[k], coeff)
            gy, dc = torch.autograd.grad(z, (y, coeff), grad_outputs=gx)
            gx, gc = gy, gc + dc
        return {"loss": float(loss.detach()), "grad_coeff": gc, "grad_x": gx}
    out, logs = [], []
    with torch.no_grad():
        for spec, x, colour, t in doms:
            x, m = x.double(), None
            for _ in range(case["steps"]):
                x, t, m = _step(spec, x, colour, t)
            out.append(x)
            logs.append(m)
    got = {"x": out[0] if len(out) == 1 else torch.cat([x.reshape(-1) for x in out]), "type": None}
    if case["metrics"]:
        got["metrics"] = logs
    return got
