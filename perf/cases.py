"""The work that a user has this library do, as cases with inputs, one pass and
what a pass cannot do without.

Every case goes through the Python binding's public entry points.  The field
``kind`` names the entry point:

- ``solve``: `fmm.Solver.solve_into`, a reused solve context (T and status);
- ``noalloc``: `fmm.solve_noalloc_into`, the solve without a workspace;
- ``batch``: `fmm.BatchSolver.solve`, many problems in one launch;
- ``adjoint``: `fmm.AdjointSolver.run`, dL/dF of solved problems;
- ``train``: `fmm.EikonalShots`, forward and backward under autograd.

``field`` names the speeds: ``one`` (F = 1, case 3 of the paper), ``iid``
(independent uniform speeds in [0.5, 2], rough media), ``gauss`` (log-normal
field clipped to [0.25, 4], the random-speed workload), ``smooth`` (2^tanh(g),
the batch workload), ``tomo`` (max(1 + 0.3 g, 0.1), the tomography model),
``case4`` to ``case6`` (the paper's Eqs. 14 to 16; case 6 has barriers) and
``spheres`` (F = 1, two-sided reinitialisation around a union of spheres).
``stride_h`` is the restart stride in units of h, 0 for the library's default.
"""
import math

import numpy as np
import torch

from paper_1502_07303_amd import fmm, inputs

DTYPES = {"f32": torch.float32, "f64": torch.float64}


def _case(name, kind, shape, field, dtype="f64", sources=1, stride_h=0.0, width=math.inf, barriers=0.0,
          scale=(1.0, 1.0, 1.0), problems=1):
    c = {"name": name, "kind": kind, "n0": shape[0], "n1": shape[1], "n2": shape[2], "field": field, "dtype": dtype,
         "sources": sources, "stride_h": float(stride_h), "width": 0.0 if math.isinf(width) else float(width),
         "barriers": float(barriers), "s0": float(scale[0]), "s1": float(scale[1]), "s2": float(scale[2]),
         "problems": problems}
    if name is None:
        del c["name"]
    return c


def listed():
    return [
        # the smallest call: one small local travel-time problem of a serving
        # loop that allocates nothing; launches and restart latency count
        _case("noalloc_24x20x28", "noalloc", (24, 20, 28), "iid", "f64", sources=2),
        # a ragged grid (no axis a multiple of the tile edge), FP32 speeds with
        # impassable points, a reused solver
        _case("ragged_37x29x45_f32", "solve", (37, 29, 45), "iid", "f32", sources=2, barriers=0.06),
        # distance from one point on a uniform grid, the paper's case 3 at its
        # recommended stride
        _case("point_64", "solve", (64, 64, 64), "one"),
        # the paper's case 6: the front winds through perforated shells, many
        # restarts with little work in each
        _case("shells_64", "solve", (64, 64, 64), "case6"),
        # a grid with another spacing along each axis, rough FP64 speeds
        _case("spacing_101x87x118", "solve", (101, 87, 118), "iid", "f64", sources=2, stride_h=3.0,
              scale=(1.0, 1.7, 0.6)),
        # level-set reinitialisation: both sides of eight spheres out to a band
        _case("spheres_256", "solve", (256, 256, 256), "spheres", "f64", sources=8, width=0.1),
        # first arrivals in a random medium, the headline workload, on the
        # largest grid it is used on and at the stride its autotuner picks
        _case("random_1024_f32", "solve", (1024, 1024, 1024), "gauss", "f32", sources=4, stride_h=3.5),
        # the same medium with FP64 speeds on a middle-sized odd grid, at the
        # default stride
        _case("random_301x256x333_f64", "solve", (301, 256, 333), "gauss", "f64", sources=4),
        # many uneven problems at once (edges 32 to 192), tuned stride
        _case("batch_64", "batch", (32, 192, 0), "smooth", "f64", sources=4, stride_h=4.0, problems=64),
        # a small gradient: one source, a ragged grid, FP32 speeds
        _case("adjoint_40x33x52_f32", "adjoint", (40, 33, 52), "smooth", "f32"),
        # the tomography gradient: sixteen shots over one model summed into one dL/dF
        _case("adjoint_256_shots16", "adjoint", (256, 256, 256), "tomo", "f64", stride_h=4.0, problems=16),
        # one step of a travel-time inversion as a training loop takes it:
        # forward, misfit at receivers, backward
        _case("train_96_shots4", "train", (96, 96, 96), "tomo", "f64", stride_h=4.0, problems=4),
    ]


def _edge(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _shape(rng, lo, hi):
    """Three edges around one size between lo and hi, each its own."""
    e = _edge(rng, lo, hi)
    return tuple(max(lo, min(hi, int(round(e * rng.uniform(0.75, 1.3))))) for _ in range(3))


def draw(rng):
    kind = rng.choice(["noalloc", "solve", "solve", "solve", "batch", "adjoint", "adjoint", "train"])
    dtype = rng.choice(["f32", "f64"])
    stride_h = rng.choice([0.0, 2.0, 3.0, 3.5, 4.0])
    if kind == "noalloc":
        return _case(None, kind, _shape(rng, 16, 140), rng.choice(["iid", "smooth"]), dtype, rng.randint(1, 4),
                     stride_h)
    if kind == "solve":
        field = rng.choice(["one", "iid", "gauss", "gauss", "case4", "case6", "spheres"])
        if field == "spheres":
            n = _edge(rng, 64, 320)
            return _case(None, kind, (n, n, n), field, "f64", rng.randint(2, 8), stride_h, rng.uniform(0.05, 0.2))
        if field in ("case4", "case6"):
            n = _edge(rng, 32, 200)
            return _case(None, kind, (n, n, n), field, "f64", 1, stride_h)
        shape = _shape(rng, 24, 560)
        scale = (1.0, 1.0, 1.0)
        if rng.random() < 0.25:
            scale = tuple(round(rng.uniform(0.5, 2.0), 2) for _ in range(3))
        return _case(None, kind, shape, field, dtype, rng.randint(1, 4), stride_h,
                     barriers=0.06 if field == "iid" and rng.random() < 0.5 else 0.0, scale=scale)
    if kind == "batch":
        lo = _edge(rng, 12, 64)
        hi = lo + _edge(rng, 8, 128)
        return _case(None, kind, (lo, hi, 0), "smooth", dtype, 4, stride_h, problems=_edge(rng, 4, 64))
    if kind == "adjoint":
        shots = rng.choice([1, 2, 4, 8])
        return _case(None, kind, _shape(rng, 16, 256), rng.choice(["smooth", "tomo"]), dtype, 1, stride_h,
                     problems=shots)
    return _case(None, kind, _shape(rng, 24, 128), "tomo", rng.choice(["f32", "f64"]), 1, stride_h,
                 problems=rng.randint(1, 6))


# ---------------------------------------------------------------------------
# Inputs

def _speeds(field, shape, dtype, seed, device, barriers=0.0):
    n = max(shape)
    if field in ("one", "spheres"):
        return torch.ones(shape, dtype=dtype, device=device)
    if field == "iid":
        gen = torch.Generator(device=device)
        gen.manual_seed(seed)
        F = 0.5 + 1.5 * torch.rand(shape, generator=gen, dtype=torch.float64, device=device)
        if barriers > 0.0:
            F[torch.rand(shape, generator=gen, device=device) < barriers] = 0.0
        return F.to(dtype)
    if field in ("case4", "case6"):
        return inputs.paper_case(int(field[4:]), n, device=device).F.to(dtype)
    if field == "gauss":
        g = inputs.gaussian_field(n, seed, 0.05, device=device, shape=shape)
        return torch.clamp(torch.exp(0.5 * g), 0.25, 4.0).to(dtype).contiguous()
    g = inputs.gaussian_field(n, seed, 0.1, device=device, shape=shape)
    if field == "smooth":
        return torch.exp(math.log(2.0) * torch.tanh(g)).to(dtype).contiguous()
    return torch.clamp(1.0 + 0.3 * g, min=0.1).to(dtype).contiguous()


def _spheres(n, count, seed, device):
    """Seeds next to the surface of a union of spheres, valued by the signed
    distance function (as `inputs.spheres`, on the device)."""
    rng = np.random.default_rng(seed)
    centres = rng.uniform(0.2, 0.8, size=(count, 3))
    radii = rng.uniform(0.05, 0.2, size=count)
    x = torch.arange(n, dtype=torch.float64, device=device) * (1.0 / (n - 1))
    phi = torch.full((n, n, n), math.inf, dtype=torch.float64, device=device)
    for c, r in zip(centres.tolist(), radii.tolist()):
        d = ((x - c[0]) ** 2)[:, None, None] + ((x - c[1]) ** 2)[None, :, None] + ((x - c[2]) ** 2)[None, None, :]
        phi = torch.minimum(phi, torch.sqrt(d) - r)
    neg, adj = phi < 0, phi == 0
    for ax in range(3):
        flip = neg.narrow(ax, 0, n - 1) != neg.narrow(ax, 1, n - 1)
        adj.narrow(ax, 0, n - 1).logical_or_(flip)
        adj.narrow(ax, 1, n - 1).logical_or_(flip)
    idx = torch.nonzero(adj.reshape(-1)).reshape(-1)
    return idx, phi.reshape(-1)[idx].contiguous()


def _scale(case):
    s = (case["s0"], case["s1"], case["s2"])
    return None if s == (1.0, 1.0, 1.0) else s


def _width(case):
    return case["width"] or math.inf


def _stride(case, h):
    return case["stride_h"] * h if case["stride_h"] else None


def _one(case, seed, device):
    """Speeds, spacing and seeds of a solve."""
    shape = (case["n0"], case["n1"], case["n2"])
    h = 1.0 / (max(shape) - 1)
    F = _speeds(case["field"], shape, DTYPES[case["dtype"]], seed, device, case["barriers"])
    if case["field"] == "spheres":
        idx, val = _spheres(shape[0], case["sources"], seed, device)
        return F, h, idx, val
    if case["field"] in ("one", "case4", "case6"):
        # the source near the centre (inside the innermost shell of case 6)
        rng = np.random.default_rng(seed + 7919)
        c = [n // 2 + int(rng.integers(-(n // 16), n // 16 + 1)) for n in shape]
        at = np.array([(c[0] * shape[1] + c[1]) * shape[2] + c[2]])
    else:
        rng = np.random.default_rng(seed + 7919)
        at = np.sort(rng.choice(F.numel(), size=case["sources"], replace=False))
    idx = torch.from_numpy(at.astype(np.int64)).to(device)
    if case["barriers"]:
        F.view(-1)[idx] = 1.0  # sources lie in the medium
    return F, h, idx, torch.zeros(len(at), dtype=torch.float64, device=device)


def _batch(case, seed, device):
    """The problems of a batch: edges from n0 to n1, one to four sources each."""
    rng = np.random.default_rng(1000 + case["problems"])  # the sizes belong to the case, not to the seed
    edges = [int(e) for e in rng.integers(case["n0"], case["n1"] + 1, size=case["problems"])]
    rng = np.random.default_rng(seed)
    out = []
    for i, n in enumerate(edges):
        F = _speeds(case["field"], (n, n, n), DTYPES[case["dtype"]], seed * 1009 + i, device)
        at = np.sort(rng.choice(n ** 3, size=int(rng.integers(1, case["sources"] + 1)), replace=False))
        out.append({"F": F, "h": 1.0 / (n - 1), "seed_idx": torch.from_numpy(at.astype(np.int64)).to(device),
                    "seed_val": torch.zeros(len(at), dtype=torch.float64, device=device)})
    return out


def _shots(case, seed, device):
    """One model, point sources on its first face of axis 2, receivers on the
    last, and a misfit gradient at the receivers of each shot."""
    shape = (case["n0"], case["n1"], case["n2"])
    h = 1.0 / (max(shape) - 1)
    F = _speeds(case["field"], shape, DTYPES[case["dtype"]], seed, device)
    rng = np.random.default_rng(seed + 31337)
    face = shape[0] * shape[1]
    src = rng.choice(face, size=case["problems"], replace=False) * shape[2]
    rec = rng.choice(face, size=min(1024, face // 4), replace=False) * shape[2] + shape[2] - 1
    seeds = [(torch.tensor([int(s)], dtype=torch.int64, device=device),
              torch.zeros(1, dtype=torch.float64, device=device)) for s in src]
    rec = torch.from_numpy(rec.astype(np.int64)).to(device)
    w = torch.from_numpy(rng.normal(size=(case["problems"], rec.numel()))).to(device)
    return F, h, seeds, rec, w


class _State:
    def __init__(self, case, **kw):
        self.case = case
        self.__dict__.update(kw)


def prepare(case, seed):
    dev = torch.device("cuda")
    kind = case["kind"]
    if kind in ("solve", "noalloc"):
        F, h, idx, val = _one(case, seed, dev)
        T = torch.empty(F.shape, dtype=torch.float64, device=dev)
        status = torch.empty(F.shape, dtype=torch.uint8, device=dev)
        if kind == "noalloc":
            opts = fmm.make_opts(band_width=_width(case), stride=_stride(case, h), axis_scale=_scale(case))
            return _State(case, F=F, h=h, idx=idx, val=val, T=T, status=status, opts=opts)
        solver = fmm.Solver(F.shape, idx.numel(), h, band_width=_width(case), stride=_stride(case, h), device=dev,
                            speed_dtype=F.dtype, axis_scale=_scale(case))
        return _State(case, F=F, idx=idx, val=val, T=T, status=status, solver=solver)
    if kind == "batch":
        probs = _batch(case, seed, dev)
        # the outputs of all problems in one buffer, as a caller that goes on
        # with them as one array keeps them
        sizes = [p["F"].numel() for p in probs]
        T = torch.empty(sum(sizes), dtype=torch.float64, device=dev)
        status = torch.empty(sum(sizes), dtype=torch.uint8, device=dev)
        Ts = [v.view(p["F"].shape) for v, p in zip(T.split(sizes), probs)]
        sts = [v.view(p["F"].shape) for v, p in zip(status.split(sizes), probs)]
        solver = fmm.BatchSolver(probs, stride_h=case["stride_h"] or None, T_out=Ts, status_out=sts)
        return _State(case, solver=solver, T=T, status=status)
    F, h, seeds, rec, w = _shots(case, seed, dev)
    if kind == "train":
        opts = {"stride_h": case["stride_h"]} if case["stride_h"] else {}
        return _State(case, F=F, h=h, seeds=seeds, rec=rec, w=w, opts=opts)
    # an adjoint call has the forward solution in hand
    probs, dF = [], torch.empty(F.shape, dtype=torch.float64, device=dev)
    b = fmm.BatchSolver([{"F": F, "h": h, "seed_idx": i, "seed_val": v} for i, v in seeds],
                        stride_h=case["stride_h"] or None)
    b.solve()
    b.stats()
    for k in range(len(seeds)):
        gT = torch.zeros(F.shape, dtype=torch.float64, device=dev)
        gT.view(-1)[rec] = w[k]
        probs.append({"F": F, "h": h, "T": b.T[k], "status": b.status[k], "dL_dT": gT, "dL_dF": dF})
    return _State(case, solver=fmm.AdjointSolver(probs), dF=dF)


def run(s):
    kind = s.case["kind"]
    if kind == "solve":
        s.solver.solve_into(s.F, s.idx, s.val, s.T, s.status)
        return s.T, s.status
    if kind == "noalloc":
        fmm.solve_noalloc_into(s.F, s.h, s.idx, s.val, s.T, s.status, opts=s.opts)
        return s.T, s.status
    if kind == "batch":
        s.solver.solve()
        return s.T, s.status
    if kind == "adjoint":
        s.solver.run()
        return s.dF
    F = s.F.detach().requires_grad_(True)
    T, status = fmm.EikonalShots.apply(F, s.h, s.seeds, s.opts)
    loss = (T.reshape(len(s.seeds), -1)[:, s.rec] * s.w).sum()
    loss.backward()
    return {"T": T.detach(), "status": status, "dL_dF": F.grad}


def work(case):
    """Each input read once, each output written once; operations of one local
    solve per point (about 40: ordering, three discriminants, two roots)."""
    f = 4 if case["dtype"] == "f32" else 8
    if case["kind"] == "batch":
        rng = np.random.default_rng(1000 + case["problems"])
        n = int(sum(int(e) ** 3 for e in rng.integers(case["n0"], case["n1"] + 1, size=case["problems"])))
        return {"bytes": n * (f + 9), "flops": 40 * n}
    n = case["n0"] * case["n1"] * case["n2"]
    m = case["problems"]
    if case["kind"] in ("solve", "noalloc"):
        return {"bytes": n * (f + 9), "flops": 40 * n}
    if case["kind"] == "adjoint":
        # T, status and dL/dT of each shot, F and dL/dF once
        return {"bytes": n * (17 * m + f + 8), "flops": 25 * n * m}
    return {"bytes": n * (9 * m + 17 * m + 2 * f), "flops": 65 * n * m}


# ---------------------------------------------------------------------------
# The same results in plain torch, 64 bits: the discrete upwind equations as a
# fixed point of whole-grid updates.

EXACT_POINTS = 2_200_000


def _neighbours(T, ax, fill):
    """Values of the minus and the plus neighbour along an axis."""
    pad = torch.full_like(T.narrow(ax, 0, 1), fill)
    n = T.shape[ax]
    return (torch.cat([pad, T.narrow(ax, 0, n - 1)], ax), torch.cat([T.narrow(ax, 1, n - 1), pad], ax))


def _root(a, w, r):
    """Smallest causal root of sum_i w_i max(u - a_i, 0)^2 = r^2 and how many
    of the sorted values it uses (first-order Godunov)."""
    order = torch.argsort(torch.stack(a), dim=0, stable=True)
    a = torch.gather(torch.stack(a), 0, order)
    w = torch.tensor(w, dtype=torch.float64, device=a.device)[order]
    inf = torch.full_like(r, math.inf)
    u = torch.where(torch.isfinite(a[0]), a[0] + r / torch.sqrt(w[0]), inf)
    used = torch.isfinite(a[0]).to(torch.int64)
    for k in (2, 3):
        W = w[:k].sum(0)
        spread = torch.zeros_like(r)
        for i in range(k):
            for j in range(i + 1, k):
                spread = spread + w[i] * w[j] * (a[j] - a[i]) ** 2
        D = W * r * r - spread
        v = ((w[:k] * a[:k]).sum(0) + torch.sqrt(torch.clamp(D, min=0.0))) / W
        ok = torch.isfinite(a[k - 1]) & (D >= 0) & (v > a[k - 1]) & (v < u)
        u = torch.where(ok, v, u)
        used = torch.where(ok, torch.full_like(used, k), used)
    return u, used


def _march(F, h, idx, val, scale):
    """|T| of one side: seeds fixed, F <= 0 never solved."""
    w = [1.0 / (s * s) for s in (scale or (1.0, 1.0, 1.0))]
    F = F.to(torch.float64)
    T = torch.full(F.shape, math.inf, dtype=torch.float64, device=F.device)
    T.view(-1)[idx] = val
    free = F > 0
    free.view(-1)[idx] = False
    r = torch.where(free, h / torch.where(free, F, torch.ones_like(F)), torch.full_like(F, math.inf))
    while True:
        a = [torch.minimum(*_neighbours(T, ax, math.inf)) for ax in range(3)]
        u, _ = _root(a, w, torch.where(free, r, torch.ones_like(r)))
        new = torch.where(free, torch.minimum(T, u), T)
        if torch.equal(new, T):
            return T
        T = new


def _gradient(F, h, T, idx, g):
    """dL/dF of one shot (uniform spacing, one side): the transposed
    linearised equations, swept until nothing changes."""
    F = F.to(torch.float64)
    solved = torch.isfinite(T) & (F > 0)
    solved.view(-1)[idx] = False
    nb = [_neighbours(T, ax, math.inf) for ax in range(3)]
    a = [torch.where(torch.minimum(*p) < T, torch.minimum(*p), torch.full_like(T, math.inf)) for p in nb]
    _, used = _root(a, [1.0, 1.0, 1.0], h / F)
    rank = torch.argsort(torch.argsort(torch.stack(a), dim=0, stable=True), dim=0, stable=True)
    zero = torch.zeros_like(T)
    # weight of the upwind value on each axis, and on which side it lies
    d = [torch.where(solved & (rank[ax] < used), T - a[ax], zero) for ax in range(3)]
    S = torch.where(solved, d[0] + d[1] + d[2], torch.ones_like(T))
    minus = [(nb[ax][0] <= nb[ax][1]) for ax in range(3)]
    lt = torch.where(solved, g, zero)
    while True:
        new = torch.where(solved, g, zero)
        for ax in range(3):
            c = d[ax] / S * lt
            lo, hi = torch.where(minus[ax], c, zero), torch.where(minus[ax], zero, c)
            new = new + _neighbours(lo, ax, 0.0)[1] + _neighbours(hi, ax, 0.0)[0]
        new = torch.where(solved, new, zero)
        if torch.equal(new, lt):
            return torch.where(solved, -(h * h) / (F ** 3 * S) * lt, zero)
        lt = new


def _exact_shot(F, h, idx, g):
    T = _march(F, h, idx, torch.zeros(1, dtype=torch.float64, device=F.device), None)
    return T, _gradient(F, h, T, idx, g(T))


def exact(case, seed):
    dev = torch.device("cuda" if torch.cuda.is_available() else "cpu")
    kind = case["kind"]
    if kind == "batch":
        rng = np.random.default_rng(1000 + case["problems"])
        edges = rng.integers(case["n0"], case["n1"] + 1, size=case["problems"])
        if sum(int(e) ** 3 for e in edges) > EXACT_POINTS:
            return None
        T = [_march(p["F"], p["h"], p["seed_idx"], p["seed_val"], None).reshape(-1) for p in _batch(case, seed, dev)]
        return torch.cat(T), None
    if case["n0"] * case["n1"] * case["n2"] * case["problems"] > EXACT_POINTS:
        return None
    if kind in ("solve", "noalloc"):
        F, h, idx, val = _one(case, seed, dev)
        if case["field"] != "spheres":
            T = _march(F, h, idx, val, _scale(case))
            return torch.where(T <= _width(case), T, torch.full_like(T, math.inf)), None
        # the seeds separate the two sides: each is marched with the other's seeds as walls
        side = []
        for neg in (False, True):
            here = (val < 0) == neg
            walls = F.clone()
            walls.view(-1)[idx[~here]] = 0.0
            side.append(_march(walls, h, idx[here], val[here].abs(), None))
        a = torch.minimum(side[0], side[1])
        T = torch.where(side[1] < side[0], -a, a)
        T = torch.where(a <= _width(case), T, torch.full_like(T, math.inf))
        T.view(-1)[idx] = val  # seeds come back as they were given
        return T, None
    F, h, seeds, rec, w = _shots(case, seed, dev)
    Ts, total = [], 0.0
    for k, (idx, _) in enumerate(seeds):
        g = torch.zeros(F.shape, dtype=torch.float64, device=dev)
        g.view(-1)[rec] = w[k]
        T, dF = _exact_shot(F, h, idx, lambda T: g)
        Ts.append(T)
        total = total + dF
    if kind == "adjoint":
        return total
    return {"T": torch.stack(Ts), "status": None, "dL_dF": total}
