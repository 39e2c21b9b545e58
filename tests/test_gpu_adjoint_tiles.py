"""The adjoint's two sweeps around the sizes at which they differ: tiles of 8^3
(one tile, exact multiples, remainders of one cell and of seven), grids with an
axis under 8 (the level sweep), mixed batches, many problems on one output, and
gradients with infinities and NaN.  The reference solves the oracle's upwind
system by back substitution in descending |T| and counts its dependency levels.

Bar: both sides do the same few roundings per point and sum at most six
contributions in another order, so they agree to a few ulps of the largest
gradient; 1e-12 of it is the suite's bar for the adjoint on given T."""
import numpy as np
import pytest
import torch

from oracle import adjoint as oadj
from paper_1502_07303_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fmm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1502_07303_amd import fmm as m
    m.load_library()
    return m


def reference(F, h, T, status, g, scale=None):
    """(dL/dF, dependency levels) by back substitution."""
    sets = oadj.upwind_sets(F, h, T, status, scale)
    w = [1.0, 1.0, 1.0] if scale is None else [1.0 / (s * s) for s in scale]
    u, f, gf = np.abs(T.reshape(-1)), F.reshape(-1).astype(np.float64), g.reshape(-1)
    sign = np.where(T.reshape(-1) < 0.0, -1.0, 1.0)
    lt = {p: sign[p] * gf[p] for p, U in sets.items() if U}
    lev = {p: 1 for p in lt}
    out = np.zeros(T.size)
    with np.errstate(invalid="ignore"):
        for p in sorted(lt, key=lambda q: -u[q]):
            S = sum(w[ax] * (u[p] - u[q]) for q, ax in sets[p])
            out[p] = -(h * h) / (f[p] ** 3 * S) * lt[p]
            for q, ax in sets[p]:
                if q in lt:
                    lt[q] += w[ax] * (u[p] - u[q]) / S * lt[p]
                    lev[q] = max(lev[q], lev[p] + 1)
    return out.reshape(T.shape), max(lev.values(), default=0)


def solved(oracle_mod, shape, seed, dtype, scale=None, zero=0.0, width=np.inf):
    w = inputs.random_small(shape, n_sources=1 + seed % 2, seed=seed, dtype=dtype, zero_frac=zero)
    F, idx, val = w.numpy()
    T, st, _, _ = oracle_mod.solve(F, w.h, idx, val, width=width, axis_scale=scale)
    return F, w.h, T, st


SHAPES = [(8, 8, 8), (16, 8, 24), (9, 8, 15), (17, 9, 10), (15, 23, 8), (7, 12, 9), (1, 20, 30), (13, 1, 1)]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("dtype,scale", [(torch.float64, None), (torch.float32, None), (torch.float64, (1.0, 1.7, 0.6))])
def test_adjoint_shapes(fmm, oracle_mod, shape, dtype, scale):
    dev = torch.device("cuda:0")
    for seed, zero, width in ((1, 0.0, np.inf), (2, 0.1, np.inf), (3, 0.0, 0.3)):
        F, h, T, st = solved(oracle_mod, shape, seed, dtype, scale, zero, width)
        g = np.random.default_rng(seed).normal(size=shape)
        ref, levels = reference(F, h, T, st, g, scale)
        gF = torch.empty(shape, dtype=torch.float64, device=dev)
        a = fmm.AdjointSolver([{"F": torch.from_numpy(F).to(dev), "h": h, "T": torch.from_numpy(T).to(dev),
                                "status": torch.from_numpy(st).to(dev), "dL_dT": torch.from_numpy(g).to(dev),
                                "dL_dF": gF, "axis_scale": scale}])
        a.run()
        s = a.stats()
        assert s.n_levels == levels, (seed, s.n_levels, levels)
        assert np.max(np.abs(gF.cpu().numpy() - ref)) <= 1e-12 * max(np.max(np.abs(ref)), 1e-300), seed


@pytest.mark.parametrize("thin", [False, True])
def test_adjoint_mixed_batch(fmm, oracle_mod, thin):
    """Uneven grids and spacings in one batch; 70 problems on one output (more
    than one gather pass); with a thin grid the whole batch takes the other
    sweep."""
    dev = torch.device("cuda:0")
    probs, want, outs = [], [], []
    for k, (shape, scale) in enumerate([((9, 17, 8), None), ((12, 8, 21), (1.3, 1.0, 0.7)), ((16, 16, 16), None)] +
                                       ([((5, 9, 11), None)] if thin else [])):
        F, h, T, st = solved(oracle_mod, shape, 10 + k, torch.float64, scale)
        g = np.random.default_rng(k).normal(size=shape)
        want.append(reference(F, h, T, st, g, scale)[0])
        outs.append(torch.empty(shape, dtype=torch.float64, device=dev))
        probs.append({"F": torch.from_numpy(F).to(dev), "h": h, "T": torch.from_numpy(T).to(dev),
                      "status": torch.from_numpy(st).to(dev), "dL_dT": torch.from_numpy(g).to(dev),
                      "dL_dF": outs[-1], "axis_scale": scale})
    F, h, T, st = solved(oracle_mod, (10, 9, 8), 30, torch.float64)
    shared = torch.empty((10, 9, 8), dtype=torch.float64, device=dev)
    total = np.zeros((10, 9, 8))
    Fd, Td, sd = (torch.from_numpy(v).to(dev) for v in (F, T, st))
    for k in range(70):
        g = np.random.default_rng(100 + k).normal(size=total.shape)
        total += reference(F, h, T, st, g)[0]
        probs.insert(2 * k % len(probs), {"F": Fd, "h": h, "T": Td, "status": sd,
                                          "dL_dT": torch.from_numpy(g).to(dev), "dL_dF": shared})
    a = fmm.AdjointSolver(probs)
    for _ in range(2):
        a.run()
        a.stats()
        for o, r in zip(outs + [shared], want + [total]):
            assert np.max(np.abs(o.cpu().numpy() - r)) <= 1e-12 * np.max(np.abs(r))


def test_adjoint_special_gradients(fmm, oracle_mod):
    """Infinities and NaN, the NaN of all bits set among them, reach exactly the
    points they reach in the reference; nothing waits for them."""
    dev = torch.device("cuda:0")
    F, h, T, st = solved(oracle_mod, (18, 17, 20), 5, torch.float64)
    rng = np.random.default_rng(1)
    g = rng.normal(size=T.shape)
    at = rng.choice(T.size, size=12, replace=False)
    g.reshape(-1)[at[:4]] = np.inf
    g.reshape(-1)[at[4:8]] = np.nan
    g.reshape(-1).view(np.uint64)[at[8:]] = np.uint64(0xFFFFFFFFFFFFFFFF)
    g[T == T.max()] = np.nan
    ref, _ = reference(F, h, T, st, g)
    out = fmm.adjoint(*(torch.from_numpy(v).to(dev) if isinstance(v, np.ndarray) else v for v in (F, h, T, st, g)))
    out = out.cpu().numpy()
    assert np.array_equal(np.isnan(out), np.isnan(ref))
    assert np.array_equal(np.isinf(out), np.isinf(ref))
    fin = np.isfinite(ref)
    assert np.max(np.abs(out[fin] - ref[fin])) <= 1e-12 * np.max(np.abs(ref[fin]))


@pytest.mark.parametrize("k", [-1000, -960, -600, 600, 980])
def test_adjoint_extreme_gradients(fmm, oracle_mod, k):
    """A gradient times 2^k gives the adjoint times 2^k: the sweep's division
    without scaling hands over where its steps would under- or overflow.  Bar:
    the suite's 1e-12, point by point where the result is well above the
    subnormals (there the sums round as they do unscaled)."""
    dev = torch.device("cuda:0")
    F, h, T, st = solved(oracle_mod, (17, 9, 10), 3, torch.float64)
    g = np.random.default_rng(4).normal(size=F.shape)
    out = []
    for s in (0, k):
        gF = torch.empty(F.shape, dtype=torch.float64, device=dev)
        fmm.AdjointSolver([{"F": torch.from_numpy(F).to(dev), "h": h, "T": torch.from_numpy(T).to(dev),
                            "status": torch.from_numpy(st).to(dev), "dL_dT": torch.from_numpy(np.ldexp(g, s)).to(dev),
                            "dL_dF": gF}]).run()
        out.append(gF.cpu().numpy())
    well = np.abs(out[0]) > 1e-5 * np.max(np.abs(out[0]))
    assert well.sum() > F.size // 2
    assert np.all(np.abs(np.ldexp(out[1][well], -k) - out[0][well]) <= 1e-12 * np.abs(out[0][well]))


@pytest.mark.parametrize("dtype,scale", [(torch.float64, None), (torch.float32, (1.0, 1.7, 0.6))])
def test_adjoint_in_the_level_sweeps_workspace(fmm, oracle_mod, dtype, scale):
    """A workspace too small for the tiles but not for the level sweep is taken
    (the level sweep solves it: same levels, the suite's bar), one below is not."""
    dev = torch.device("cuda:0")
    F, h, T, st = solved(oracle_mod, (17, 9, 10), 5, dtype, scale)
    g = np.random.default_rng(6).normal(size=F.shape)
    ref, levels = reference(F, h, T, st, g, scale)
    for nbytes, ok in ((lambda full: full - 1, True), (lambda full: 30 * F.size + 8192, True),
                       (lambda full: 28 * F.size, False)):
        gF = torch.empty(F.shape, dtype=torch.float64, device=dev)
        a = fmm.AdjointSolver([{"F": torch.from_numpy(F).to(dev), "h": h, "T": torch.from_numpy(T).to(dev),
                                "status": torch.from_numpy(st).to(dev), "dL_dT": torch.from_numpy(g).to(dev),
                                "dL_dF": gF, "axis_scale": scale}])
        a.nbytes = nbytes(a.nbytes)
        if not ok:
            with pytest.raises(fmm.FmmError):
                a.run()
            continue
        a.run()
        assert a.stats().n_levels == levels
        assert np.max(np.abs(gF.cpu().numpy() - ref)) <= 1e-12 * np.max(np.abs(ref))


def test_adjoint_written_over_the_model(fmm, oracle_mod):
    """dL_dF may be the memory of an F, of its own problem or of another (every
    input is read before an output is written).  Bar: the suite's 1e-12."""
    dev = torch.device("cuda:0")
    qs, refs = [], []
    for seed in (1, 2):
        F, h, T, st = solved(oracle_mod, (17, 9, 10), seed, torch.float64)
        g = np.random.default_rng(seed).normal(size=F.shape)
        refs.append(reference(F, h, T, st, g)[0])
        qs.append({"F": torch.from_numpy(F).to(dev), "h": h, "T": torch.from_numpy(T).to(dev),
                   "status": torch.from_numpy(st).to(dev), "dL_dT": torch.from_numpy(g).to(dev)})
    models = [q["F"].clone() for q in qs]
    for own in (True, False):
        for q, m in zip(qs, models):
            q["F"].copy_(m)
        for k in range(2):
            qs[k]["dL_dF"] = qs[k if own else 1 - k]["F"]
        a = fmm.AdjointSolver(qs)
        a.run()
        a.stats()
        for q, ref in zip(qs, refs):
            assert np.max(np.abs(q["dL_dF"].cpu().numpy() - ref)) <= 1e-12 * np.max(np.abs(ref)), own
