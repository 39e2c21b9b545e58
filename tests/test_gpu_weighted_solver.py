"""The local solvers bit for bit through whole solves: on a grid whose even cells
are all seeds, every odd cell is one evaluation of the solver from its six seeds,
so its T does not depend on any order.  The reference writes the general form out
in numpy (IEEE divisions and roots): all discriminants, roots and comparisons, for
uniform and per-axis spacing, speeds and seed values over wide ranges, values
around both decisions and ties.  Bar: every bit."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def general(v, s, r, weighted):
    """The smallest causal root: v (3, n) upwind values, s per-axis factors."""
    s = np.repeat(np.asarray(s, dtype=np.float64)[:, None], v.shape[1], 1)
    a, s = v.copy(), s.copy()
    for i, j in ((0, 1), (1, 2), (0, 1)):
        c = a[i] > a[j]
        a[i], a[j] = np.where(c, a[j], a[i]), np.where(c, a[i], a[j])
        s[i], s[j] = np.where(c, s[j], s[i]), np.where(c, s[i], s[j])
    a1, a2, a3 = a
    r2 = r * r
    with np.errstate(all="ignore"):
        d12, d13, d23 = a2 - a1, a3 - a1, a3 - a2
        if weighted:
            w1, w2, w3 = 1.0 / (s * s)
            best = a1 + r * s[0]
            D2 = (w1 + w2) * r2 - (w1 * w2) * (d12 * d12)
            u2 = ((w1 * a1 + w2 * a2) + np.sqrt(D2)) / (w1 + w2)
            D3 = ((w1 + w2) + w3) * r2 - (((w1 * w2) * (d12 * d12) + (w1 * w3) * (d13 * d13)) + (w2 * w3) * (d23 * d23))
            u3 = (((w1 * a1 + w2 * a2) + w3 * a3) + np.sqrt(D3)) / ((w1 + w2) + w3)
        else:
            best = a1 + r
            D2 = 2.0 * r2 - d12 * d12
            u2 = ((a1 + a2) + np.sqrt(D2)) * 0.5
            D3 = 3.0 * r2 - ((d12 * d12 + d13 * d13) + d23 * d23)
            u3 = (((a1 + a2) + a3) + np.sqrt(D3)) / 3.0
        best = np.where((a2 < np.inf) & (D2 >= 0.0) & (u2 > a2) & (u2 < best), u2, best)
        best = np.where((a3 < np.inf) & (D3 >= 0.0) & (u3 > a3) & (u3 < best), u3, best)
    return best


SCALES = [None, (1.0, 1.7, 0.6), (3.0, 3.0, 3.0), (1e-3, 1.0, 1e3), (1e-60, 2e-60, 1e-60), (1e100, 1e99, 1e100),
          (1e-160, 1e-150, 1.0)]


@pytest.mark.parametrize("scale", SCALES)
@pytest.mark.parametrize("kind", ["plain", "ties", "decisions", "wide"])
def test_solver_bits(kind, scale):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1502_07303_amd import fmm
    dev = torch.device("cuda:0")
    n = (40, 44, 48)
    rng = np.random.default_rng(3)
    s = (1.0, 1.0, 1.0) if scale is None else scale
    h = 2.0 ** -5
    F = rng.uniform(0.5, 2.0, n)
    V = rng.uniform(0.0, 1.0, n) * h
    if kind == "wide":
        F = np.exp2(rng.uniform(-400, 400, n))
        V = np.exp2(rng.uniform(-420, 400, n))
    V *= max(s) if kind == "plain" else s[0]
    i, j, k = np.indices(n)
    odd = (i + j + k) % 2 == 1
    if kind == "ties":
        V = np.floor(4.0 * V / V.max()) * V.max()
        F[:] = 1.0
    if kind == "decisions":
        # values a distance from the cell's own first root that shrinks to its last bits
        F[:] = 1.0
        V = np.where((i // 2 + j // 2 + k // 2) % 2 == 0, V * 0.01, h * s[0] * (1.0 + rng.choice([-1.0, 0.0, 1.0], n) *
                                                                       np.exp2(-rng.uniform(0, 53, n))))
    V = np.where(odd, np.inf, V)
    P = np.pad(V, 1, constant_values=np.inf)
    m = [np.minimum(P[:-2, 1:-1, 1:-1], P[2:, 1:-1, 1:-1]), np.minimum(P[1:-1, :-2, 1:-1], P[1:-1, 2:, 1:-1]),
         np.minimum(P[1:-1, 1:-1, :-2], P[1:-1, 1:-1, 2:])]
    want = general(np.stack([x[odd] for x in m]), s, h / F[odd], scale is not None)
    idx = np.flatnonzero(~odd.reshape(-1)).astype(np.int64)
    T, st, _ = fmm.solve(torch.from_numpy(F).to(dev), h, torch.from_numpy(idx).to(dev),
                         torch.from_numpy(V.reshape(-1)[idx].copy()).to(dev), stride=np.inf, axis_scale=scale)
    got = T.cpu().numpy()[odd]
    bad = np.flatnonzero(got.view(np.uint64) != want.view(np.uint64))
    assert bad.size == 0, (bad.size, got[bad[:3]], want[bad[:3]])
