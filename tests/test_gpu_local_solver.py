"""The device local solver where it decides which root to form: triples around
the two decisions (a value one root short of joining), absent values, values far
above r (travel times of large grids), and r near the ends of its range.  Bar:
bit for bit the oracle's result, as for random triples."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fmm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1502_07303_amd import fmm as m
    m.load_library()
    return m


def triples(kind, n, rng):
    r = np.exp2(rng.uniform(-20, 10, n))
    a1 = np.where(rng.random(n) < 0.1, 0.0, r * np.exp2(rng.uniform(-4, 22, n)))
    off = np.exp2(-rng.uniform(0, 52, n)) * rng.choice([-1.0, 0.0, 1.0], n)  # distance from the decision
    d = rng.uniform(0, 1.0, n) * r
    inf = np.full(n, np.inf)
    if kind == "two_values":       # a2 = a1 + r: the second value just joins or just does not
        a2 = a1 + r * (1 + off)
        a3 = np.where(rng.random(n) < 0.5, inf, a2 + rng.uniform(0, 1, n) * r)
    elif kind == "three_values":   # a3 = the root of the first two
        a2 = a1 + d
        a3 = a1 + (d + np.sqrt(2 * r * r - d * d)) / 2 * (1 + 0.1 * off)
    elif kind == "ties":
        a2 = np.where(rng.random(n) < 0.5, a1, a1 + r)
        a3 = np.where(rng.random(n) < 0.5, a2, a1 + r)
    else:                          # ends of the range
        r = rng.choice([0.0, np.inf, 1e-300, 1e-160, 1e-115, 1e-114, 1e148, 1e149, 1e154, 1e300], n)
        s = np.where(np.isfinite(r) & (r > 0), r, 1.0)
        a1, a2, a3 = (s * rng.choice([0.0, 0.5, 1.0, 3.0], n) for _ in range(3))
        a3 = np.where(rng.random(n) < 0.2, inf, a3)
    a = np.stack([a1, a2, a3], 1)
    return np.ascontiguousarray(rng.permuted(a, axis=1)), np.ascontiguousarray(r)


@pytest.mark.parametrize("kind", ["two_values", "three_values", "ties", "range"])
def test_local_solver_decisions_bitwise(fmm, oracle_mod, kind):
    a, r = triples(kind, 1 << 18, np.random.default_rng(11))
    dev = torch.device("cuda:0")
    got = fmm.eval_godunov(torch.from_numpy(a).to(dev), torch.from_numpy(r).to(dev)).cpu().numpy()
    want = oracle_mod.godunov_batch(a, r)
    bad = np.flatnonzero(got.view(np.uint64) != np.asarray(want).view(np.uint64))
    assert bad.size == 0, (bad.size, a[bad[:3]], r[bad[:3]], got[bad[:3]], want[bad[:3]])
