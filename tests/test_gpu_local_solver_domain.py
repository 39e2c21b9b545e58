"""fmm_eval_godunov outside the march's domain: negative r (the one-value root
a1 + r, as no larger root lies below it), negative and infinite upwind values.
Bar: bit for bit the oracle's result."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["negative_r", "negative_a", "infinite_a"])
def test_local_solver_domain(oracle_mod, kind):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1502_07303_amd import fmm
    fmm.load_library()
    rng = np.random.default_rng(5)
    n = 1 << 16
    r = np.exp2(rng.uniform(-300, 300, n))
    a = rng.uniform(-1.0 if kind == "negative_a" else 0.0, 1.0, (n, 3)) * r[:, None] * np.exp2(rng.uniform(-3, 3, (n, 1)))
    if kind == "negative_r":
        r = -r
        r[:16] = -0.0
        r[16:32] = -np.inf
    if kind == "infinite_a":
        a[rng.random((n, 3)) < 0.3] = np.inf
        a[rng.random((n, 3)) < 0.1] = -np.inf
    got = fmm.eval_godunov(torch.from_numpy(a).cuda(), torch.from_numpy(r).cuda()).cpu().numpy()
    want = oracle_mod.godunov_batch(a, r)
    nan = np.isnan(want)
    assert np.array_equal(np.isnan(got), nan)
    bad = np.flatnonzero((got.view(np.uint64) != want.view(np.uint64)) & ~nan)
    assert bad.size == 0, (bad.size, a[bad[:3]], r[bad[:3]], got[bad[:3]], want[bad[:3]])
