"""Which sweep a batch is sized for: the tile sweep's where every grid has 8 points
along each axis, or the 8^3 tiles hold at most three cells per point of the batch.
Either way dL/dF and the dependency levels are those of the oracle's upwind system
solved by back substitution; bar 1e-12 of the largest gradient, the suite's for the
adjoint on given T."""
import numpy as np
import pytest
import torch

from test_gpu_adjoint_tiles import reference, solved

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shapes,tiled", [
    ([(7, 24, 17)], True), ([(3, 16, 16)], True), ([(2, 16, 16)], False), ([(7, 10, 10)], True), ([(7, 9, 9)], False),
    ([(3, 11, 11)], False), ([(9, 9, 9)], True), ([(1, 16, 16)], False), ([(1, 1, 40)], False), ([(6, 6, 6)], True),
    ([(4, 4, 4)], False), ([(16, 17, 16), (1, 9, 20)], True), ([(1, 9, 20), (9, 8, 12), (1, 1, 9)], False),
    ([(8, 8, 8), (1, 8, 8), (8, 8, 8)], True), ([(1, 9, 9), (8, 8, 8)], False), ([(1, 9, 9)] * 5 + [(5, 5, 5)], False)])
@pytest.mark.parametrize("dtype,scale", [(torch.float64, None), (torch.float32, (1.0, 1.7, 0.6))])
def test_route(oracle_mod, shapes, tiled, dtype, scale):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1502_07303_amd import fmm
    dev = torch.device("cuda:0")
    probs, want, levels = [], [], 0
    for k, shape in enumerate(shapes):
        F, h, T, st = solved(oracle_mod, shape, k + 1, dtype, scale, zero=0.05)
        g = np.random.default_rng(k).normal(size=shape)
        r, lev = reference(F, h, T, st, g, scale)
        want.append(r)
        levels = max(levels, lev)
        probs.append({"F": torch.from_numpy(F).to(dev), "h": h, "T": torch.from_numpy(T).to(dev),
                      "status": torch.from_numpy(st).to(dev), "dL_dT": torch.from_numpy(g).to(dev),
                      "dL_dF": torch.empty(shape, dtype=torch.float64, device=dev), "axis_scale": scale})
    a = fmm.AdjointSolver(probs)
    cells = sum(512 * int(np.prod([-(-n // 8) for n in s])) for s in shapes)
    thin = min(min(s) for s in shapes) < 8
    assert tiled == (not thin or cells <= 3 * sum(int(np.prod(s)) for s in shapes))
    assert (a.nbytes >= 36 * cells) == tiled
    for _ in range(2):
        a.run()
        assert a.stats().n_levels == levels
        for q, r in zip(probs, want):
            assert np.max(np.abs(q["dL_dF"].cpu().numpy() - r)) <= 1e-12 * np.max(np.abs(r))
