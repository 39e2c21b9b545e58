"""The tile sweep against the level sweep (a workspace a byte short of the tiles'
takes it) field for field on one T, at sizes where a phase has more tiles than the
launch has wavefronts: items are claimed, segments drained and helped with.

Bar: the same few roundings per point in another order, 1e-12 of the largest
gradient, as for the adjoint on given T; dependency levels and points equal."""
import numpy as np
import pytest
import torch

from paper_1502_07303_amd import inputs

pytestmark = pytest.mark.gpu


def both(fmm, probs):
    out = []
    for short in (0, 1):
        for q in probs:
            q["dL_dF"].fill_(float("nan"))
        a = fmm.AdjointSolver(probs)
        a.nbytes -= short
        a.run()
        s = a.stats()
        out.append((s.n_levels, s.n_points, [q["dL_dF"].clone() for q in probs]))
    return out


@pytest.mark.parametrize("shape,shots,dtype,scale,shared", [
    ((256, 256, 256), 16, torch.float64, None, True), ((120, 128, 137), 2, torch.float32, None, True),
    ((97, 130, 161), 1, torch.float64, (1.0, 1.7, 0.6), True), ((8, 200, 410), 3, torch.float64, None, False)])
def test_sweeps_agree(shape, shots, dtype, scale, shared):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1502_07303_amd import fmm
    dev = torch.device("cuda:0")
    h = 1.0 / (max(shape) - 1)
    g = inputs.gaussian_field(max(shape), 5, 0.1, device=dev, shape=shape)
    F = torch.clamp(1.0 + 0.3 * g, min=0.1).to(dtype).contiguous()
    rng = np.random.default_rng(8)
    seeds = [(torch.from_numpy(rng.choice(F.numel(), size=1).astype(np.int64)).to(dev),
              torch.zeros(1, dtype=torch.float64, device=dev)) for _ in range(shots)]
    b = fmm.BatchSolver([{"F": F, "h": h, "seed_idx": i, "seed_val": v} for i, v in seeds], stride_h=4.0,
                        axis_scale=scale)
    b.solve()
    b.stats()
    one = torch.empty(shape, dtype=torch.float64, device=dev)
    probs = []
    for k in range(shots):
        gen = torch.Generator(device=dev)
        gen.manual_seed(k)
        probs.append({"F": F, "h": h, "T": b.T[k], "status": b.status[k],
                      "dL_dT": torch.randn(shape, generator=gen, dtype=torch.float64, device=dev),
                      "dL_dF": one if shared else torch.empty_like(one), "axis_scale": scale})
    tile, level = both(fmm, probs)
    assert tile[:2] == level[:2]
    for x, y in zip(tile[2], level[2]):
        assert float((x - y).abs().max()) <= 1e-12 * float(y.abs().max())
