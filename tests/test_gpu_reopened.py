"""n_reopened counts values lowered after they had been accepted: with an
unbounded level (stride = +inf and no band) a cell's first value is no reopening.
Exact: a line from one end lowers no value at all, and a problem of one tile is
solved by one wavefront in a fixed order, the same for +inf and for a finite level
above every value."""
import math

import pytest
import torch

from paper_1502_07303_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fmm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1502_07303_amd import fmm as m
    m.load_library()
    return m


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("edge,n", [(4, 4), (4, 19), (8, 8), (8, 37), (16, 16), (16, 50)])
def test_first_values_are_no_reopenings(fmm, edge, n, dtype):
    dev = torch.device("cuda:0")
    F = torch.ones((1, 1, n), dtype=dtype, device=dev)
    T, st, s = fmm.solve(F, 1.0, torch.zeros(1, dtype=torch.int64, device=dev),
                         torch.zeros(1, dtype=torch.float64, device=dev), stride=math.inf, tile_edge=edge)
    assert torch.equal(T.view(-1).cpu(), torch.arange(n, dtype=torch.float64))
    assert s.n_accepted == n - 1 and s.n_solves >= n - 1
    assert s.n_reopened == 0


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("edge", [4, 8])
def test_infinite_level_counts_as_a_finite_one(fmm, edge, dtype):
    dev = torch.device("cuda:0")
    w = inputs.random_small((edge, edge, edge), n_sources=1, seed=7, dtype=dtype)
    got = []
    for stride in (1e300, math.inf):
        T, st, s = fmm.solve(w.F.to(dev), w.h, w.seed_idx.to(dev), w.seed_val.to(dev), stride=stride, tile_edge=edge)
        got.append((T.cpu(), s.n_solves, s.n_reopened))
    assert torch.equal(got[0][0], got[1][0])
    assert got[0][1:] == got[1][1:]
    assert got[0][2] <= got[0][1] - (edge ** 3 - 1)
