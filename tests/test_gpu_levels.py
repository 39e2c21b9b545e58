"""Levels inside a tile march: with inner steps (each level from a scan for the
pending minimum) and without (the restart's bound at once, the minimum gathered
with the write-back), on one- and two-sided problems, FP32 and FP64, all tile
edges.  Bars: the oracle's status bytes and values within 1e-12 max|T|; the
restart count depends only on the pending minima, so it is the same for both."""
import math

import pytest
import torch

from helpers import parity_report
from paper_1502_07303_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fmm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1502_07303_amd import fmm as m
    m.load_library()
    return m


def workload(name):
    if name == "rough":
        return inputs.random_small((37, 29, 45), n_sources=2, seed=3, zero_frac=0.05)
    if name == "rough_f32":
        return inputs.random_small((33, 40, 18), n_sources=3, seed=4, dtype=torch.float32)
    return inputs.spheres(n=40, n_spheres=3, seed=1, width=0.15)


@pytest.mark.parametrize("name", ["rough", "rough_f32", "spheres"])
@pytest.mark.parametrize("edge", [4, 8, 16])
@pytest.mark.parametrize("stride_h", [1.0, 3.0, math.inf])
def test_inner_steps(fmm, oracle_mod, name, edge, stride_h):
    dev = torch.device("cuda:0")
    w = workload(name)
    F, idx, val = w.numpy()
    To, so, _, _ = oracle_mod.solve(F, w.h, idx, val, width=w.width)
    restarts = set()
    for inner in (None, 0.25 * w.h, w.h):
        T, st, s = fmm.solve(w.F.to(dev), w.h, w.seed_idx.to(dev), w.seed_val.to(dev), band_width=w.width,
                             stride=stride_h * w.h, tile_edge=edge, inner_stride=inner, time_limit_s=30)
        rep = parity_report(T.cpu().numpy(), st.cpu().numpy(), To, so)
        assert rep["same_status"] and rep["rel"] <= 1e-12, (inner, rep)
        restarts.add(int(s.n_restarts))
    if stride_h == 1.0:
        assert len(restarts) == 1, restarts
