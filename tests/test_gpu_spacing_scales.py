"""The weighted local solver where its short root and quotient hand over to the
library's: spacings far apart or extreme, flat fields (ties, zero
discriminants) and impassable points.  Bar: identical status bytes and 1e-12 of
max|T|, as for the other spacings."""
import numpy as np
import pytest
import torch

import helpers
from paper_1502_07303_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fmm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1502_07303_amd import fmm as m
    m.load_library()
    return m


@pytest.mark.parametrize("flat", [False, True])
@pytest.mark.parametrize("scale", [(1.0, 1.0, 1e3), (1e-3, 1.0, 1e3), (2.0, 2.0, 2.0), (1e-60, 1e-60, 3e-60),
                                   (1e60, 2e60, 1e60)])
def test_spacing_scales(fmm, oracle_mod, scale, flat):
    dev = torch.device("cuda:0")
    w = inputs.random_small((19, 22, 17), n_sources=2, seed=8, dtype=torch.float64, zero_frac=0.05)
    F, idx, val = w.numpy()
    if flat:
        F = np.where(F > 0.0, 1.0, F)
    T, st, s = fmm.solve(torch.from_numpy(F).to(dev), w.h, torch.from_numpy(idx).to(dev), torch.from_numpy(val).to(dev),
                         stride=3.0 * w.h * max(scale), axis_scale=scale)
    To, so, _, _ = oracle_mod.solve(F, w.h, idx, val, axis_scale=scale)
    rep = helpers.parity_report(T.cpu().numpy(), st.cpu().numpy(), To, so)
    assert rep["same_status"] and rep["rel"] <= 1e-12, rep
