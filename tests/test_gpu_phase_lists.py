"""Work lists of a phase around the sizes at which its distribution changes:
one item, fewer items than segments, exactly as many items as the launch has
wavefront groups (nothing is claimed), one fewer and one more, and several
items per group.  Every tile of the first list holds one seed away from its
faces, so the list's length is the number of seeds."""
import numpy as np
import pytest
import torch

from helpers import parity_report

pytestmark = pytest.mark.gpu

SHAPE = (16, 480, 576)  # 2 x 60 x 72 = 8640 tiles of 8^3


@pytest.fixture(scope="module")
def fmm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1502_07303_amd import fmm as m
    m.load_library()
    return m


@pytest.fixture(scope="module")
def speeds():
    return np.random.default_rng(5).uniform(0.5, 2.0, size=SHAPE)


# groups of a launch on 256 CUs: 2560 (8^3, FP64 speeds), 3072 (FP32)
@pytest.mark.parametrize("dtype,groups", [(torch.float64, 2560), (torch.float32, 3072)])
@pytest.mark.parametrize("length", ["1", "7", "groups-1", "groups", "groups+1", "all"])
def test_phase_list_lengths(fmm, oracle_mod, speeds, dtype, groups, length):
    dev = torch.device("cuda:0")
    n = {"1": 1, "7": 7, "groups-1": groups - 1, "groups": groups, "groups+1": groups + 1, "all": 8640}[length]
    F = torch.from_numpy(speeds).to(dtype)
    t = np.arange(n)
    c = np.stack([t // (60 * 72), (t // 72) % 60, t % 72], 1) * 8 + 3
    idx = ((c[:, 0] * SHAPE[1] + c[:, 1]) * SHAPE[2] + c[:, 2]).astype(np.int64)
    val = np.random.default_rng(n).uniform(0.0, 0.01, size=n)
    h = 1.0 / 575
    width = 6 * h
    To, so, _, _ = oracle_mod.solve(F.numpy(), h, idx, val, width=width)
    for stride in (1.5 * h, float("inf")):
        T, st, _ = fmm.solve(F.to(dev), h, torch.from_numpy(idx).to(dev), torch.from_numpy(val).to(dev),
                             band_width=width, stride=stride, time_limit_s=30)
        rep = parity_report(T.cpu().numpy(), st.cpu().numpy(), To, so)
        assert rep["same_status"] and rep["rel"] <= 1e-12, (n, stride, rep)
