"""The staged kernel where its own bookkeeping ends: a bit per row and column of the filter window (15 of each), padding wider than
that, tensors smaller than one load, shares of K that are empty."""
import numpy as np
import pytest

import oracle
from gpu_helpers import GpuCase
from paper_2304_09049_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bias", ["0", "1"])
@pytest.mark.parametrize("plan", ["12", "12k4", "14k2", "14k4", "17", "24"])
def test_staged_windows_and_shares(plan, bias, monkeypatch):
    monkeypatch.setenv("DG_ONEHOT_PLAN", plan)
    monkeypatch.setenv("DG_STAGED_BIAS", bias)
    lw, la = [-9, -2, 3, 8], [-5, 0, 4, 9]
    for (B, H, W, Cin, Cout, KH, KW, pad) in [(1, 9, 6, 128, 40, 15, 1, (14, 0)), (1, 5, 9, 128, 36, 1, 15, (0, 7)), (1, 4, 4, 128, 33, 3, 3, (19, 20)),
                                              (1, 16, 3, 128, 32, 16, 1, (0, 0)), (2, 1, 1, 128, 4, 3, 3, (1, 1)), (1, 1, 1, 256, 1, 1, 1, (0, 0))]:
        c = wl.small_conv(B, H, W, Cin, Cout, KH, KW, (1, 1), pad, seed=KH + KW + Cout)
        case = GpuCase(c, levels=(lw, la))
        assert ("staged" in case.kernel_name("onehot_smfmac")) == (KH <= 15)
        want = oracle.conv2d(c.Wc, c.Ac, lw, la, stride=(1, 1), pad=pad)
        assert np.array_equal(case.run("onehot_smfmac").cpu().numpy(), want), (B, H, W, Cin, Cout, KH, KW, pad)
