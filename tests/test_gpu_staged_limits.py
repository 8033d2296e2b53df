"""The staged kernel where its own bookkeeping ends: a byte per bound of the filter window (127 rows and columns), padding wider than
that, tensors smaller than one load, shares of K that are empty; with int8 entries, 4-bit slots, two planes and half runs."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import GpuCase
from paper_2304_09049_amd import binding as dg
from paper_2304_09049_amd import workloads as wl

pytestmark = pytest.mark.gpu

SHAPES = [(1, 9, 6, 128, 40, 15, 1, (14, 0)), (1, 5, 9, 128, 36, 1, 15, (0, 7)), (1, 4, 4, 128, 33, 3, 3, (19, 20)),
          (1, 16, 3, 128, 32, 16, 1, (0, 0)), (2, 1, 1, 128, 4, 3, 3, (1, 1)), (1, 1, 1, 256, 1, 1, 1, (0, 0)),
          (1, 3, 40, 128, 20, 1, 16, (0, 15)), (1, 6, 7, 128, 9, 17, 18, (8, 9)), (1, 2, 70, 128, 5, 1, 127, (0, 126)),
          (2, 70, 1, 128, 5, 127, 1, (63, 0)), (1, 66, 1, 128, 4, 128, 1, (64, 0)), (1, 1, 66, 128, 4, 1, 128, (0, 64)),
          (1, 5, 5, 128, 8, 3, 3, (130, 1)), (1, 5, 5, 128, 8, 3, 3, (1, 140)),
          (2, 9, 8, 256, 36, 3, 3, (1, 1)), (1, 7, 19, 2176, 33, 1, 1, (0, 0))]      # K = 2304 and 2176: either table of the 32 x 128 tile


@pytest.mark.parametrize("bias", ["0", "1"])
@pytest.mark.parametrize("plan", ["12", "12k4", "14", "14k2", "14k4", "16", "17", "24"])
def test_staged_windows_and_shares(plan, bias, monkeypatch):
    monkeypatch.setenv("DG_ONEHOT_PLAN", plan)
    monkeypatch.setenv("DG_STAGED_BIAS", bias)
    lw, la = [-9, -2, 3, 8], [-5, 0, 4, 9]
    for (B, H, W, Cin, Cout, KH, KW, pad) in SHAPES:
        c = wl.small_conv(B, H, W, Cin, Cout, KH, KW, (1, 1), pad, seed=KH + KW + Cout)
        case = GpuCase(c, levels=(lw, la))
        assert ("staged" in case.kernel_name("onehot_smfmac")) == (max(KH, KW) <= 127)
        want = oracle.conv2d(c.Wc, c.Ac, lw, la, stride=(1, 1), pad=pad)
        assert np.array_equal(case.run("onehot_smfmac").cpu().numpy(), want), (B, H, W, Cin, Cout, KH, KW, pad)


@pytest.mark.parametrize("plan", ["12", "14"])
def test_staged_windows_of_half_runs(plan, monkeypatch):
    monkeypatch.setenv("DG_ONEHOT_PLAN", plan)
    lw, la = [-9, -2, 3, 8], [-5, 0, 4, 9]
    for (B, H, W, Cin, Cout, KH, KW, pad) in SHAPES:
        Cin = 64 if KH * KW > 20 else 192
        c = wl.small_conv(B, H, W, Cin, Cout, KH, KW, (1, 1), pad, seed=KH + KW + Cout)
        case = GpuCase(c, levels=(lw, la))
        assert ("staged" in case.kernel_name("onehot_smfmac")) == (max(KH, KW) <= 127)
        want = oracle.conv2d(c.Wc, c.Ac, lw, la, stride=(1, 1), pad=pad)
        assert np.array_equal(case.run("onehot_smfmac").cpu().numpy(), want), (B, H, W, Cin, Cout, KH, KW, pad)


@pytest.mark.parametrize("plan", ["2", "2k4", "4", "4k2", "4k4"])
def test_two_plane_windows_and_shares(plan, monkeypatch):
    monkeypatch.setenv("DG_STAGED_2P_PLAN", plan)
    lw, la = (127, -128, 5, 3), (-128, 127, 1, 2)
    for (B, H, W, Cin, Cout, KH, KW, pad) in SHAPES + [(1, 5, 9, 192, 36, 1, 17, (0, 7))]:
        c = wl.small_conv(B, H, W, Cin, Cout, KH, KW, (1, 1), pad, seed=KH + KW + Cout)
        case = GpuCase(c, levels=(lw, la), entry=dg.DG_LUT_I16)
        assert ("2p_staged" in case.kernel_name()) == (max(KH, KW) <= 127)
        want = oracle.conv2d(c.Wc, c.Ac, lw, la, stride=(1, 1), pad=pad)
        assert np.array_equal(case.run().cpu().numpy(), want), (B, H, W, Cin, Cout, KH, KW, pad)


@pytest.mark.parametrize("plan", ["12", "12k4", "14", "14k2", "14k4", "17", "24"])
def test_nibble_windows_and_shares(plan, monkeypatch):
    monkeypatch.setenv("DG_NIBBLES", "1")
    monkeypatch.setenv("DG_ONEHOT_PLAN", plan)
    lw, la = list(range(-8, 8)), list(range(16))
    lut = dg.dg_build_lut_bits(4, lw, la, dg.DG_LUT_I8)
    rng = np.random.default_rng(7)
    for (B, H, W, Cin, Cout, KH, KW, pad) in SHAPES:
        Cin //= 2                                            # (two 2-bit positions each)
        Wc = rng.integers(0, 16, (Cout, KH, KW, Cin), dtype=np.uint8)
        Xc = rng.integers(0, 16, (B, H, W, Cin), dtype=np.uint8)
        desc = dg.conv_desc(B, H, W, Cin, Cout, KH, KW, (1, 1), pad)
        assert ("4as2_staged" in dg.dg_conv_kernel_name(lut, desc)) == (max(KH, KW) <= 127)
        Wp = dg.dg_pack_codes_bits(torch.from_numpy(Wc).cuda(), Cout, KH * KW * Cin, 4)
        Xp = dg.dg_pack_codes_bits(torch.from_numpy(Xc).cuda(), B * H * W, Cin, 4)
        want = oracle.conv2d(Wc, Xc, lw, la, stride=(1, 1), pad=pad)
        got = dg.dg_conv2d_lut(lut, Wp, Xp, desc).cpu().numpy()
        assert np.array_equal(got, want), (B, H, W, Cin, Cout, KH, KW, pad)
