"""Entries beyond int8 on the staged sparse-instruction kernel: every tile and sharing of K, whole and half runs, both output
layouts, int32, scaled and re-quantised output, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2304_09049_amd import binding as dg
from paper_2304_09049_amd import workloads as wl

pytestmark = pytest.mark.gpu

LW, LA = (127, -128, 5, 3), (-128, 127, 1, 2)          # the widest entries; no zero activation level


@pytest.mark.parametrize("plan", ["2", "2k4", "4", "4k2", "4k4"])
def test_two_plane_staged(plan, monkeypatch):
    monkeypatch.setenv("DG_STAGED_2P_PLAN", plan)
    lut = dg.dg_build_lut(LW, LA, dg.DG_LUT_I16)
    name = {"2": "onehot_smfmac_2p_staged_32x64", "4": "onehot_smfmac_2p_staged_32x128"}[plan[0]]
    name += "_" + plan[1:] if plan[1:] else ""
    for (B, H, W, Cin, Cout, k, stride, pad) in [(2, 13, 11, 128, 40, 3, (1, 1), (1, 1)), (1, 30, 30, 256, 68, 3, (2, 2), (1, 1)),
                                                 (3, 9, 10, 384, 33, 1, (1, 1), (0, 0)), (1, 8, 9, 128, 100, 5, (1, 2), (2, 2)),
                                                 (1, 15, 17, 192, 36, 3, (1, 1), (1, 1)), (1, 6, 7, 64, 32, 1, (1, 1), (0, 0))]:
        c = wl.small_conv(B, H, W, Cin, Cout, k, k, stride, pad, seed=H + Cin, scale=True)
        desc = dg.conv_desc(B, H, W, Cin, Cout, k, k, stride, pad)
        # (taps of half runs have one tile)
        assert dg.dg_conv_kernel_name(lut, desc) == (name if Cin % 128 == 0 else "onehot_smfmac_2p_staged_32x64")
        Wp = dg.dg_pack_weights(torch.from_numpy(c.Wc).cuda(), Cout, k * k * Cin)
        Xp = dg.dg_pack_activations(torch.from_numpy(c.Ac).cuda(), B * H * W, Cin)
        scale = torch.from_numpy(c.scale).cuda()
        want = oracle.conv2d(c.Wc, c.Ac, LW, LA, stride=stride, pad=pad)
        y = oracle.scale_epilogue_nhwc(want, c.scale)
        assert np.array_equal(dg.dg_conv2d_lut(lut, Wp, Xp, desc).cpu().numpy(), want), (Cin, k)
        assert np.array_equal(dg.dg_conv2d_lut(lut, Wp, Xp, desc, scale=scale).cpu().numpy(), y), (Cin, k, "scaled")
        if Cout % 4 == 0:
            qs = float(np.float32(3.0 / max(1e-6, float(np.percentile(np.abs(y), 90)))))
            packed = dg.dg_conv2d_lut_requant(lut, Wp, Xp, desc, scale, qs, 0.5, 0).cpu().numpy()
            codes = oracle.quantize_codes(y, qs, 0.5, 0, 3)
            assert np.array_equal(packed.reshape(-1, Cout // 4), oracle.pack_codes(codes.reshape(-1, Cout))), (Cin, k, "requant")
    for M, N, K in ((33, 130, 128), (70, 300, 1024), (5, 1000, 384)):
        g = wl.small_gemm(M, N, K, seed=M)
        Wp, Ap = dg.dg_pack_weights(torch.from_numpy(g.Wc).cuda(), M, K), dg.dg_pack_activations(torch.from_numpy(g.Ac).cuda(), N, K)
        want = oracle.gemm(g.Wc, g.Ac, LW, LA)
        for strides, shape in (((1, M), (N, M)), ((N, 1), (M, N))):
            out = torch.full(shape, -7, dtype=torch.int32, device="cuda")
            got = dg.dg_gemm_lut(lut, Wp, Ap, M, N, K, out=out, strides=strides).cpu().numpy()
            assert np.array_equal(got, want.T if strides[0] == 1 else want), (M, N, K, strides)
