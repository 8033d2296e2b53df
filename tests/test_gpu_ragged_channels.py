"""Layers whose channel count is no multiple of 32, on the sparse matrix instruction: every tile, window width and division of
a filter tap between the lane halves, packed and from unpacked codes, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2304_09049_amd import binding as dg
from paper_2304_09049_amd import workloads as wl

pytestmark = pytest.mark.gpu

LW, LA = (-2, -1, 0, 1), (3, 1, -2, 5)          # no zero activation level: padding must add nothing all the same
CONVS = [  # B, H, W, Cin, Cout, KH, KW, stride, pad: 4 to 131 packed bytes per tap, even, odd and single taps, no edge in step
    (2, 17, 15, 48, 70, 3, 3, (1, 1), (1, 1)), (1, 31, 33, 16, 64, 5, 5, (1, 1), (2, 2)), (2, 20, 21, 20, 36, 3, 3, (2, 1), (1, 1)),
    (3, 19, 23, 44, 100, 1, 1, (1, 1), (0, 0)), (1, 40, 40, 52, 96, 1, 1, (2, 2), (0, 0)), (1, 14, 14, 112, 130, 3, 3, (1, 1), (1, 1)),
    (1, 9, 9, 200, 64, 5, 5, (1, 1), (2, 2)), (1, 12, 13, 524, 33, 1, 1, (1, 1), (0, 0)), (1, 12, 13, 260, 34, 3, 2, (1, 1), (1, 0)),
    (2, 16, 16, 36, 44, 2, 3, (1, 2), (1, 1)), (1, 30, 30, 24, 50, 3, 1, (1, 1), (1, 0)), (1, 5, 5, 76, 3, 1, 1, (1, 1), (0, 0))]
GEMMS = [(70, 300, 80), (64, 600, 144), (300, 65, 560), (33, 1000, 52), (129, 513, 1040), (1, 1, 20)]


@pytest.mark.parametrize("plan", ["auto", "11", "21", "22", "11s1", "21s1", "22s1", "11s3", "22s2"])
def test_ragged_channels(plan, monkeypatch):
    monkeypatch.setenv("DG_RAGGED", "1")
    monkeypatch.setenv("DG_RAGGED_CODES", "1")
    if plan != "auto":
        monkeypatch.setenv("DG_RAGGED_PLAN", plan)
    lut = dg.dg_build_lut(LW, LA)
    for (B, H, W, Cin, Cout, KH, KW, stride, pad) in CONVS:
        c = wl.small_conv(B, H, W, Cin, Cout, KH, KW, stride, pad, seed=H + Cin, scale=True)
        desc = dg.conv_desc(B, H, W, Cin, Cout, KH, KW, stride, pad)
        assert dg.dg_conv_kernel_name(lut, desc).startswith("onehot_smfmac_ragged_")
        assert ("codes_" in dg.dg_conv_codes_kernel_name(lut, desc)) == (KH * KW > 1 or stride == (1, 1) or Cin % 16 != 0)
        X, scale = torch.from_numpy(c.Ac).cuda(), torch.from_numpy(c.scale).cuda()
        Wp = dg.dg_pack_weights(torch.from_numpy(c.Wc).cuda(), Cout, KH * KW * Cin)
        Xp = dg.dg_pack_activations(X, B * H * W, Cin)
        want = oracle.conv2d(c.Wc, c.Ac, LW, LA, stride=stride, pad=pad)
        wants = oracle.scale_epilogue_nhwc(want, c.scale)
        for s, w in ((None, want), (scale, wants)):
            got = dg.dg_conv2d_lut(lut, Wp, Xp, desc, scale=s).cpu().numpy()
            assert np.array_equal(got, w), (desc.Cin, "packed", s is not None)
            got = dg.dg_conv2d_lut_codes(lut, Wp, X, desc, work=torch.empty_like(Xp), scale=s).cpu().numpy()
            assert np.array_equal(got, w), (desc.Cin, "codes", s is not None)
    for (M, N, K) in GEMMS:
        g = wl.small_gemm(M, N, K, seed=M)
        A = torch.from_numpy(g.Ac).cuda()
        Wp, Ap = dg.dg_pack_weights(torch.from_numpy(g.Wc).cuda(), M, K), dg.dg_pack_activations(A, N, K)
        scale = torch.from_numpy(np.random.default_rng(K).uniform(0.01, 0.1, M).astype(np.float32)).cuda()
        want = oracle.gemm(g.Wc, g.Ac, LW, LA)
        wants = want.astype(np.float32) * scale.cpu().numpy()[:, None]
        # column-major, row-major (run transposed where packed, the scale then goes with the rows), neither axis contiguous
        for strides, shape in (((1, M), (N, M)), ((N, 1), (M, N)), ((3, 3 * M + 1), (N, 3 * M + 1))):
            for s, w in ((None, want), (scale, wants)):
                for codes in (False, True):
                    out = torch.zeros(shape, dtype=torch.int32 if s is None else torch.float32, device="cuda")
                    kw = dict(out=out, strides=strides, scale=s)
                    if codes:
                        dg.dg_gemm_lut_codes(lut, Wp, A, M, N, K, work=torch.empty_like(Ap), **kw)
                    else:
                        dg.dg_gemm_lut(lut, Wp, Ap, M, N, K, **kw)
                    got = out.cpu().numpy()
                    got = got if shape == (M, N) and strides[1] == 1 else got[:, :M * strides[0]:strides[0]].T
                    assert np.array_equal(got, w), ((M, N, K), strides, s is not None, codes)


def test_ragged_channels_rule(monkeypatch):
    """Which layers take it by themselves; unaligned operands; entries beyond int8 stay where they were."""
    lut, wide = dg.dg_build_lut(LW, LA), dg.dg_build_lut((100, -100, 3, 1), (90, 1, -90, 0), dg.DG_LUT_I16)
    big, tiny = dg.conv_desc(8, 29, 27, 48, 120, 5, 5, (1, 1), (2, 2)), dg.conv_desc(1, 5, 5, 48, 16, 3, 3, (1, 1), (1, 1))
    narrow, whole = dg.conv_desc(8, 29, 27, 12, 120, 5, 5, (1, 1), (2, 2)), dg.conv_desc(8, 29, 27, 96, 120, 5, 5, (1, 1), (2, 2))
    assert dg.dg_conv_kernel_name(lut, big) == "onehot_smfmac_ragged_32x32"
    assert dg.dg_conv_codes_kernel_name(lut, big) == "codes_onehot_smfmac_ragged_64x32"
    for table, desc in ((lut, tiny), (lut, narrow), (lut, whole), (wide, big)):
        assert "ragged" not in dg.dg_conv_kernel_name(table, desc)
    c = wl.small_conv(2, 30, 29, 44, 40, 3, 3, (1, 1), (1, 1), seed=3)
    want = oracle.conv2d(c.Wc, c.Ac, LW, LA, stride=(1, 1), pad=(1, 1))
    X, desc = torch.from_numpy(c.Ac).cuda(), dg.conv_desc(2, 30, 29, 44, 40, 3, 3, (1, 1), (1, 1))
    Wp, Xp = dg.dg_pack_weights(torch.from_numpy(c.Wc).cuda(), 40, 9 * 44), dg.dg_pack_activations(X, 2 * 30 * 29, 44)
    for shift in (1, 2, 3):                      # operands at any byte
        Wu = torch.empty(Wp.numel() + shift, dtype=torch.uint8, device="cuda")[shift:].copy_(Wp.flatten())
        Xu = torch.empty(Xp.numel() + shift, dtype=torch.uint8, device="cuda")[shift:].copy_(Xp.flatten())
        got = dg.dg_conv2d_lut(lut, Wu, Xu, desc).cpu().numpy()
        assert np.array_equal(got, want), shift
