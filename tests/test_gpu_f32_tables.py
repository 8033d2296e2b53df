"""Binary32 tables on the matrix cores: bit for bit the oracle's sums (one addition per position, ascending k), on ragged shapes,
taps that are no whole words, entries that cancel, round, overflow and are zero or negative zero; and the
tables that stay with the plain kernel."""
import numpy as np
import pytest
import torch

import oracle
from paper_2304_09049_amd import binding as dg
from paper_2304_09049_amd import workloads as wl

pytestmark = pytest.mark.gpu

TABLES = {"normal": ([-1.27, -0.32, 0.3217, 1.19], [0.05, 0.451, 0.98, 1.78]), "cancel": ([1e8, -1e8, 1.0, 0.37], [1.0, 0.5, 1e-9, 3.0]),
          "zeros": ([-0.0, 0.0, -1.1, 2.3], [0.0, -0.0, 0.7, -1.3]), "overflow": ([3e38, 1e38, -2.5e38, 1.0], [1.0, 0.9, 0.5, -1.0]),
          "small": ([1e-15, -3e-15, 2e-15, 7e-15], [1e-15, 2e-15, -5e-15, 3e-15])}         # (down to 1e-30; the kernel takes entries from 2^-100 = 7.9e-31)


@pytest.mark.parametrize("table", list(TABLES))
def test_f32_tables(table, monkeypatch):
    monkeypatch.setenv("DG_F32_MFMA", "1")
    lw, la = (np.array(x, np.float32) for x in TABLES[table])
    lut, entries = dg.dg_build_lut_f32(lw, la), oracle.build_lut_f32(lw, la)
    with np.errstate(over="ignore", invalid="ignore"):
        for (B, H, W, Cin, Cout, KH, KW, stride, pad) in [(2, 9, 8, 16, 10, 3, 3, (1, 2), (1, 1)), (1, 13, 11, 20, 33, 3, 3, (1, 1), (1, 1)),
                                                          (1, 7, 9, 44, 16, 5, 5, (1, 1), (2, 2)), (3, 6, 5, 128, 50, 1, 1, (1, 1), (0, 0)),
                                                          (1, 10, 10, 64, 17, 2, 3, (2, 1), (0, 1)), (1, 5, 5, 24, 3, 3, 1, (1, 1), (1, 0))]:
            c = wl.small_conv(B, H, W, Cin, Cout, KH, KW, stride, pad, seed=H + Cin, scale=True)
            desc = dg.conv_desc(B, H, W, Cin, Cout, KH, KW, stride, pad)
            assert dg.dg_conv_kernel_name(lut, desc) == "onehot_mfma_f32"
            Wp = dg.dg_pack_weights(torch.from_numpy(c.Wc).cuda(), Cout, KH * KW * Cin)
            Xp = dg.dg_pack_activations(torch.from_numpy(c.Ac).cuda(), B * H * W, Cin)
            want = oracle.conv2d_table_f32(c.Wc, c.Ac, entries, stride=stride, pad=pad)
            got = dg.dg_conv2d_lut(lut, Wp, Xp, desc).cpu().numpy()
            assert np.array_equal(got, want, equal_nan=True), (table, Cin)
            got = dg.dg_conv2d_lut(lut, Wp, Xp, desc, scale=torch.from_numpy(c.scale).cuda()).cpu().numpy()
            assert np.array_equal(got, want * c.scale[None, None, None, :], equal_nan=True), (table, Cin, "scaled")
        for M, N, K in ((33, 57, 320), (70, 130, 52), (5, 300, 1040)):
            g = wl.small_gemm(M, N, K, seed=M)
            Wp, Ap = dg.dg_pack_weights(torch.from_numpy(g.Wc).cuda(), M, K), dg.dg_pack_activations(torch.from_numpy(g.Ac).cuda(), N, K)
            want = oracle.gemm_table_f32(g.Wc, g.Ac, entries)
            for strides, shape in (((N, 1), (M, N)), ((1, M), (N, M))):
                out = torch.zeros(shape, dtype=torch.float32, device="cuda")
                got = dg.dg_gemm_lut(lut, Wp, Ap, M, N, K, out=out, strides=strides).cpu().numpy()
                assert np.array_equal(got, want.T if strides[0] == 1 else want, equal_nan=True), (table, M, N, K, strides)


def test_f32_tables_large_padding():
    """One image row of 65536 pixels under a filter of 16385 rows with 16384 rows of padding: a pixel's own offset and a tap's are
    2^32 bytes and more, of either sign; only one row of the filter meets the image for each output row."""
    W, Cin, Cout, reach = 1 << 16, 16, 16, 1 << 14
    lw, la = (np.array(x, np.float32) for x in TABLES["normal"])
    lut, entries = dg.dg_build_lut_f32(lw, la), oracle.build_lut_f32(lw, la).reshape(4, 4)
    desc = dg.conv_desc(1, 1, W, Cin, Cout, reach + 1, 1, (reach, 1), (reach, 0))
    assert dg.dg_conv_kernel_name(lut, desc) == "onehot_mfma_f32"
    rng = np.random.default_rng(3)
    Wc, Xc = wl.draw_codes(rng, (Cout, reach + 1, 1, Cin)), wl.draw_codes(rng, (1, 1, W, Cin))
    Wp = dg.dg_pack_weights(torch.from_numpy(Wc).cuda(), Cout, (reach + 1) * Cin)
    Xp = dg.dg_pack_activations(torch.from_numpy(Xc).cuda(), W, Cin)
    got = dg.dg_conv2d_lut(lut, Wp, Xp, desc).cpu().numpy()
    assert got.shape == (1, 2, W, Cout)
    for oh, kh in ((0, reach), (1, 0)):
        want = np.zeros((W, Cout), np.float32)
        for ci in range(Cin):
            want = want + entries[Wc[:, kh, 0, ci][None, :], Xc[0, 0, :, ci][:, None]]
        assert np.array_equal(got[0, oh], want), oh


def test_f32_tables_rule():
    big, small = dg.conv_desc(4, 28, 28, 128, 128, 3, 3, (1, 1), (1, 1)), dg.conv_desc(1, 5, 5, 16, 8, 3, 3, (1, 1), (1, 1))
    good = dg.dg_build_lut_f32([-1.0, 0.3, 2.0, 0.0], [0.1, 0.2, 0.0, 4.0])
    assert dg.dg_conv_kernel_name(good, big) == "onehot_mfma_f32" and dg.dg_conv_kernel_name(good, big, "lds") == "lds_f32"
    assert dg.dg_conv_kernel_name(good, small) == "lds_f32"
    for lw, la in (([1e30, 1.0, 2.0, 3.0], [1e30, 1.0, 2.0, 3.0]), ([float("nan"), 1.0, 2.0, 3.0], [0.0, 1.0, 2.0, 3.0]),
                   ([1e-20, 1.0, 2.0, 3.0], [1e-20, 1.0, 2.0, 3.0])):
        assert dg.dg_conv_kernel_name(dg.dg_build_lut_f32(lw, la), big) == "lds_f32"
