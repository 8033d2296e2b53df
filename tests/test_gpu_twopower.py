"""Products of levels on the FP6 / FP4 matrix instruction: every tile, K of whole and of broken runs, every way to the output, against the
oracle; and sums at the end of the range that is taken."""
import numpy as np
import pytest
import torch

import oracle
from paper_2304_09049_amd import binding as dg
from paper_2304_09049_amd import workloads as wl

pytestmark = pytest.mark.gpu

NAMES = {"1": "twopower_64x128", "12": "twopower_64x128_k2", "2": "twopower_128x256", "4": "twopower_128x512"}
# levels of both signs, code 0 with a number of its own on either side; every FP6 step; sums of two powers up to 16; factors; one level
TABLES = [((-7, 5, -2, 3), (7, -8, 0, 5)), ((-15, 13, 1, 11), (-2, -1, 0, 1)), ((60, -44, 30, -22), (10, 9, -10, 3)), ((0, 3, 0, -9), (16, -12, 9, 1)),
          ((0, 0, 0, 5), (1, 2, 4, 7)), ((8, 8, 8, 8), (-3, -3, -3, -3)), ((36, -52, 7, 1), (-1, 6, 5, -9))]
GEMMS = [(70, 300, 64), (129, 513, 320), (127, 65, 256), (300, 257, 448), (64, 1025, 512), (257, 130, 1088), (1, 3, 128), (128, 512, 768), (40, 90, 2240)]


@pytest.mark.parametrize("plan", ["1", "12", "2", "4"])
def test_twopower_kernel(plan, monkeypatch):
    monkeypatch.setenv("DG_TWOPOWER", plan)
    for i, (M, N, K) in enumerate(GEMMS):
        lw, la = TABLES[i % len(TABLES)]
        lut = dg.dg_build_lut(lw, la, dg.DG_LUT_I16)
        g = wl.small_gemm(M, N, K, seed=M)
        assert dg.dg_gemm_kernel_name(lut, M, N, K) == NAMES[plan], i
        Wp, Ap = dg.dg_pack_weights(torch.from_numpy(g.Wc).cuda(), M, K), dg.dg_pack_activations(torch.from_numpy(g.Ac).cuda(), N, K)
        scale = torch.from_numpy(np.random.default_rng(K).uniform(0.01, 0.1, M).astype(np.float32)).cuda()
        want = oracle.gemm(g.Wc, g.Ac, lw, la)
        wants = want.astype(np.float32) * scale.cpu().numpy()[:, None]
        # column-major, row-major, rows of whole 64-byte pieces, neither axis contiguous
        wide = (N + 15) // 16 * 16
        for strides, shape, view in (((1, M), (N, M), lambda o: o.T), ((N, 1), (M, N), lambda o: o), ((wide, 1), (M, wide), lambda o: o[:, :N]),
                                     ((3, 3 * M + 1), (N, 3 * M + 1), lambda o: o[:, : 3 * M : 3].T)):
            for s, w in ((None, want), (scale, wants)):
                out = torch.full(shape, -7, dtype=torch.int32 if s is None else torch.float32, device="cuda")
                dg.dg_gemm_lut(lut, Wp, Ap, M, N, K, out=out, strides=strides, scale=s)
                got = out.cpu().numpy()
                assert np.array_equal(view(got), w), ((M, N, K), strides, s is not None)
                assert (got == -7).sum() - (w == -7).sum() == got.size - w.size, ((M, N, K), strides, "stored outside")


@pytest.mark.parametrize("plan", ["1", "12", "2", "4"])
def test_twopower_kernel_on_layers(plan, monkeypatch):
    """1x1 layers without stride and padding, packed and from codes that are packed first."""
    monkeypatch.setenv("DG_TWOPOWER", plan)
    lw, la = TABLES[0]
    lut = dg.dg_build_lut(lw, la)
    for B, H, W, Cin, Cout in ((2, 9, 13, 320, 132), (3, 14, 14, 704, 64)):
        c = wl.small_conv(B, H, W, Cin, Cout, 1, 1, (1, 1), (0, 0), seed=Cin, scale=True)
        desc = dg.conv_desc(B, H, W, Cin, Cout, 1, 1, (1, 1), (0, 0))
        assert dg.dg_conv_kernel_name(lut, desc) == NAMES[plan]
        codes, scale = torch.from_numpy(c.Ac).cuda(), torch.from_numpy(c.scale).cuda()
        Wp = dg.dg_pack_weights(torch.from_numpy(c.Wc).cuda(), Cout, Cin)
        Xp = dg.dg_pack_activations(codes, B * H * W, Cin)
        want = oracle.conv2d(c.Wc, c.Ac, lw, la, stride=(1, 1), pad=(0, 0))
        assert np.array_equal(dg.dg_conv2d_lut(lut, Wp, Xp, desc).cpu().numpy(), want)
        got = dg.dg_conv2d_lut_codes(lut, Wp, codes, desc, work=torch.empty_like(Xp), scale=scale).cpu().numpy()
        assert np.array_equal(got, oracle.scale_epilogue_nhwc(want, c.scale))


@pytest.mark.parametrize("plan", ["1", "12", "4"])
def test_sums_to_the_end_of_the_range(plan, monkeypatch):
    """Sums of every magnitude up to the largest that is taken, 7 * 9 * K just below 2^24 (7 is 8 - 1), in steps of the smallest entry: exact."""
    M, N, K = 64, 40, 266240
    lw, la = (-7, 1, 3, 7), (-1, 1, 2, 7)
    rng = np.random.default_rng(5)
    Wc, Ac = rng.integers(0, 4, (M, K), dtype=np.uint8), rng.integers(0, 4, (N, K), dtype=np.uint8)
    for m in range(0, M, 2):                                # rows that climb to ever larger sums, on columns of the largest code
        Wc[m, : K * (m + 2) // M] = 3
    Ac[: N // 2] = 3
    Wc[1], Ac[1, ::7] = 0, 0
    monkeypatch.setenv("DG_TWOPOWER", plan)
    lut = dg.dg_build_lut(lw, la)
    assert dg.dg_gemm_kernel_name(lut, M, N, K) == NAMES[plan]
    Wp, Ap = dg.dg_pack_weights(torch.from_numpy(Wc).cuda(), M, K), dg.dg_pack_activations(torch.from_numpy(Ac).cuda(), N, K)
    want = np.rint(np.asarray(lw, np.float64)[Wc] @ np.asarray(la, np.float64)[Ac].T).astype(np.int64)      # (below 2^53: exact)
    assert np.abs(want).max() == 49 * K                     # (63 K with the powers taken apart)
    assert np.array_equal(dg.dg_gemm_lut(lut, Wp, Ap, M, N, K).cpu().numpy(), want)


AUTOS = [(1305, 1621, 1856, "twopower_64x128"), (2275, 903, 4544, "twopower_64x128_k2"), (3992, 1839, 2944, "twopower_128x256"),
         (3698, 3332, 3648, "twopower_128x512")]


@pytest.mark.parametrize("M,N,K,kernel", AUTOS)
def test_autos_own_plans(M, N, K, kernel):
    """Products of a size at which AUTO chooses each tile by itself: every sum, row- and column-major."""
    lw, la = TABLES[0]
    rng = np.random.default_rng(N)
    Wc, Ac = rng.integers(0, 4, (M, K), dtype=np.uint8), rng.integers(0, 4, (N, K), dtype=np.uint8)
    lut = dg.dg_build_lut(lw, la)
    assert dg.dg_gemm_kernel_name(lut, M, N, K) == kernel
    Wp, Ap = dg.dg_pack_weights(torch.from_numpy(Wc).cuda(), M, K), dg.dg_pack_activations(torch.from_numpy(Ac).cuda(), N, K)
    # (sums of whole numbers below 56 K < 2^24: exact in binary32 in any order)
    want = torch.from_numpy(np.asarray(lw, np.float32)[Wc]) @ torch.from_numpy(np.asarray(la, np.float32)[Ac]).T
    want = want.to(torch.int32).numpy()
    assert np.array_equal(want[:40, -40:], oracle.gemm(Wc[:40], Ac[-40:], lw, la))
    assert np.array_equal(dg.dg_gemm_lut(lut, Wp, Ap, M, N, K).cpu().numpy(), want)
    out = torch.zeros((N, M), dtype=torch.int32, device="cuda")
    dg.dg_gemm_lut(lut, Wp, Ap, M, N, K, out=out, strides=(1, M))
    assert np.array_equal(out.cpu().numpy().T, want)
