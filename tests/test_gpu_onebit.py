"""Tables that are two one-bit lookups of the activation code, on the FP4 matrix instruction: every tile, with and without a filter
window, K of whole and of broken runs, every way to the output, against the oracle; and sums at the end of the range that is taken."""
import numpy as np
import pytest
import torch

import oracle
from paper_2304_09049_amd import binding as dg
from paper_2304_09049_amd import workloads as wl

pytestmark = pytest.mark.gpu

TABLES = [((-2, -1, 0, 1), (0, 1, 2, 3)), ((12, -8, 3, -6), (0, 1, 2, 3)), ((-10, 5, 0, 15), (0, -2, -4, -6)), ((0, 0, 0, 0), (0, 1, 2, 3)),
          ((-100, 50, 0, 75), (0, 1, 2, 3))]                # (the last: entries down to -300, beyond int8)
NAMES = {"1": "onebit_64x128", "2": "onebit_64x256", "4": "onebit_64x512", "12": "onebit_64x128_k2", "21": "onebit_64x256_64x128"}
CONVS = [  # B, H, W, Cin, Cout, KH, KW, stride, pad: 1 to 25 taps, tiles and runs whole and not, taps outside on every side, padding without a window
    (1, 9, 11, 64, 36, 3, 3, (1, 1), (1, 1)), (2, 20, 13, 64, 132, 5, 5, (1, 1), (2, 2)), (1, 17, 19, 192, 64, 3, 2, (2, 1), (2, 0)),
    (3, 14, 14, 256, 200, 1, 1, (1, 1), (0, 0)), (2, 15, 14, 320, 68, 1, 1, (2, 2), (1, 1)), (1, 8, 40, 128, 100, 1, 4, (1, 3), (0, 3)),
    (1, 28, 28, 576, 4, 3, 3, (1, 1), (1, 1)), (2, 3, 3, 64, 64, 3, 3, (1, 1), (2, 2))]
GEMMS = [(70, 300, 64), (64, 1025, 320), (300, 65, 2304), (129, 513, 1088), (1, 3, 128)]


@pytest.mark.parametrize("plan", ["1", "2", "4", "12", "21"])
def test_onebit_kernel(plan, monkeypatch):
    monkeypatch.setenv("DG_ONEBIT", plan)
    for i, (B, H, W, Cin, Cout, KH, KW, stride, pad) in enumerate(CONVS):
        lw, la = TABLES[i % len(TABLES)]
        lut = dg.dg_build_lut(lw, la, dg.DG_LUT_I16)
        c = wl.small_conv(B, H, W, Cin, Cout, KH, KW, stride, pad, seed=H + Cin, scale=True)
        desc = dg.conv_desc(B, H, W, Cin, Cout, KH, KW, stride, pad)
        assert dg.dg_conv_kernel_name(lut, desc) == NAMES[plan], i
        scale = torch.from_numpy(c.scale).cuda()
        Wp = dg.dg_pack_weights(torch.from_numpy(c.Wc).cuda(), Cout, KH * KW * Cin)
        Xp = dg.dg_pack_activations(torch.from_numpy(c.Ac).cuda(), B * H * W, Cin)
        want = oracle.conv2d(c.Wc, c.Ac, lw, la, stride=stride, pad=pad)
        wants = oracle.scale_epilogue_nhwc(want, c.scale)
        assert np.array_equal(dg.dg_conv2d_lut(lut, Wp, Xp, desc).cpu().numpy(), want), (i, "int32")
        assert np.array_equal(dg.dg_conv2d_lut(lut, Wp, Xp, desc, scale=scale).cpu().numpy(), wants), (i, "scaled")
        got = dg.dg_conv2d_lut_requant(lut, Wp, Xp, desc, scale, 1.5, 0.5, 0).cpu().numpy()
        codes = np.clip(np.rint(np.float32(1.5) * wants + np.float32(0.5)), 0, 3).astype(np.uint8).reshape(-1, Cout // 4, 4)
        assert np.array_equal(got, (codes << np.array([0, 2, 4, 6], dtype=np.uint8)).sum(-1).astype(np.uint8).reshape(-1)), (i, "requantised")
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
                out = torch.zeros(shape, dtype=torch.int32 if s is None else torch.float32, device="cuda")
                dg.dg_gemm_lut(lut, Wp, Ap, M, N, K, out=out, strides=strides, scale=s)
                assert np.array_equal(view(out.cpu().numpy()), w), ((M, N, K), strides, s is not None)


def test_onebit_kernel_on_unpacked_codes(monkeypatch):
    """The same from codes one per byte, whose higher bits count for nothing; the work buffer is left alone."""
    monkeypatch.setenv("DG_ONEBIT_CODES", "1")
    for i, (B, H, W, Cin, Cout, KH, KW, stride, pad) in enumerate(CONVS + [(1, 12, 30, 256, 70, 1, 1, (1, 1), (0, 0)), (1, 12, 30, 64, 64, 1, 1, (1, 1), (0, 0)),
                                                                           (16, 56, 56, 256, 72, 1, 1, (1, 1), (0, 0)), (8, 28, 28, 512, 96, 1, 1, (1, 1), (0, 0))]):
        if KH * KW * Cin > 3072:                            # (two kernels)
            continue
        lw, la = TABLES[i % (5 if i < 8 else 4)]            # (entries beyond int8 are packed while loading only by the split-K kernel)
        lut = dg.dg_build_lut(lw, la, dg.DG_LUT_I16)
        c = wl.small_conv(B, H, W, Cin, Cout, KH, KW, stride, pad, seed=H + Cin, scale=True)
        desc = dg.conv_desc(B, H, W, Cin, Cout, KH, KW, stride, pad)
        assert dg.dg_conv_codes_kernel_name(lut, desc) == "codes_onebit_64x128", i
        scale = torch.from_numpy(c.scale).cuda()
        high = torch.randint(0, 64, (c.Ac.size,), dtype=torch.uint8, device="cuda", generator=torch.Generator("cuda").manual_seed(i)) * 4
        X = torch.from_numpy(c.Ac).cuda().reshape(-1) + high
        Wp = dg.dg_pack_weights(torch.from_numpy(c.Wc).cuda(), Cout, KH * KW * Cin)
        work = torch.full((B * H * W * Cin // 4,), 77, dtype=torch.uint8, device="cuda")
        want = oracle.conv2d(c.Wc, c.Ac, lw, la, stride=stride, pad=pad)
        assert np.array_equal(dg.dg_conv2d_lut_codes(lut, Wp, X, desc, work=work).cpu().numpy(), want), (i, "int32")
        got = dg.dg_conv2d_lut_codes(lut, Wp, X, desc, work=work, scale=scale).cpu().numpy()
        assert np.array_equal(got, oracle.scale_epilogue_nhwc(want, c.scale)), (i, "scaled")
        assert bool((work == 77).all()), i


def test_tables_of_other_forms_stay_with_the_general_kernels(monkeypatch):
    """A level that FP4 does not have, activation levels that are not evenly spaced from zero: taken whole, with the kernel above forced;
    and a table given entry by entry that is of its form."""
    monkeypatch.setenv("DG_ONEBIT", "1")
    B, H, W, Cin, Cout = 1, 15, 17, 128, 68
    c = wl.small_conv(B, H, W, Cin, Cout, 3, 3, (1, 1), (1, 1), seed=3)
    desc = dg.conv_desc(B, H, W, Cin, Cout, 3, 3, (1, 1), (1, 1))
    Wp = dg.dg_pack_weights(torch.from_numpy(c.Wc).cuda(), Cout, 9 * Cin)
    Xp = dg.dg_pack_activations(torch.from_numpy(c.Ac).cuda(), B * H * W, Cin)
    for lw, la in (((-2, 5, 0, 1), (0, 1, 2, 3)), ((-2, -1, 0, 1), (1, 2, 3, 4)), ((-2, -1, 0, 1), (0, 1, 2, 4)), ((-2, -1, 0, 1), (0, 1, 3, 4)),
                   ((-2, -1, 0, 1), (0, 2, 1, 3)), ((-7, 7, 14, 1), (0, 1, 2, 3))):
        lut = dg.dg_build_lut(lw, la)
        assert not dg.dg_conv_kernel_name(lut, desc).startswith("onebit"), (lw, la)
        got = dg.dg_conv2d_lut(lut, Wp, Xp, desc).cpu().numpy()
        assert np.array_equal(got, oracle.conv2d(c.Wc, c.Ac, lw, la, stride=(1, 1), pad=(1, 1))), (lw, la)
    lw, la = (-3, -1, 1, 3), (0, 1, 2, 3)
    lut = dg.dg_build_lut_entries([w * a for w in lw for a in la])
    assert dg.dg_conv_kernel_name(lut, desc) == "onebit_64x128"
    assert np.array_equal(dg.dg_conv2d_lut(lut, Wp, Xp, desc).cpu().numpy(), oracle.conv2d(c.Wc, c.Ac, lw, la, stride=(1, 1), pad=(1, 1)))


def test_sums_to_the_end_of_the_range(monkeypatch):
    """Sums of every magnitude up to the largest that is taken, 3 * 4 * K just below 2^24, in steps of the smallest entry: exact."""
    M, N, K = 64, 40, 1398016
    lw, la = (-4, 1, 3, 4), (0, 1, 2, 3)
    rng = np.random.default_rng(5)
    Wc, Ac = rng.integers(0, 4, (M, K), dtype=np.uint8), rng.integers(0, 4, (N, K), dtype=np.uint8)
    for m in range(0, M, 2):                                # rows that climb to ever larger sums, on columns of the largest code
        Wc[m, : K * (m + 2) // M] = 3
    Ac[: N // 2] = 3
    Wc[1], Ac[1, ::7] = 0, 0
    lut = dg.dg_build_lut(lw, la)
    Wp, Ap = dg.dg_pack_weights(torch.from_numpy(Wc).cuda(), M, K), dg.dg_pack_activations(torch.from_numpy(Ac).cuda(), N, K)
    want = np.rint(np.asarray(lw, np.float64)[Wc] @ np.asarray(la, np.float64)[Ac].T).astype(np.int64)      # (below 2^53: exact)
    assert 2 ** 24 - 2 ** 10 <= np.abs(want).max() < 2 ** 24
    for plan in ("1", "12"):
        monkeypatch.setenv("DG_ONEBIT", plan)
        assert dg.dg_gemm_kernel_name(lut, M, N, K) == NAMES[plan]
        assert np.array_equal(dg.dg_gemm_lut(lut, Wp, Ap, M, N, K).cpu().numpy(), want), plan


AUTOS = [(1000, 2045, 512, "onebit_64x128"), (738, 360, 5568, "onebit_64x128_k2"), (1000, 8100, 1280, "onebit_64x256"),
         (1024, 4220, 2304, "onebit_64x256_64x128"), (1000, 16301, 2112, "onebit_64x512")]


@pytest.mark.parametrize("M,N,K,kernel", AUTOS)
def test_autos_own_plans(M, N, K, kernel):
    """Products of a size at which AUTO chooses each tile by itself: every sum, row- and column-major."""
    lw, la = TABLES[1]
    rng = np.random.default_rng(N)
    Wc, Ac = rng.integers(0, 4, (M, K), dtype=np.uint8), rng.integers(0, 4, (N, K), dtype=np.uint8)
    lut = dg.dg_build_lut(lw, la)
    assert dg.dg_gemm_kernel_name(lut, M, N, K) == kernel
    Wp, Ap = dg.dg_pack_weights(torch.from_numpy(Wc).cuda(), M, K), dg.dg_pack_activations(torch.from_numpy(Ac).cuda(), N, K)
    # (sums of whole numbers below 36 K < 2^24: exact in binary32 in any order)
    want = torch.from_numpy(np.asarray(lw, np.float32)[Wc]) @ torch.from_numpy(np.asarray(la, np.float32)[Ac]).T
    want = want.to(torch.int32).numpy()
    assert np.array_equal(want[:40, -40:], oracle.gemm(Wc[:40], Ac[-40:], lw, la))
    assert np.array_equal(dg.dg_gemm_lut(lut, Wp, Ap, M, N, K).cpu().numpy(), want)
    out = torch.zeros((N, M), dtype=torch.int32, device="cuda")
    dg.dg_gemm_lut(lut, Wp, Ap, M, N, K, out=out, strides=(1, M))
    assert np.array_equal(out.cpu().numpy().T, want)


@pytest.mark.parametrize("B", [20, 21])
def test_window_and_shared_k_on_both_sides_of_the_caches(B, monkeypatch):
    """Weights and activations of 2^24 codes, from which on another form runs: sampled sums, re-quantised ones of the same pixels."""
    H, Cin, Cout, k = 56, 256, 68, 3
    assert (B * H * H * Cin + Cout * k * k * Cin > 1 << 24) == (B == 21)
    monkeypatch.setenv("DG_ONEBIT", "12")
    lw, la = TABLES[1]
    lut, desc = dg.dg_build_lut(lw, la, dg.DG_LUT_I16), dg.conv_desc(B, H, H, Cin, Cout, k, k, (1, 1), (1, 1))
    assert dg.dg_conv_kernel_name(lut, desc) == NAMES["12"]
    rng = np.random.default_rng(B)
    Wc, Xc = wl.draw_codes(rng, (Cout, k, k, Cin)), wl.draw_codes(rng, (B, H, H, Cin))
    size = B * H * H * Cout
    pos = np.unique(np.concatenate([rng.integers(0, size, 20000), np.arange(4 * Cout), size - 1 - np.arange(4 * Cout)]))
    want = oracle.conv2d_sampled(Wc, Xc, lw, la, pos, stride=(1, 1), pad=(1, 1))
    Wp, Xp = dg.dg_pack_weights(torch.from_numpy(Wc).cuda(), Cout, k * k * Cin), dg.dg_pack_activations(torch.from_numpy(Xc).cuda(), B * H * H, Cin)
    assert np.array_equal(dg.dg_conv2d_lut(lut, Wp, Xp, desc).cpu().numpy().reshape(-1)[pos], want)
    scale = rng.uniform(0.001, 0.01, Cout).astype(np.float32)
    got = dg.dg_conv2d_lut_requant(lut, Wp, Xp, desc, torch.from_numpy(scale).cuda(), 1.5, 0.5, 0).cpu().numpy().reshape(-1)
    codes = np.clip(np.rint(np.float32(1.5) * (want.astype(np.float32) * scale[pos % Cout]) + np.float32(0.5)), 0, 3).astype(np.uint8)
    assert np.array_equal(got[pos // 4] >> (2 * (pos % 4)) & 3, codes)


@pytest.mark.parametrize("codes", [False, True])
def test_padding_pixel_at_the_end_of_the_32_bit_offsets(codes, monkeypatch):
    """A padded 1x1 layer whose pixels below the image would lie just under byte 2^31: every output is padding, hence zero, wherever in the
    pixel's row the piece of K lies."""
    monkeypatch.setenv("DG_ONEBIT_CODES" if codes else "DG_ONEBIT", "1")
    Cin, Cout, W = 192, 64, 5592405 if codes else 22369621
    used = 2 * W * (Cin if codes else Cin // 4)
    assert 2 ** 31 - Cin < used < 2 ** 31
    lut = dg.dg_build_lut((-2, -1, 0, 1), (0, 1, 2, 3))
    desc = dg.conv_desc(1, 2, W, Cin, Cout, 1, 1, (3, W), (1, 0))           # rows -1 and 2 of two, column 0
    Wp = torch.zeros(Cout * Cin // 4, dtype=torch.uint8, device="cuda")
    X = torch.full((used,), 255, dtype=torch.uint8, device="cuda")
    name = dg.dg_conv_codes_kernel_name if codes else dg.dg_conv_kernel_name
    assert name(lut, desc) == ("codes_onebit_64x128" if codes else "onebit_64x128")
    if codes:
        got = dg.dg_conv2d_lut_codes(lut, Wp, X, desc, work=torch.empty(used // 4, dtype=torch.uint8, device="cuda"))
    else:
        got = dg.dg_conv2d_lut(lut, Wp, X, desc)
    assert got.shape == (1, 2, 1, Cout) and not got.any()


@pytest.mark.parametrize("value", ["3", "8", "-1", "", "1x"])
def test_override_values_that_are_none(value, monkeypatch):
    """Values that DG_ONEBIT does not have count as not set: the whole output is written."""
    monkeypatch.setenv("DG_ONEBIT", value)
    lw, la = TABLES[0]
    c = wl.small_conv(2, 20, 13, 64, 132, 3, 3, (1, 1), (1, 1), seed=7)
    desc = dg.conv_desc(2, 20, 13, 64, 132, 3, 3, (1, 1), (1, 1))
    Wp = dg.dg_pack_weights(torch.from_numpy(c.Wc).cuda(), 132, 9 * 64)
    Xp = dg.dg_pack_activations(torch.from_numpy(c.Ac).cuda(), 2 * 20 * 13, 64)
    out = torch.full((2, 20, 13, 132), 1 << 30, dtype=torch.int32, device="cuda")
    dg.dg_conv2d_lut(dg.dg_build_lut(lw, la), Wp, Xp, desc, out=out)
    assert np.array_equal(out.cpu().numpy(), oracle.conv2d(c.Wc, c.Ac, lw, la, stride=(1, 1), pad=(1, 1)))


@pytest.mark.parametrize("layer", [(1, 300, 128, 128, 128, 3, 2), (14, 113, 109, 128, 60, 3, 2), (39, 28, 28, 384, 232, 1, 1), (3, 57, 55, 128, 132, 5, 1)])
def test_codes_in_place_of_packing(layer, monkeypatch):
    """Layers that are not packed first: the work buffer is asked for and left alone, higher bits of a code count for nothing."""
    B, H, W, Cin, Cout, k, s = layer
    if k == 5:
        monkeypatch.setenv("DG_ONEBIT_CODES", "2")          # (a layer that is packed first otherwise)
    lw, la = (-2, -1, 0, 1), (0, 1, 2, 3)
    lut, desc = dg.dg_build_lut(lw, la), dg.conv_desc(B, H, W, Cin, Cout, k, k, (s, s), (k // 2, k // 2))
    OH, OW = ((x + 2 * (k // 2) - k) // s + 1 for x in (H, W))
    rng = np.random.default_rng(H + Cout)
    Wc, Xc = wl.draw_codes(rng, (Cout, k, k, Cin)), wl.draw_codes(rng, (B, H, W, Cin))
    Wp, X = dg.dg_pack_weights(torch.from_numpy(Wc).cuda(), Cout, k * k * Cin), torch.from_numpy(Xc + 4 * (Xc ^ 1)).cuda()
    work = torch.full((B * H * W * Cin // 4,), 77, dtype=torch.uint8, device="cuda")
    size = B * OH * OW * Cout
    pos = np.unique(np.concatenate([rng.integers(0, size, 20000), np.arange(4 * Cout), size - 1 - np.arange(4 * Cout)]))
    want = oracle.conv2d_sampled(Wc, Xc, lw, la, pos, stride=(s, s), pad=(k // 2, k // 2))
    assert dg.dg_conv_codes_kernel_name(lut, desc) == "codes_onebit_64x128"
    got = dg.dg_conv2d_lut_codes(lut, Wp, X, desc, work=work).cpu().numpy().reshape(-1)
    assert np.array_equal(got[pos], want) and bool((work == 77).all())
    if k != 5:
        with pytest.raises(dg.DgError, match="needed"):
            dg.dg_conv2d_lut_codes(lut, Wp, X, desc, work=work[:-16])
