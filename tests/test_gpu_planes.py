"""Layers by the codes' bits, from unpacked codes and from packed 2-bit ones: every tile, 2-, 3- and 4-bit codes, K of whole and of broken runs and shares without any, taps
outside on every side, against the oracle; and AUTO's own choices."""
import numpy as np
import pytest
import torch

import oracle
from paper_2304_09049_amd import binding as dg
from paper_2304_09049_amd import workloads as wl

pytestmark = pytest.mark.gpu

NAMES = {"2": "codes_planes_64x64_k4", "4": "codes_planes_64x128_k2"}
TABLES = {  # activation level 0 is 0; 2-bit: any others, entries beyond int8; 3- and 4-bit: evenly spaced levels on both sides
    2: [((-50, -7, 9, 44), (0, 9, 31, 100)), ((127, -128, 5, 0), (0, -128, 127, 1)), ((-120, 40, 80, 0), (0, 6, -3, 9))],
    3: [(range(-4, 4), range(8)), (range(21, -11, -4), range(0, 24, 3)), ((5,) * 8, range(0, -8, -1))],
    4: [(range(-8, 8), range(16)), (range(-120, 120, 15), range(0, 112, 7)), (range(15, -1, -1), range(0, -16, -1))]}
CONVS = [  # B, H, W, Cin, Cout, KH, KW, stride, pad
    (1, 9, 11, 64, 36, 3, 3, (1, 1), (1, 1)), (2, 20, 13, 64, 132, 5, 5, (1, 1), (2, 2)), (1, 17, 19, 192, 64, 3, 2, (2, 1), (2, 0)),
    (3, 14, 14, 256, 200, 1, 1, (1, 1), (0, 0)), (2, 15, 14, 320, 68, 1, 1, (2, 2), (1, 1)), (1, 8, 40, 128, 100, 1, 4, (1, 3), (0, 3)),
    (1, 6, 28, 576, 4, 3, 3, (1, 1), (1, 1)), (2, 3, 3, 64, 64, 3, 3, (1, 1), (2, 2)), (1, 12, 12, 64, 65, 1, 1, (1, 1), (0, 0))]
# how many times as many images the 2-bit layers have: smaller ones pack while loading, whatever DG_PLANES says
TIMES = (96, 6, 48, 4, 48, 48, 1, 256, 1)


def run_layer(bits, plan, layer, lw, la, seed):
    B, H, W, Cin, Cout, KH, KW, stride, pad = layer
    lut = dg.dg_build_lut_bits(bits, lw, la, dg.DG_LUT_I16)
    desc = dg.conv_desc(B, H, W, Cin, Cout, KH, KW, stride, pad)
    assert dg.dg_conv_codes_kernel_name(lut, desc) == NAMES[plan], layer
    rng = np.random.default_rng(seed)
    Wc, Xc = wl.draw_codes(rng, (Cout, KH, KW, Cin), nlev=1 << bits), wl.draw_codes(rng, (B, H, W, Cin), nlev=1 << bits)
    high = rng.integers(0, 256 >> bits, Xc.shape, dtype=np.uint8) << bits                      # (counts for nothing)
    codes = torch.from_numpy(Xc | high).cuda()
    Wp = dg.dg_pack_codes_bits(torch.from_numpy(Wc).cuda(), Cout, KH * KW * Cin, bits)
    scale = torch.from_numpy(rng.uniform(0.01, 0.1, Cout).astype(np.float32)).cuda()
    work = torch.full((dg.dg_packed_bytes_bits(B * H * W, Cin, bits),), 77, dtype=torch.uint8, device="cuda")
    want = oracle.conv2d(Wc, Xc, lw, la, stride=stride, pad=pad)
    assert np.array_equal(dg.dg_conv2d_lut_codes(lut, Wp, codes, desc, work=work).cpu().numpy(), want), (layer, "int32")
    got = dg.dg_conv2d_lut_codes(lut, Wp, codes, desc, work=work, scale=scale).cpu().numpy()
    assert np.array_equal(got, oracle.scale_epilogue_nhwc(want, scale.cpu().numpy())), (layer, "scaled")
    assert bool((work == 77).all()), layer
    with pytest.raises(dg.DgError):                         # (a buffer is asked for as ever)
        dg.dg_conv2d_lut_codes(lut, Wp, codes, desc, work=work[:-1].clone())


@pytest.mark.parametrize("plan", ["2", "4"])
@pytest.mark.parametrize("bits", [2, 3, 4])
def test_planes_kernel(bits, plan, monkeypatch):
    monkeypatch.setenv("DG_PLANES", plan)
    for i, layer in enumerate(CONVS):
        lw, la = (list(x) for x in TABLES[bits][i % 3])
        run_layer(bits, plan, (layer[0] * TIMES[i],) + layer[1:] if bits == 2 else layer, lw, la, 100 * bits + i)


@pytest.mark.parametrize("plan", ["2", "4"])
def test_every_two_bit_table(plan, monkeypatch):
    """Three sums to an output, each counting for another part of the table: odd images, and an output width that is no whole tile."""
    monkeypatch.setenv("DG_PLANES", plan)
    for i, (lw, la) in enumerate(TABLES[2]):
        run_layer(2, plan, (12, 14, 14, 256, 200, 1, 1, (1, 1), (0, 0)), list(lw), list(la), i)
        run_layer(2, plan, (96, 9, 11, 64, 36, 3, 3, (1, 1), (1, 1)), list(lw), list(la), i)


LIMITS = {2: ((127, -128, 5, 0), (0, -128, 127, 1), 65472), 3: (range(21, -11, -4), range(0, 24, 3), 171136), 4: (range(-120, 120, 15), range(0, 112, 7), 37248)}


@pytest.mark.parametrize("bits,kernel", [(2, "2"), (2, "4"), (2, "packed"), (3, "2"), (3, "4"), (4, "2"), (4, "4")])
def test_sums_to_the_end_of_the_range(bits, kernel, monkeypatch):
    """The longest K that is taken, a bit's sum just below 2^23 in magnitude (2-bit: 128 K, 3-bit: 7 * 7 K, 4-bit: 15 * 15 K), the multiplications of whose
    24 bits would lose the next one's: rows and columns that climb to the largest codes."""
    lw, la, K = (list(LIMITS[bits][0]), list(LIMITS[bits][1]), LIMITS[bits][2])
    top = (1 << bits) - 1
    monkeypatch.setenv("DG_PLANES_PACKED" if kernel == "packed" else "DG_PLANES", "1" if kernel == "packed" else kernel)
    M, N = 68, 130 if bits != 2 or kernel == "packed" else 1030
    lut, desc = dg.dg_build_lut_bits(bits, lw, la, dg.DG_LUT_I16), dg.conv_desc(1, N, 1, K, M, 1, 1, (1, 1), (0, 0))
    name = dg.dg_conv_kernel_name(lut, desc) if kernel == "packed" else dg.dg_conv_codes_kernel_name(lut, desc)
    assert name == ("planes_64x128" if kernel == "packed" else NAMES[kernel])
    rng = np.random.default_rng(bits)
    Wc, Xc = rng.integers(0, top + 1, (M, K), dtype=np.uint8), rng.integers(0, top + 1, (N, K), dtype=np.uint8)
    for m in range(M):                                      # 2-bit: the codes whose level is the largest and the smallest
        Wc[m, : K * (m + 1) // M] = (m % 2 if bits == 2 else top)
    for n in range(0, N, 2):
        Xc[n, : K * (n + 2) // N] = 1 + n // 2 % 3 if bits == 2 else top
    Wc[-2:], Xc[N // 2 : N // 2 + 3] = ([[0], [1]] if bits == 2 else top), (np.arange(1, 4)[:, None] if bits == 2 else top)
    want = np.rint(np.asarray(lw, np.float64)[Wc] @ np.asarray(la, np.float64)[Xc].T).astype(np.int64).T             # (below 2^53: exact)
    assert np.abs(want).max() < 1 << 31
    Wp, X = dg.dg_pack_codes_bits(torch.from_numpy(Wc).cuda(), M, K, bits), torch.from_numpy(Xc).cuda()
    if kernel == "packed":
        got = dg.dg_conv2d_lut(lut, Wp, dg.dg_pack_codes_bits(X, N, K, bits), desc)
    else:
        work = torch.empty(dg.dg_packed_bytes_bits(N, K, bits), dtype=torch.uint8, device="cuda")
        got = dg.dg_conv2d_lut_codes(lut, Wp, X.view(1, N, 1, K), desc, work=work)
    assert np.array_equal(got.cpu().numpy().reshape(N, M), want)


def test_planes_kernel_on_packed_codes(monkeypatch):
    monkeypatch.setenv("DG_PLANES_PACKED", "1")
    for i, (B, H, W, Cin, Cout, KH, KW, stride, pad) in enumerate(CONVS):
        for lw, la in TABLES[2]:
            lut = dg.dg_build_lut(lw, la, dg.DG_LUT_I16)
            desc = dg.conv_desc(B, H, W, Cin, Cout, KH, KW, stride, pad)
            assert dg.dg_conv_kernel_name(lut, desc) == "planes_64x128", i
            rng = np.random.default_rng(i)
            Wc, Xc = wl.draw_codes(rng, (Cout, KH, KW, Cin)), wl.draw_codes(rng, (B, H, W, Cin))
            Wp = dg.dg_pack_weights(torch.from_numpy(Wc).cuda(), Cout, KH * KW * Cin)
            Xp = dg.dg_pack_activations(torch.from_numpy(Xc).cuda(), B * H * W, Cin)
            scale = torch.from_numpy(rng.uniform(0.01, 0.1, Cout).astype(np.float32)).cuda()
            want = oracle.conv2d(Wc, Xc, lw, la, stride=stride, pad=pad)
            assert np.array_equal(dg.dg_conv2d_lut(lut, Wp, Xp, desc).cpu().numpy(), want), (i, "int32")
            got = dg.dg_conv2d_lut(lut, Wp, Xp, desc, scale=scale).cpu().numpy()
            assert np.array_equal(got, oracle.scale_epilogue_nhwc(want, scale.cpu().numpy())), (i, "scaled")
    # a column-major product takes it, a row-major one does not
    lw, la = TABLES[2][0]
    lut, (M, N, K) = dg.dg_build_lut(lw, la, dg.DG_LUT_I16), (70, 300, 448)
    g = wl.small_gemm(M, N, K, seed=1)
    Wp, Ap = dg.dg_pack_weights(torch.from_numpy(g.Wc).cuda(), M, K), dg.dg_pack_activations(torch.from_numpy(g.Ac).cuda(), N, K)
    want = oracle.gemm(g.Wc, g.Ac, lw, la)
    for strides, shape in (((1, M + 3), (N, M + 3)), ((N, 1), (M, N))):
        out = torch.full(shape, -7, dtype=torch.int32, device="cuda")
        dg.dg_gemm_lut(lut, Wp, Ap, M, N, K, out=out, strides=strides)
        got = out.cpu().numpy()
        assert np.array_equal(got[:, :M].T if strides[0] == 1 else got, want) and (strides[0] != 1 or (got[:, M:] == -7).all()), strides


@pytest.mark.parametrize("shape,kernel", [((16, 28, 256, 256, 3, 1), "planes_64x128"), ((4, 112, 128, 40, 3, 1), "planes_64x128"),
                                          ((8, 28, 128, 128, 3, 1), "onehot_smfmac_2p_staged_32x128_k4"), ((2, 14, 384, 360, 3, 1), "onehot_mfma_2p_splitk_s14")])
def test_autos_own_choice_on_packed_codes(shape, kernel):
    B, H, Cin, Cout, k, s = shape
    lw, la = TABLES[2][0]
    lut = dg.dg_build_lut(lw, la, dg.DG_LUT_I16)
    desc = dg.conv_desc(B, H, H, Cin, Cout, k, k, (s, s), (k // 2, k // 2))
    assert dg.dg_conv_kernel_name(lut, desc) == kernel
    rng = np.random.default_rng(Cin + Cout)
    Wc, Xc = wl.draw_codes(rng, (Cout, k, k, Cin)), wl.draw_codes(rng, (B, H, H, Cin))
    size = B * H * H * Cout
    pos = np.unique(np.concatenate([rng.integers(0, size, 20000), np.arange(4 * Cout), size - 1 - np.arange(4 * Cout)]))
    want = oracle.conv2d_sampled(Wc, Xc, lw, la, pos, stride=(s, s), pad=(k // 2, k // 2))
    Wp = dg.dg_pack_weights(torch.from_numpy(Wc).cuda(), Cout, k * k * Cin)
    Xp = dg.dg_pack_activations(torch.from_numpy(Xc).cuda(), B * H * H, Cin)
    assert np.array_equal(dg.dg_conv2d_lut(lut, Wp, Xp, desc).cpu().numpy().reshape(-1)[pos], want)


@pytest.mark.parametrize("plan", ["2", "4"])
def test_matrix_products(plan, monkeypatch):
    """Column-major ones; row-major ones are packed first."""
    monkeypatch.setenv("DG_PLANES", plan)
    for bits, (M, N, K) in ((3, (70, 129, 192)), (4, (64, 300, 1152)), (4, (130, 64, 64))):
        lw, la = (list(x) for x in TABLES[bits][0])
        lut = dg.dg_build_lut_bits(bits, lw, la, dg.DG_LUT_I16)
        rng = np.random.default_rng(K)
        Wc, Ac = wl.draw_codes(rng, (M, K), nlev=1 << bits), wl.draw_codes(rng, (N, K), nlev=1 << bits)
        Wp = dg.dg_pack_codes_bits(torch.from_numpy(Wc).cuda(), M, K, bits)
        codes, want = torch.from_numpy(Ac).cuda(), oracle.gemm(Wc, Ac, lw, la)
        for strides, shape in (((1, M), (N, M)), ((N, 1), (M, N))):
            work = torch.full((dg.dg_packed_bytes_bits(N, K, bits),), 77, dtype=torch.uint8, device="cuda")
            out = torch.zeros(shape, dtype=torch.int32, device="cuda")
            dg.dg_gemm_lut_codes(lut, Wp, codes, M, N, K, work=work, out=out, strides=strides)
            assert np.array_equal(out.cpu().numpy(), want.T if strides[0] == 1 else want), (M, N, K, strides)
            assert bool((work == 77).all()) == (strides[0] == 1)


@pytest.mark.parametrize("bits,shape,kernel", [(4, (8, 28, 128, 128, 3, 1), "codes_planes_64x64_k4"), (3, (8, 28, 128, 128, 3, 1), "codes_planes_64x64_k4"),
                                               (2, (8, 28, 256, 256, 3, 1), "codes_planes_64x128_k2"), (2, (3, 28, 256, 256, 3, 1), "codes_planes_64x64_k4"),
                                               (3, (5, 112, 128, 112, 3, 2), "codes_planes_64x128_k2"),
                                               (4, (4, 112, 64, 112, 3, 1), "onehot_smfmac_4as2_staged_32x128"),
                                               (2, (2, 14, 384, 360, 3, 1), "onehot_mfma_2p_splitk_s14")])
def test_autos_own_choice(bits, shape, kernel):
    B, H, Cin, Cout, k, s = shape
    lw, la = (list(x) for x in TABLES[bits][0])
    lut = dg.dg_build_lut_bits(bits, lw, la, dg.DG_LUT_I16)
    desc = dg.conv_desc(B, H, H, Cin, Cout, k, k, (s, s), (k // 2, k // 2))
    assert dg.dg_conv_codes_kernel_name(lut, desc) == kernel
    rng = np.random.default_rng(Cin + Cout)
    Wc, Xc = wl.draw_codes(rng, (Cout, k, k, Cin), nlev=1 << bits), wl.draw_codes(rng, (B, H, H, Cin), nlev=1 << bits)
    OH = (H + 2 * (k // 2) - k) // s + 1
    size = B * OH * OH * Cout
    pos = np.unique(np.concatenate([rng.integers(0, size, 20000), np.arange(4 * Cout), size - 1 - np.arange(4 * Cout)]))
    want = oracle.conv2d_sampled(Wc, Xc, lw, la, pos, stride=(s, s), pad=(k // 2, k // 2))
    Wp = dg.dg_pack_codes_bits(torch.from_numpy(Wc).cuda(), Cout, k * k * Cin, bits)
    work = torch.empty(dg.dg_packed_bytes_bits(B * H * H, Cin, bits), dtype=torch.uint8, device="cuda")
    got = dg.dg_conv2d_lut_codes(lut, Wp, torch.from_numpy(Xc).cuda(), desc, work=work).cpu().numpy()
    assert np.array_equal(got.reshape(-1)[pos], want)


def test_tables_of_other_forms_are_packed_first(monkeypatch):
    """Uneven levels on either side, an activation level 0 that is not 0, no product of levels."""
    monkeypatch.setenv("DG_PLANES", "2")
    desc = dg.conv_desc(2, 12, 12, 64, 40, 3, 3, (1, 1), (1, 1))
    tables = [dg.dg_build_lut((-50, -7, 9, 44), (1, 9, 31, 100), dg.DG_LUT_I16), dg.dg_build_lut_entries([0, 300, 600, 900, 0, 1, 2, 4, 0, 0, 0, 0, 0, 1, 1, 1], dg.DG_LUT_I16),
              dg.dg_build_lut_bits(4, list(range(-8, 6)) + [7, 6], list(range(16))), dg.dg_build_lut_bits(4, list(range(-8, 8)), list(range(1, 17)), dg.DG_LUT_I16),
              dg.dg_build_lut_bits(3, list(range(-4, 4)), [0, 1, 2, 3, 4, 5, 7, 6])]
    for i, lut in enumerate(tables):
        assert not dg.dg_conv_codes_kernel_name(lut, desc).startswith("codes_planes"), i
    assert dg.dg_conv_codes_kernel_name(dg.dg_build_lut_bits(4, list(range(-8, 8)), list(range(16))), desc, "onehot_mfma").startswith("onehot_mfma")


@pytest.mark.parametrize("bits,shape,table", [(4, (3, 28, 128, 128, 3, 1), None), (3, (4, 28, 128, 96, 3, 1), None), (2, (6, 28, 384, 64, 3, 1), None),
                                              (2, (14, 112, 128, 96, 3, 2), ((-2, -1, 0, 1), (0, 1, 2, 3)))])
@pytest.mark.parametrize("ahead", [0, 4096])
def test_results_in_the_codes_place(bits, shape, table, ahead):
    """Layers that ask for a work buffer have read their codes before they store: results over the codes, and over their last bytes alone, are the same."""
    B, H, Cin, Cout, k, s = shape
    lw, la = (list(x) for x in table or TABLES[bits][0])
    lut = dg.dg_build_lut_bits(bits, lw, la, dg.DG_LUT_I16)
    desc = dg.conv_desc(B, H, H, Cin, Cout, k, k, (s, s), (k // 2, k // 2))
    assert dg.dg_conv_codes_kernel_name(lut, desc).startswith("codes_planes" if table is None else "codes_onebit")
    rng = np.random.default_rng(Cout)
    Wc, Xc = wl.draw_codes(rng, (Cout, k, k, Cin), nlev=1 << bits), wl.draw_codes(rng, (B, H, H, Cin), nlev=1 << bits)
    want = oracle.conv2d(Wc, Xc, lw, la, stride=(s, s), pad=(k // 2, k // 2))
    Wp = dg.dg_pack_codes_bits(torch.from_numpy(Wc).cuda(), Cout, k * k * Cin, bits)
    work = torch.empty(dg.dg_packed_bytes_bits(B * H * H, Cin, bits), dtype=torch.uint8, device="cuda")
    start = Xc.size - ahead if ahead else 0                 # of the results
    memory = torch.zeros(max(Xc.size, start + 4 * want.size), dtype=torch.uint8, device="cuda")
    codes, out = memory[: Xc.size].view(Xc.shape), memory[start : start + 4 * want.size].view(torch.int32).view(want.shape)
    codes.copy_(torch.from_numpy(Xc))
    dg.dg_conv2d_lut_codes(lut, Wp, codes, desc, work=work, out=out)
    assert np.array_equal(out.cpu().numpy(), want)
