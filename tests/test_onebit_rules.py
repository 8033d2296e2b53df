"""Which calls AUTO takes to the kernel for tables that are two one-bit lookups: the names it gives on both sides of each line of the rule (256
compute units, as without a device)."""
import pytest

from paper_2304_09049_amd import binding as dg

UNSIGNED = (0, 1, 2, 3)
WIDE = (-100, 50, 0, 75)          # entries beyond int8, which cost the other kernels twice as much


@pytest.fixture(autouse=True)
def no_overrides(monkeypatch):
    for name in ("DG_ONEBIT", "DG_ONEBIT_CODES", "DG_ONEHOT_PLAN", "DG_ONEHOT_WAVES", "DG_ONEHOT_CODES_TILED"):
        monkeypatch.delenv(name, raising=False)


def gemm(M, N, K, lw=(-2, -1, 0, 1), la=UNSIGNED):
    return dg.dg_gemm_kernel_name(dg.dg_build_lut(lw, la, dg.DG_LUT_I16), M, N, K)


def conv(B, H, W, Cin, Cout, k, stride=1, lw=(-2, -1, 0, 1), pad=None):
    lut, pad = dg.dg_build_lut(lw, UNSIGNED, dg.DG_LUT_I16), k // 2 if pad is None else pad
    desc = dg.conv_desc(B, H, W, Cin, Cout, k, k, (stride, stride), (pad, pad))
    return dg.dg_conv_kernel_name(lut, desc), dg.dg_conv_codes_kernel_name(lut, desc)


def test_sizes():
    # 129 and 130 tiles of 64 x 128 in place of the staged kernel, 34 and 35 of the direct loads
    assert conv(1, 129, 128, 128, 64, 3)[0] == "onehot_smfmac_staged_32x64" and conv(1, 130, 128, 128, 64, 3)[0] == "onebit_64x128"
    assert gemm(34 * 64, 128, 5568) == "onehot_mfma_64x32_k4" and gemm(35 * 64, 128, 5568) == "onebit_64x128_k2"
    # 46 and 66 of the split-K kernel (35 with entries beyond int8)
    assert conv(2, 28, 28, 512, 144, 3)[0] == gemm(450, 530, 4608) == "onehot_mfma_splitk_s12" and gemm(80, 4112, 2880) == "onebit_64x128_k2"
    assert gemm(1416, 135, 6912) == "onehot_mfma_splitk_s10" and gemm(2240, 65, 5568, lw=WIDE) == "onebit_64x128_k2"
    # 1.5e9 operations
    assert not gemm(1100, 256, 2624).startswith("onebit") and gemm(1100, 256, 2752) == "onebit_64x128_k2"
    # 139 and 140 tiles from unpacked codes
    assert conv(1, 139, 128, 64, 48, 3)[1] == "codes_onehot_smfmac_64x32" and conv(1, 140, 128, 64, 48, 3)[1] == "codes_onebit_64x128"
    # layers of the stationary-weight kernel stay there
    assert conv(32, 56, 56, 256, 64, 1) == ("onehot_smfmac_ws_32xK", "codes_onehot_smfmac_ws_32xK")


def test_half_empty_tiles():
    """64 columns or fewer and 32 rows or fewer leave half of a tile empty."""
    assert gemm(4096, 64, 5568) == "onehot_mfma_splitk_s8" and gemm(4096, 65, 5568) == "onebit_64x128_k2"
    assert gemm(11008, 64, 4096) == "onehot_smfmac_staged_32x64_k4" and gemm(11008, 65, 4096) == "onebit_64x128_k2"
    assert gemm(11008, 32, 4096, lw=WIDE) == "onebit_64x128_k2" and gemm(4096, 64, 5568, lw=WIDE) == "onehot_mfma_2p_splitk_s8"
    assert conv(1, 8, 8, 576, 12000, 1)[1] == "codes_onehot_smfmac_64x32_k4" and conv(1, 5, 13, 576, 12000, 1)[1] == "codes_onebit_64x128"
    # 32 rows: not in place of staged tiles of that height, but of others
    assert conv(32, 56, 56, 128, 32, 3)[0] == "onehot_smfmac_staged_32x128" and conv(32, 56, 56, 128, 36, 3)[0] == "onebit_64x256"
    assert conv(16, 56, 56, 384, 16, 3)[0] == "onehot_smfmac_staged_32x128_k2" and conv(16, 112, 112, 64, 16, 3)[0] == "onebit_64x128"
    assert gemm(32, 262144, 320) == "onehot_smfmac_64x32"
    assert gemm(32, 262144, 448) == "onebit_64x128" and gemm(33, 262144, 320).startswith("onebit")


def test_large_outputs_of_short_sums():
    # pixels' rows: narrow tiles for one or two runs, wide ones for three; none of 4000 sums and more for one
    assert conv(1, 400, 250, 192, 1000, 1)[0] == conv(1, 400, 250, 384, 1000, 1)[0] == "onebit_64x128"
    assert conv(1, 400, 250, 576, 1000, 1)[0] == "onebit_64x256_64x128"
    assert conv(1, 160, 128, 192, 4096, 1)[0] == "onehot_smfmac_64x64" and conv(1, 160, 128, 320, 4096, 1)[0] == "onebit_64x256"
    assert conv(1, 32, 128, 192, 4096, 1)[0] == "onebit_64x128"
    # channels' rows: wide
    assert gemm(4096, 20480, 192) == gemm(1024, 65536, 192) == "onebit_64x256"


@pytest.mark.parametrize("M,N,K,kernel", [
    (1024, 2048, 512, "onebit_64x128"), (1024, 2048, 2048, "onebit_64x128_k2"),                  # 256 tiles: K shared from eight runs on
    (1024, 2176, 2048, "onebit_64x128"),                                                          # 272: two rounds
    (1024, 4096, 2304, "onebit_64x128"), (1024, 4224, 2304, "onebit_64x256_64x128"),              # 512, 528: wide tiles, the rest narrow
    (1000, 8100, 1280, "onebit_64x256"), (1000, 8100, 1024, "onebit_64x128"),                    # five runs and four
    (1000, 16301, 2112, "onebit_64x512"), (1000, 16301, 2048, "onebit_64x256"),                  # nine runs and eight
])
def test_tiles(M, N, K, kernel):
    assert gemm(M, N, K) == kernel


def test_tables():
    big = (1024, 2048, 512)
    for lw in ((-2, -1, 0, 1), (12, -8, 3, -6), (0, 0, 0, 0), (7, 14, 21, 28), (-100, 50, 0, 75), (-128, 64, 96, 32)):
        assert gemm(*big, lw=lw) == "onebit_64x128", lw
    assert gemm(*big, la=(0, -2, -4, -6)) == "onebit_64x128"
    for lw in ((-2, 5, 0, 1), (-7, 7, 14, 1), (0, 1, 2, 9), (127, 126, 0, 1)):                   # levels that FP4 has not
        assert not gemm(*big, lw=lw).startswith("onebit"), lw
    for la in ((1, 2, 3, 4), (0, 1, 2, 4), (0, 1, 3, 4), (0, 2, 1, 3), (-2, -1, 0, 1), (3, 2, 1, 0)):
        assert not gemm(*big, la=la).startswith("onebit"), la
    wide = dg.dg_build_lut_bits(3, list(range(-4, 4)), list(range(8)))
    assert not dg.dg_gemm_kernel_name(wide, *big).startswith("onebit")
    # sums whose quarters a binary32 number no longer holds: 3 * 12 * K from 2^24 on
    assert gemm(2560, 128, 466048 - 64, lw=(12, 8, 3, 1)).startswith("onebit")
    assert not gemm(2560, 128, 466048, lw=(12, 8, 3, 1)).startswith("onebit")


def test_shapes():
    assert gemm(1024, 2048, 576).startswith("onebit") and not gemm(1024, 2048, 544).startswith("onebit")       # Cin % 64
    # 32 filter taps and 33
    lut = dg.dg_build_lut((-2, -1, 0, 1), UNSIGNED)
    name = [dg.dg_conv_kernel_name(lut, dg.conv_desc(4, 64, 64, 128, 128, *k, (1, 1), (0, 0))) for k in ((4, 8), (3, 11))]
    assert name[0].startswith("onebit") and not name[1].startswith("onebit")
    # 2^24 - 1 workgroups of 256 threads, and one more than a launch takes
    assert gemm(2 ** 30 - 64, 1, 320, lw=WIDE) == "onebit_64x128" and gemm(2 ** 30 - 1, 1, 320, lw=WIDE).startswith("onehot_mfma_2p_")
    # other variants are never replaced
    desc = dg.conv_desc(32, 56, 56, 256, 256, 3, 3, (1, 1), (1, 1))
    assert dg.dg_conv_kernel_name(lut, desc, "onehot_smfmac") == "onehot_smfmac_staged_32x224"
    assert dg.dg_conv_kernel_name(lut, desc, "onehot_mfma").startswith("onehot_mfma_")
    assert not dg.dg_conv_codes_kernel_name(lut, dg.conv_desc(1, 140, 128, 64, 48, 3, 3, (1, 1), (1, 1)), "onehot_smfmac").startswith("codes_onebit")


def test_codes_in_place_of_packing():
    # 150 tiles, five readings of a pixel's codes, 1152 positions; K that two halves of a workgroup share; a 1x1 layer whose pixels are packed sparsely
    assert conv(1, 300, 128, 128, 128, 3, 2)[1] == "codes_onebit_64x128" and conv(1, 296, 128, 128, 128, 3, 2)[1] == "onebit_64x128"
    assert conv(1, 300, 256, 128, 128, 3, 2)[1] == "codes_onebit_64x128" and conv(1, 300, 256, 128, 132, 3, 2)[1] == "onebit_64x128"
    assert conv(1, 400, 512, 1152, 64, 1)[1] == "codes_onebit_64x128" and conv(1, 400, 512, 1216, 64, 1)[1] == "onebit_64x256_64x128"
    assert conv(6, 54, 64, 256, 88, 3, 2)[1] == "onebit_64x128_k2" and conv(16, 56, 56, 256, 256, 3)[1] == "onebit_64x256_64x128"


def test_codes_of_many_rounds_are_packed_first():
    """Several tiles of channels that read the codes of many rounds of tiles measured up to 39 % longer than packing first: no more than four rounds
    (1024 tiles), with two tiles and one tap six (1536), with one tile any."""
    for layer in ((10, 56, 56, 512, 296, 1), (14, 112, 112, 384, 260, 1), (19, 112, 112, 576, 112, 1), (3, 112, 112, 512, 252, 1), (9, 112, 112, 320, 124, 1),
                  (12, 112, 224, 128, 124, 3, 2)):
        assert conv(*layer)[1] == conv(*layer)[0] and conv(*layer)[0].startswith("onebit_"), layer
    assert conv(1, 256, 128, 384, 256, 1)[1] == "codes_onebit_64x128" and conv(1, 257, 128, 384, 256, 1)[1].startswith("onebit_")
    assert conv(1, 768, 128, 320, 128, 1)[1] == "codes_onebit_64x128" and conv(1, 769, 128, 320, 128, 1)[1].startswith("onebit_")
    assert conv(2, 512, 256, 128, 128, 3, 2)[1] == "codes_onebit_64x128" and conv(2, 514, 256, 128, 128, 3, 2)[1].startswith("onebit_")
    assert conv(24, 112, 112, 576, 64, 1)[1] == "codes_onebit_64x128"
