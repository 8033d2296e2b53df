"""Which calls AUTO takes to the kernels that read codes by their bits: their names on both sides of the rules (256 compute units, as without a
device)."""
import pytest

from paper_2304_09049_amd import binding as dg


@pytest.fixture(autouse=True)
def no_overrides(monkeypatch):
    for name in ("DG_PLANES", "DG_PLANES_PACKED", "DG_ONEBIT", "DG_ONEBIT_CODES", "DG_ONEHOT_PLAN", "DG_ONEHOT_WAVES", "DG_NIBBLES", "DG_STAGED_2P",
                 "DG_STAGED_2P_PLAN"):
        monkeypatch.delenv(name, raising=False)


def names(bits, B, H, W, Cin, Cout, k, s=1):
    """The kernel on packed codes, and from codes."""
    lut = dg.dg_build_lut_bits(bits, list(range(-(1 << bits) // 2, (1 << bits) // 2)), list(range(1 << bits)))
    desc = dg.conv_desc(B, H, W, Cin, Cout, k, k, (s, s), (k // 2, k // 2))
    return dg.dg_conv_kernel_name(lut, desc), dg.dg_conv_codes_kernel_name(lut, desc)


@pytest.mark.parametrize("bits,layer", [(4, (315, 1, 1, 128, 1564, 1)), (3, (341, 1, 1, 128, 744, 1)), (4, (17, 36, 36, 64, 352, 1, 2)), (3, (19, 28, 28, 64, 544, 1, 2)),
                                        (4, (727, 1, 1, 128, 516, 1)), (4, (1855, 1, 1, 192, 140, 1)), (3, (729, 1, 1, 256, 324, 1)), (4, (286, 1, 1, 256, 1628, 1)),
                                        (4, (8, 28, 28, 64, 780, 1, 2)), (3, (734, 1, 1, 64, 424, 1)), (4, (715, 1, 1, 384, 252, 1)), (3, (15, 7, 7, 320, 844, 1, 2))])
def test_short_sums_of_few_blocks_are_packed_first(bits, layer):
    """Layers that measured 3 to 25 % longer by the codes' bits."""
    packed, codes = names(bits, *layer)
    assert packed.startswith("onehot_smfmac_4as2_") and codes == packed


@pytest.mark.parametrize("bits,layer,kernel", [(4, (8, 28, 28, 128, 128, 3), "codes_planes_64x64_k4"), (3, (8, 28, 28, 128, 128, 3), "codes_planes_64x64_k4"),
                                               (3, (5, 112, 112, 128, 112, 3, 2), "codes_planes_64x128_k2"), (4, (8, 56, 56, 128, 48, 1), "codes_planes_64x128_k2"),
                                               (3, (5, 56, 56, 64, 24, 1), "codes_planes_64x128_k2")])
def test_layers_by_their_bits(bits, layer, kernel):
    packed, codes = names(bits, *layer)
    assert packed.startswith("onehot_smfmac_4as2_") and codes == kernel


WIDE = ((127, -128, 5, 0), (0, -128, 127, 1))


def test_large_outputs_of_half_runs_stay_in_two_planes():
    lut = dg.dg_build_lut(*WIDE, dg.DG_LUT_I16)
    name = lambda B, H, W, Cin, Cout, s: dg.dg_conv_kernel_name(lut, dg.conv_desc(B, H, W, Cin, Cout, 1, 1, (s, s), (0, 0)))
    for layer in ((26, 56, 56, 64, 1480, 2), (23, 28, 27, 64, 1968, 1), (3, 112, 112, 64, 652, 1)):          # up to 3 % longer by their bits
        assert name(*layer).startswith("onehot_mfma_2p_"), layer
    assert name(4, 56, 56, 64, 804, 1) == name(26, 56, 56, 128, 1480, 2) == "planes_64x128"


@pytest.mark.parametrize("bits,K", [(2, 65472), (3, 171136), (4, 37248)])
def test_the_end_of_the_range(bits, K, monkeypatch):
    """The largest K times the largest of a bit's products below 2^23: 128 (2-bit codes), 7 * 7 and 15 * 15."""
    lw, la = WIDE if bits == 2 else (range(1 << bits), range(1 << bits))
    lut = dg.dg_build_lut_bits(bits, list(lw), list(la), dg.DG_LUT_I16)
    name = lambda f, k: f(lut, dg.conv_desc(1, 1030, 1, k, 68, 1, 1, (1, 1), (0, 0)))
    monkeypatch.setenv("DG_PLANES", "2")
    assert name(dg.dg_conv_codes_kernel_name, K) == "codes_planes_64x64_k4" and not name(dg.dg_conv_codes_kernel_name, K + 64).startswith("codes_planes")
    if bits == 2:
        monkeypatch.setenv("DG_PLANES_PACKED", "1")
        assert name(dg.dg_conv_kernel_name, K) == "planes_64x128" and not name(dg.dg_conv_kernel_name, K + 64).startswith("planes")


def test_offsets_of_31_bits(monkeypatch):
    monkeypatch.setenv("DG_PLANES", "2")
    monkeypatch.setenv("DG_PLANES_PACKED", "1")
    for bits, (lw, la) in ((2, WIDE), (4, (range(16), range(16)))):
        lut = dg.dg_build_lut_bits(bits, list(lw), list(la), dg.DG_LUT_I16)
        for W, taken in ((1023, True), (1024, False)):       # 2^31 codes
            desc = dg.conv_desc(32, 1024, W, 64, 64, 1, 1, (1, 1), (0, 0))
            assert dg.dg_conv_codes_kernel_name(lut, desc).startswith("codes_planes") == taken, (bits, W)
            assert bits != 2 or (dg.dg_conv_kernel_name(lut, desc) == "planes_64x128") == taken, W


def test_two_bit_tables():
    """AUTO's own choices of tile; what is no product of levels, has an activation level 0 that is not 0, or fits int8 has other kernels."""
    lut = dg.dg_build_lut(*WIDE, dg.DG_LUT_I16)
    desc = lambda B, H, Cin, Cout, k: dg.conv_desc(B, H, H, Cin, Cout, k, k, (1, 1), (k // 2, k // 2))
    assert dg.dg_conv_codes_kernel_name(lut, desc(8, 28, 256, 256, 3)) == "codes_planes_64x128_k2"
    assert dg.dg_conv_codes_kernel_name(lut, desc(3, 28, 256, 256, 3)) == "codes_planes_64x64_k4"
    assert dg.dg_conv_kernel_name(lut, desc(16, 28, 256, 256, 3)) == "planes_64x128"
    for other in (dg.dg_build_lut(WIDE[0], (1, -128, 127, 0), dg.DG_LUT_I16), dg.dg_build_lut((-7, 5, -2, 3), (0, 7, -8, 5), dg.DG_LUT_I16),
                  dg.dg_build_lut_entries([0, 300, 600, 900, 0, 1, 2, 4, 0, 0, 0, 0, 0, 1, 1, 1], dg.DG_LUT_I16)):
        for d in (desc(8, 28, 256, 256, 3), desc(16, 28, 256, 256, 3)):
            assert "planes" not in dg.dg_conv_codes_kernel_name(other, d) and "planes" not in dg.dg_conv_kernel_name(other, d)
