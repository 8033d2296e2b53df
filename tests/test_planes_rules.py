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
                                        (4, (8, 28, 28, 64, 780, 1, 2)), (3, (734, 1, 1, 64, 424, 1))])
def test_short_sums_of_few_blocks_are_packed_first(bits, layer):
    """Layers that measured 3 to 25 % longer by the codes' bits."""
    packed, codes = names(bits, *layer)
    assert packed.startswith("onehot_smfmac_4as2_") and codes == packed


@pytest.mark.parametrize("bits,layer,kernel", [(4, (8, 28, 28, 128, 128, 3), "codes_planes_64x64_k4"), (3, (8, 28, 28, 128, 128, 3), "codes_planes_64x64_k4"),
                                               (3, (5, 112, 112, 128, 112, 3, 2), "codes_planes_64x128_k2")])
def test_layers_by_their_bits(bits, layer, kernel):
    packed, codes = names(bits, *layer)
    assert packed.startswith("onehot_smfmac_4as2_") and codes == kernel
