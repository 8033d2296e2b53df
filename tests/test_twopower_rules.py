"""Which calls AUTO takes to the kernel for products of levels: its names for tables of each form and on both sides of the sizes (256 compute
units, as without a device)."""
import itertools

import pytest

from paper_2304_09049_amd import binding as dg

LEVELS = ((-7, 5, -2, 3), (7, -8, 0, 5))
BIG = (8192, 8192, 8192)


@pytest.fixture(autouse=True)
def no_overrides(monkeypatch):
    for name in ("DG_ONEBIT", "DG_TWOPOWER", "DG_ONEHOT_PLAN", "DG_ONEHOT_WAVES"):
        monkeypatch.delenv(name, raising=False)


def gemm(M, N, K, lw=LEVELS[0], la=LEVELS[1], variant="auto"):
    return dg.dg_gemm_kernel_name(dg.dg_build_lut(lw, la, dg.DG_LUT_I16), M, N, K, variant)


def test_tables():
    """Every pair of levels from -8 to 7 is of the form (activation levels evenly spaced from zero have other kernels); by entries too."""
    size = (2048, 4096, 2048)
    for x in itertools.product(range(-8, 8), repeat=2):
        lw, la = (x[0], 7, -8, 5), (x[1], 5, 7, -3)
        assert gemm(*size, lw=lw, la=la).startswith("twopower_"), (lw, la)
    for lw, la in (((15, -13, 11, 1), (-2, -1, 0, 1)), ((12, -12, 6, 9), (4, 5, 6, 7)), ((0, 0, 0, 5), (9, -9, 10, 1)), ((3, 3, 3, 3), (0, 0, 0, 1))):
        assert gemm(*size, lw=lw, la=la).startswith("twopower_"), (lw, la)
    entries = [w * a for w in LEVELS[0] for a in LEVELS[1]]
    assert dg.dg_gemm_kernel_name(dg.dg_build_lut_entries(entries), *size).startswith("twopower_")
    entries[5] += 1                                         # no product of levels
    assert dg.dg_gemm_kernel_name(dg.dg_build_lut_entries(entries), *size).startswith("onehot_")
    for lw, la in (((17, 1, 0, 2), (-1, 0, 1, 4)), ((1, 2, 3, 4), (11, 1, 2, 0)), ((1, 2, 3, 4), (13, 1, -2, 0)), ((-2, 5, 0, 1), (0, 1, 2, 3)),
                   ((-100, 7, 3, 1), (1, 2, 0, -1))):      # numbers that FP6 and two powers have not; evenly spaced; entries beyond int8
        assert gemm(*size, lw=lw, la=la).startswith("onehot_"), (lw, la)
    assert gemm(*size, lw=(-2, -1, 0, 1), la=(0, 1, 2, 3)).startswith("onebit_")


def test_sizes_and_shapes():
    assert gemm(*BIG) == "twopower_128x512" and gemm(4872, 7116, 4672) == "twopower_128x256"
    assert gemm(1305, 1621, 1856) == "twopower_64x128" and gemm(2275, 903, 4544) == "twopower_64x128_k2"
    assert gemm(8192, 256, 8192) == "onehot_smfmac_staged_32x128_k4"                 # long K, few tiles
    assert gemm(1305, 1621, 1856 + 32).startswith("onehot_") and gemm(1305, 300, 1856).startswith("onehot_")         # K % 64; 1.45e9 operations
    assert gemm(304, 561, 4224).startswith("onehot_mfma_splitk")
    assert gemm(6000, 6000, 256) == "onehot_smfmac_ws_32xK"
    assert gemm(*BIG, variant="onehot_smfmac").startswith("onehot_smfmac_") and gemm(*BIG, variant="onehot_mfma").startswith("onehot_mfma_")
    lut = dg.dg_build_lut(*LEVELS)
    name = lambda k, s, p: dg.dg_conv_kernel_name(lut, dg.conv_desc(8, 56, 56, 704, 704, k, k, (s, s), (p, p)))
    assert name(1, 1, 0).startswith("twopower_") and not any(name(*x).startswith("twopower_") for x in ((3, 1, 1), (1, 2, 0), (1, 1, 1)))


def test_short_sums_on_large_outputs():
    """Below K = 640 the tiles of 128 x 256 measured up to 26 % behind the one-hot kernels, and those of 64 x 128 ahead of both."""
    for size in ((3889, 20227, 384), (6977, 7871, 384), (2269, 32266, 384), (5159, 9628, 576), (2274, 30161, 320)):
        assert gemm(*size) == "twopower_64x128", size
    assert gemm(5159, 9628, 640) == "twopower_128x256"


def test_the_end_of_the_range():
    """7 * 9 * K below 2^24 (7 is 8 - 1)."""
    assert gemm(2048, 4096, 266240, lw=(-7, 1, 3, 7), la=(-1, 1, 2, 7)).startswith("twopower_")
    assert gemm(2048, 4096, 266368, lw=(-7, 1, 3, 7), la=(-1, 1, 2, 7)).startswith("onehot_")


@pytest.mark.parametrize("value", ["0", "3", "-1", "", "1x"])
def test_override_values(value, monkeypatch):
    monkeypatch.setenv("DG_TWOPOWER", value)
    assert gemm(*BIG).startswith("onehot_" if value == "0" else "twopower_128x512")


def test_offsets_of_31_bits(monkeypatch):
    """2^31 bytes of packed codes."""
    monkeypatch.setenv("DG_TWOPOWER", "1")
    assert gemm(64, 26843545, 320) == "twopower_64x128" and not gemm(64, 26843546, 320).startswith("twopower")
