"""3- and 4-bit tables that are the sum of two 2-bit lookups, run as 2-bit layers of twice the positions: every kernel form
that takes them, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2304_09049_amd import binding as dg
from paper_2304_09049_amd import workloads as wl

pytestmark = pytest.mark.gpu

# evenly spaced levels; a split whose high part fits int8 only after a shift; unevenly spaced levels that still split
TABLES = {(4, "uniform"): (list(range(-8, 8)), list(range(16))),
          (4, "shifted"): ([1] * 8 + [-1, 0] * 4, [-120 + 16 * a for a in range(16)]),
          (4, "uneven"): ([-3, 2, 1, 0, 5, -6, 4, 7, -7, 6, 3, -1, -2, -5, -4, 2], [g + f for g in (0, 9, -4, 3) for f in (1, 0, 5, 2)]),
          (3, "uniform"): (list(range(-4, 4)), list(range(1, 9))),
          # entries beyond int8 whose two halves fit it: -240 ... 210, -224 ... 168
          (4, "beyond"): (list(range(-8, 8)), list(range(0, 32, 2))),
          (3, "beyond"): (list(range(-32, 32, 8)), list(range(8)))}
ENTRY = {name: dg.DG_LUT_I16 if name[1] == "beyond" else dg.DG_LUT_I8 for name in TABLES}
PLANS = ["auto", "split", "1", "2", "4", "1k2", "2k4", "12", "12k2", "12k4", "14", "14k4", "16", "17", "24", "ws"]
STAGED = {"12": "32x64", "14": "32x128", "16": "32x192", "17": "32x224", "24": "64x128"}
TILED = {"1": "64x32", "2": "64x64", "4": "64x128"}


def _expected(plan, Cin, k, one_by_one):
    """The name of a forced plan's kernel; None: any that neither stages nor keeps its weights, the planner's choice.  Staged tiles
    need taps of whole 128-position runs of 2-bit codes (unshared 32 x 64 and 32 x 128: halves of one), stationary weights a
    layer without a window and K = 64, 128, 256 or 512 of them; a tile is shared by no more wavefronts than K has chunks."""
    c2, (tile, _, share) = 2 * Cin, plan.partition("k")
    if plan == "ws":
        return "ws_32xK" if one_by_one and c2 in (64, 128, 256, 512) else None
    if tile in STAGED:
        if c2 % 128 == 0 or (c2 % 64 == 0 and plan in ("12", "14")):
            return "staged_" + STAGED[tile] + ("_k" + share if share else "")
        return None
    chunks = k * k * c2 // (64 if c2 % 64 == 0 else 32)
    return TILED[tile] + ("_k" + share if share and int(share) <= chunks else "")


def _run(lut, bits, Wc, Xc, desc, scale=None):
    B, H, W, Cin = Xc.shape
    Cout = Wc.shape[0]
    Wp = dg.dg_pack_codes_bits(torch.from_numpy(Wc).cuda(), Cout, Wc.size // Cout, bits)
    Xp = dg.dg_pack_codes_bits(torch.from_numpy(Xc).cuda(), B * H * W, Cin, bits)
    y = dg.dg_conv2d_lut(lut, Wp, Xp, desc, scale=scale)
    torch.cuda.synchronize()
    return y.cpu().numpy(), Wp, Xp


@pytest.mark.parametrize("plan", PLANS)
@pytest.mark.parametrize("table", list(TABLES))
def test_nibble_tables(table, plan, monkeypatch):
    bits, (lw, la) = table[0], TABLES[table]
    lut = dg.dg_build_lut_bits(bits, lw, la, ENTRY[table])
    monkeypatch.setenv("DG_NIBBLES", "1")
    if plan != "auto":
        monkeypatch.setenv("DG_ONEHOT_PLAN", plan)
    rng = np.random.default_rng(len(plan) + bits)
    nlev = 1 << bits
    ran = 0
    for (B, H, W, Cin, Cout, k, stride, pad) in [(2, 9, 7, 16, 12, 3, (2, 1), (1, 1)), (1, 13, 11, 64, 40, 3, (1, 1), (1, 1)),
                                                 (2, 8, 9, 96, 68, 3, (1, 2), (1, 1)), (1, 17, 31, 128, 100, 1, (1, 1), (0, 0)),
                                                 (1, 40, 31, 32, 36, 1, (1, 1), (0, 0)), (1, 6, 5, 256, 33, 5, (1, 1), (2, 2))]:
        desc = dg.conv_desc(B, H, W, Cin, Cout, k, k, stride, pad)
        name = dg.dg_conv_kernel_name(lut, desc)
        if plan == "split":
            assert name.startswith("onehot_smfmac_4as2_splitk_s") or (k == 1 and Cin == 32), name      # (one chunk is not split)
            ran += "splitk" in name
        elif plan == "auto":
            assert name.startswith("onehot_smfmac_4as2_"), name
            ran += 1
        elif (want := _expected(plan, Cin, k, k == 1)) is not None:
            assert name == "onehot_smfmac_4as2_" + want, (name, Cin, k)
            ran += 1
        else:
            assert name.startswith("onehot_smfmac_4as2_") and "staged" not in name and "ws" not in name, (name, Cin, k)
        Wc, Xc = wl.draw_codes(rng, (Cout, k, k, Cin), nlev=nlev), wl.draw_codes(rng, (B, H, W, Cin), nlev=nlev)
        want = oracle.conv2d(Wc, Xc, lw, la, stride=stride, pad=pad)
        got, Wp, Xp = _run(lut, bits, Wc, Xc, desc)
        assert np.array_equal(got, want), (name, B, H, W, Cin, Cout, k)
        scale = rng.uniform(0.01, 0.1, size=Cout).astype(np.float32)
        y = oracle.scale_epilogue_nhwc(want, scale)
        got, Wp, Xp = _run(lut, bits, Wc, Xc, desc, torch.from_numpy(scale).cuda())
        assert np.array_equal(got, y), (name, "scaled")
        if Cout % 4 == 0 and ENTRY[table] == dg.DG_LUT_I16:
            with pytest.raises(dg.DgError) as e:             # (the fused layer takes tables of int8 entries)
                dg.dg_conv2d_lut_requant(lut, Wp, Xp, desc, torch.from_numpy(scale).cuda(), 1.0, 0.5, 0)
            assert e.value.status == 5
        elif Cout % 4 == 0:
            qs = float(np.float32(3.0 / max(1e-6, float(np.percentile(np.abs(y), 90)))))
            packed = dg.dg_conv2d_lut_requant(lut, Wp, Xp, desc, torch.from_numpy(scale).cuda(), qs, 0.5, 0)
            torch.cuda.synchronize()
            codes = oracle.quantize_codes(y, qs, 0.5, 0, 3)
            assert np.array_equal(packed.cpu().numpy().reshape(-1, Cout // 4), oracle.pack_codes(codes.reshape(-1, Cout))), (name, "requant")
    assert ran
    for M, N, K in ((33, 130, 64), (70, 300, 256), (5, 1000, 96)):
        Wc, Ac = wl.draw_codes(rng, (M, K), nlev=nlev), wl.draw_codes(rng, (N, K), nlev=nlev)
        Wp = dg.dg_pack_codes_bits(torch.from_numpy(Wc).cuda(), M, K, bits)
        Ap = dg.dg_pack_codes_bits(torch.from_numpy(Ac).cuda(), N, K, bits)
        want = oracle.gemm(Wc, Ac, lw, la)
        for strides, shape in (((1, M), (N, M)), ((N, 1), (M, N))):
            out = torch.full(shape, -7, dtype=torch.int32, device="cuda")
            dg.dg_gemm_lut(lut, Wp, Ap, M, N, K, out=out, strides=strides)      # (row-major only if the transposed table splits)
            torch.cuda.synchronize()
            assert np.array_equal(out.cpu().numpy(), want.T if strides[0] == 1 else want), (M, N, K, strides)


@pytest.mark.parametrize("bits", [3, 4])
@pytest.mark.parametrize("B,H,Cin,Cout,k,form", [(8, 56, 128, 100, 1, "ws_32xK"), (8, 28, 128, 72, 1, "ws_32xK"), (8, 28, 128, 128, 3, "staged_"),
                                                 (8, 56, 32, 40, 1, "ws_32xK"), (2, 28, 48, 72, 3, "splitk_s")])
def test_the_rule_takes_layers_with_partial_row_blocks(B, H, Cin, Cout, k, form, bits):
    """AUTO by itself, no override, at network sizes: the two lookups wherever the table splits, also where the last block of 32
    channels is partial."""
    lw, la = TABLES[(bits, "uniform")]
    lut = dg.dg_build_lut_bits(bits, lw, la, dg.DG_LUT_I8)
    desc = dg.conv_desc(B, H, H, Cin, Cout, k, k, (1, 1), (k // 2, k // 2))
    assert dg.dg_conv_kernel_name(lut, desc).startswith("onehot_smfmac_4as2_" + form), dg.dg_conv_kernel_name(lut, desc)
    rng = np.random.default_rng(Cout)
    Wc, Xc = wl.draw_codes(rng, (Cout, k, k, Cin), nlev=1 << bits), wl.draw_codes(rng, (B, H, H, Cin), nlev=1 << bits)
    got, _, _ = _run(lut, bits, Wc, Xc, desc)
    pos = np.unique(np.concatenate([rng.integers(0, got.size, 20000), np.arange(4 * Cout), got.size - 1 - np.arange(4 * Cout)]))
    want = oracle.conv2d_sampled(Wc, Xc, lw, la, pos, stride=(1, 1), pad=(k // 2, k // 2))
    assert np.array_equal(got.reshape(-1)[pos], want)


def test_wide_entries_that_do_not_split():
    """Entries beyond int8 whose table is no sum of two lookups, or of none that fit int8, stay with the plain kernel."""
    desc = dg.conv_desc(2, 14, 14, 64, 40, 3, 3, (1, 1), (1, 1))
    for bits, lw, la in ((4, list(range(-8, 6)) + [7, 6], list(range(0, 28, 2)) + [30, 28]), (4, list(range(-128, 128, 16)), list(range(16))),
                         (3, list(range(-4, 2)) + [3, 2], [100, 3, 5, 90, 1, 2, 127, 0])):
        lut = dg.dg_build_lut_bits(bits, lw, la, dg.DG_LUT_I16)
        assert dg.dg_conv_kernel_name(lut, desc) == "lds"
    # (activations 0 ... 15: the high parts of a weight level's row are up to 12 times the level apart, within int8 up to 21)
    rng = np.random.default_rng(9)
    for lw, la, name in ((list(range(-32, 32, 4)), list(range(16)), "lds"),
                         (list(range(-16, 16, 2)), list(range(16)), "onehot_smfmac_4as2_splitk_s")):
        lut = dg.dg_build_lut_bits(4, lw, la, dg.DG_LUT_I16)
        assert dg.dg_conv_kernel_name(lut, desc).startswith(name), dg.dg_conv_kernel_name(lut, desc)
        Wc, Xc = wl.draw_codes(rng, (40, 3, 3, 64), nlev=16), wl.draw_codes(rng, (2, 14, 14, 64), nlev=16)
        got, _, _ = _run(lut, 4, Wc, Xc, desc)
        assert np.array_equal(got, oracle.conv2d(Wc, Xc, lw, la, stride=(1, 1), pad=(1, 1)))


@pytest.mark.parametrize("table", ["uniform", "beyond"])
def test_raised_nibble_table(table, monkeypatch):
    """The staged kernel on the table raised to non-negative entries (its default on large problems only)."""
    bits, (lw, la) = 4, TABLES[(4, table)]
    lut = dg.dg_build_lut_bits(bits, lw, la, ENTRY[(4, table)])
    rng = np.random.default_rng(5)
    monkeypatch.setenv("DG_NIBBLES", "1")
    monkeypatch.setenv("DG_STAGED_BIAS", "1")
    Wc, Xc = wl.draw_codes(rng, (70, 3, 3, 64), nlev=16), wl.draw_codes(rng, (2, 11, 10, 64), nlev=16)
    want = oracle.conv2d(Wc, Xc, lw, la, stride=(1, 1), pad=(1, 1))
    for plan in ("12k4", "14", "24", "17"):
        monkeypatch.setenv("DG_ONEHOT_PLAN", plan)
        got, _, _ = _run(lut, bits, Wc, Xc, dg.conv_desc(2, 11, 10, 64, 70, 3, 3, (1, 1), (1, 1)))
        assert np.array_equal(got, want), plan
