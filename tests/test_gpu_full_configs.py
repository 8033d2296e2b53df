"""GPU parity at the full benchmark sizes, in the launch configuration bench.py times (variant "auto"),
plus every other variant that accepts the shape.  Where the oracle finishes in seconds the whole output
is compared; otherwise a seeded sample of outputs (borders included) is computed one by one by the oracle."""
import numpy as np
import pytest

import oracle
from paper_2304_09049_amd import workloads as wl
from gpu_helpers import GpuCase, run_or_unsupported

pytestmark = pytest.mark.gpu

VARIANTS = ["auto", "perm", "lds", "mfma_i8", "smalln", "lut65k", "onehot_mfma", "onehot_smfmac"]
# every output compared, except on the 8192-cube GEMM (550 G multiply-adds for the oracle): there a seeded sample of
# more than 1 % of the 67 M outputs, with the first and last rows and columns (the last tiles of either axis) added
FULL = ["gemm_64x196x576", "resnet18_conv3x3_b1", "resnet50_conv1x1_b32", "vgg16_conv3x3_b16", "gemm_8192x1x8192_i16",
        "gemm_8192x16x8192_i16", "gemm_8192x256x8192_i16"]
SAMPLED = ["gemm_8192x8192x8192_i16"]
SAMPLE_FRACTION = 0.0105


def _border_heavy_positions(w, rng, count):
    """Flat NHWC output indices: a uniform sample plus every corner / some edge pixels of a few images."""
    total = w.N * w.M
    pos = [rng.integers(0, total, size=count)]
    if w.kind == "gemm":
        # output [M][N]: a sample of the first and last two rows and columns, and the four corner 40 x 40 blocks whole
        for m in (0, 1, w.M - 2, w.M - 1):
            pos.append(m * w.N + rng.integers(0, w.N, size=512))
        for n in (0, 1, w.N - 2, w.N - 1):
            pos.append(rng.integers(0, w.M, size=512) * w.N + n)
        edge = np.arange(40)
        for ms in (edge, w.M - 1 - edge):
            for ns in (edge, w.N - 1 - edge):
                pos.append((ms[:, None] * w.N + ns[None, :]).reshape(-1))
    if w.kind == "conv":
        OH = (w.H + 2 * w.pad[0] - w.KH) // w.stride[0] + 1
        OW = (w.W + 2 * w.pad[1] - w.KW) // w.stride[1] + 1
        for b in (0, w.B - 1):
            for oh in (0, 1, OH - 2, OH - 1):
                for ow in (0, 1, OW - 2, OW - 1):
                    px = (b * OH + oh) * OW + ow
                    pos.append(px * w.M + rng.integers(0, w.M, size=8))
    return np.unique(np.concatenate(pos))


def _one_call(case, inp):
    """The step bench.py times: dg_conv2d_lut_codes / dg_gemm_lut_codes on the unpacked codes (AUTO), with a work buffer
    for the problems whose packing is not fused into the kernel."""
    import torch
    from paper_2304_09049_amd import binding as dg
    Xc = torch.from_numpy(inp.Ac).cuda()
    w = inp.workload
    if w.kind == "conv":
        got = dg.dg_conv2d_lut_codes(case.lut, case.Wp, Xc, case.desc, work=torch.empty_like(case.Ap))
    else:
        got = dg.dg_gemm_lut_codes(case.lut, case.Wp, Xc, w.M, w.N, w.K, work=torch.empty_like(case.Ap))
    torch.cuda.synchronize()
    return got.cpu().numpy()


@pytest.mark.parametrize("name", FULL)
def test_full_output(name):
    w = wl.CONFIGS[name]
    inp = wl.make_inputs(w)
    case = GpuCase(inp)
    if w.kind == "conv":
        want = oracle.conv2d(inp.Wc, inp.Ac, inp.levels_w, inp.levels_a, stride=w.stride, pad=w.pad)
    else:
        want = oracle.gemm(inp.Wc, inp.Ac, inp.levels_w, inp.levels_a)
    ran = []
    for variant in VARIANTS:
        got = run_or_unsupported(case, variant)
        if got is None:
            continue
        ran.append(variant)
        assert np.array_equal(got, want), f"{name} {variant}: {np.count_nonzero(got != want)} outputs differ"
    assert "auto" in ran and "lds" in ran
    assert np.array_equal(_one_call(case, inp), want), f"{name}: packing + convolution / GEMM as one call"
    if w.scale:
        got = case.run("auto", scale=True).cpu().numpy()
        ref = oracle.scale_epilogue_nhwc(want, inp.scale)
        np.testing.assert_allclose(got, ref, rtol=1e-6, atol=0)


@pytest.mark.parametrize("name", SAMPLED)
def test_sampled_output(name):
    w = wl.CONFIGS[name]
    inp = wl.make_inputs(w)
    case = GpuCase(inp)
    rng = np.random.default_rng(123)
    count = int(np.ceil(SAMPLE_FRACTION * w.M * w.N))      # (8192-cube: 704 644 outputs, 5.8 G multiply-adds for the oracle)
    pos = _border_heavy_positions(w, rng, count)
    assert len(pos) >= 0.01 * w.M * w.N
    if w.kind == "conv":
        want = oracle.conv2d_sampled(inp.Wc, inp.Ac, inp.levels_w, inp.levels_a, pos, stride=w.stride, pad=w.pad)
    else:
        ms, ns = pos // w.N, pos % w.N            # GEMM output is [M][N]
        want = oracle.gemm_sampled(inp.Wc, inp.Ac, inp.levels_w, inp.levels_a, ms, ns)
    ran = []
    for variant in VARIANTS:
        if variant in ("lds", "lut65k") and w.ops > 2e11:
            continue                               # the plain kernels would take too long at this size
        got = run_or_unsupported(case, variant)
        if got is None:
            continue
        ran.append(variant)
        flat = got.reshape(-1)[pos]
        assert np.array_equal(flat, want), f"{name} {variant}: {np.count_nonzero(flat != want)} sampled outputs differ"
    assert "auto" in ran
    assert np.array_equal(_one_call(case, inp).reshape(-1)[pos], want), f"{name}: packing + convolution / GEMM as one call"


TWO_PLANES = [("vgg16_conv3x3_b16", "onehot_smfmac_2p_staged_32x128"), ("gemm_8192x8192x8192_i16", "onehot_smfmac_2p_staged_32x128"),
              ((16, 56, 96, 96, 3, 1), "onehot_smfmac_2p_32x128"),               # taps of no whole runs: direct loads
              ((8, 28, 256, 256, 3, 1), "onehot_smfmac_2p_staged_32x128_k4"), ((16, 28, 256, 256, 3, 1), "onehot_smfmac_2p_staged_32x128_k2"),
              ((8, 14, 256, 256, 3, 1), "onehot_smfmac_2p_staged_32x64_k4"), ((16, 56, 64, 64, 3, 1), "onehot_smfmac_2p_staged_32x64")]


@pytest.mark.parametrize("name,kernel", TWO_PLANES)
def test_sampled_output_two_plane_table(name, kernel):
    """The same full-size shapes, and a network layer for each other form, under a table with entries beyond int8 (levels up
    to +-127, no zero activation level): AUTO's sparse-instruction two-plane kernels and the dense-instruction one, against
    sampled oracle outputs."""
    from paper_2304_09049_amd import binding as dg
    if isinstance(name, str):
        w = wl.CONFIGS[name]
    else:
        B, H, Cin, Cout, k, s = name
        w = wl._conv("layer", B, H, H, Cin, Cout, k, k, (s, s), (k // 2, k // 2))
    inp = wl.make_inputs(w)
    lw, la = (127, -128, 5, 3), (-128, 127, 1, 2)
    case = GpuCase(inp, levels=(lw, la), entry=dg.DG_LUT_I16)
    assert case.kernel_name("auto") == kernel
    assert case.kernel_name("onehot_mfma").startswith("onehot_mfma_2p_")
    rng = np.random.default_rng(321)
    pos = _border_heavy_positions(w, rng, int(min(200000, 3e9 // w.K)))
    if w.kind == "conv":
        want = oracle.conv2d_sampled(inp.Wc, inp.Ac, lw, la, pos, stride=w.stride, pad=w.pad)
    else:
        want = oracle.gemm_sampled(inp.Wc, inp.Ac, lw, la, pos // w.N, pos % w.N)
    for variant in ("auto", "onehot_mfma"):
        flat = case.run(variant).cpu().numpy().reshape(-1)[pos]
        assert np.array_equal(flat, want), f"{name} {variant}: {np.count_nonzero(flat != want)} sampled outputs differ"


NOT_ONE_BIT = (-2, 5, 0, 1)       # weight levels that FP4 has not all of (2:5 is no ratio of its numbers): tables of the general form
NETWORK_LAYERS = [
    # (B, H, Cin, Cout, filter, stride), AUTO's kernel on packed codes, the one-call step's kernel, weight levels (None: the layer's own)
    ((32, 28, 320, 320, 3, 1), "onehot_smfmac_staged_32x128", "onehot_smfmac_staged_32x128", NOT_ONE_BIT),       # taps of 2.5 runs
    ((32, 56, 256, 256, 3, 1), "onehot_smfmac_staged_32x224", "onehot_smfmac_staged_32x224", NOT_ONE_BIT),
    ((32, 56, 256, 512, 1, 2), "onehot_smfmac_ws_32xK", "onehot_smfmac_ws_32xK", None),             # strided; the step packs the pixels read
    ((32, 28, 512, 512, 1, 1), "onehot_smfmac_ws_32xK", "onehot_smfmac_ws_32xK", None),             # K = 512
    ((8, 14, 1024, 256, 1, 1), "onehot_smfmac_staged_32x64_k4", "codes_onehot_smfmac_64x32_k4", None),    # the tiled kernel packs
    ((1, 56, 256, 64, 1, 1), "onehot_mfma_splitk_s4", "codes_onehot_mfma_splitk_s4", None),         # 64-position chunks
    ((8, 7, 512, 512, 3, 1), "onehot_mfma_splitk_s12", "onehot_mfma_splitk_s12", None),
    # tables that are two one-bit lookups, every tile
    ((32, 28, 128, 128, 3, 1), "onebit_64x128", "onebit_64x128", None),
    ((8, 28, 256, 256, 3, 1), "onebit_64x128_k2", "onebit_64x128_k2", None),
    ((32, 28, 320, 320, 3, 1), "onebit_64x256", "onebit_64x256", None),
    ((32, 56, 256, 256, 3, 1), "onebit_64x256_64x128", "onebit_64x256_64x128", None),
    ((16, 64, 256, 256, 3, 1), "onebit_64x512", "onebit_64x512", None),
    ((25, 56, 64, 40, 3, 2), "onehot_mfma_64x32", "codes_onebit_64x128", None),                     # it packs while loading
    ((25, 56, 64, 40, 3, 2), "onehot_mfma_64x32", "codes_onehot_smfmac_64x32", NOT_ONE_BIT),
]


@pytest.mark.parametrize("shape,kernel,step_kernel,levels_w", NETWORK_LAYERS)
def test_sampled_output_network_layers(shape, kernel, step_kernel, levels_w):
    """Full-size layers of the networks bench.py --layers times, one per kernel and rule that the small parity cases
    reach only through forced plans: AUTO's kernel on packed codes and the one-call step on unpacked codes, against
    sampled oracle outputs (borders included)."""
    from paper_2304_09049_amd import binding as dg
    B, H, Cin, Cout, k, s = shape
    w = wl._conv("layer", B, H, H, Cin, Cout, k, k, (s, s), (k // 2, k // 2))
    inp = wl.make_inputs(w)
    lw, la = inp.levels_w if levels_w is None else levels_w, inp.levels_a
    case = GpuCase(inp, levels=(lw, la))
    assert case.kernel_name("auto") == kernel
    assert dg.dg_conv_codes_kernel_name(case.lut, case.desc, "auto") == step_kernel
    rng = np.random.default_rng(B + H + Cin + Cout)
    pos = _border_heavy_positions(w, rng, int(min(60000, 2e8 // w.K)))
    want = oracle.conv2d_sampled(inp.Wc, inp.Ac, lw, la, pos, stride=w.stride, pad=w.pad)
    got = case.run("auto").cpu().numpy().reshape(-1)[pos]
    assert np.array_equal(got, want), f"{shape} {kernel}: {np.count_nonzero(got != want)} sampled outputs differ"
    got = _one_call(case, inp).reshape(-1)[pos]
    assert np.array_equal(got, want), f"{shape} {step_kernel}: {np.count_nonzero(got != want)} sampled outputs differ (one call)"


RAGGED_LAYERS = [
    # (B, H, W, Cin, Cout, filter, stride), AUTO's kernel on packed codes, the one-call step's kernel
    ((8, 29, 27, 48, 120, 5, 1), "onehot_smfmac_ragged_32x32", "codes_onehot_smfmac_ragged_64x32"),
    ((16, 28, 28, 112, 224, 3, 1), "onehot_smfmac_ragged_32x32", "onehot_smfmac_ragged_32x32"),        # unshared tiles
    ((16, 14, 14, 208, 48, 5, 1), "onehot_smfmac_ragged_32x32", "onehot_smfmac_ragged_32x32"),         # shared by 12
    ((4, 57, 57, 36, 128, 3, 1), "onehot_smfmac_ragged_32x32", "onehot_smfmac_ragged_32x32"),
    ((16, 56, 56, 20, 128, 1, 1), "onehot_smfmac_ragged_32x32", "codes_onehot_smfmac_ragged_64x64"),
    ((1, 56, 56, 16, 32, 3, 1), "onehot_smfmac_ragged_32x32", "codes_onehot_smfmac_ragged_32x32"),
    ((32, 28, 28, 80, 96, 1, 2), "onehot_smfmac_ragged_32x32", "onehot_smfmac_ragged_32x32"),          # strided; the step packs the pixels read
]


@pytest.mark.parametrize("shape,kernel,step_kernel", RAGGED_LAYERS)
def test_sampled_output_ragged_channel_layers(shape, kernel, step_kernel):
    """Channel counts that are no multiple of 32 at full size, in the plans AUTO makes by itself: packed and from codes, against
    sampled oracle outputs (borders included)."""
    from paper_2304_09049_amd import binding as dg
    B, H, W, Cin, Cout, k, s = shape
    w = wl._conv("layer", B, H, W, Cin, Cout, k, k, (s, s), (k // 2, k // 2))
    inp = wl.make_inputs(w)
    case = GpuCase(inp)
    assert case.kernel_name("auto") == kernel
    assert dg.dg_conv_codes_kernel_name(case.lut, case.desc, "auto") == step_kernel
    rng = np.random.default_rng(B + H + Cin + Cout)
    pos = _border_heavy_positions(w, rng, int(min(60000, 2e8 // w.K)))
    want = oracle.conv2d_sampled(inp.Wc, inp.Ac, inp.levels_w, inp.levels_a, pos, stride=w.stride, pad=w.pad)
    got = case.run("auto").cpu().numpy().reshape(-1)[pos]
    assert np.array_equal(got, want), f"{shape} {kernel}: {np.count_nonzero(got != want)} sampled outputs differ"
    got = _one_call(case, inp).reshape(-1)[pos]
    assert np.array_equal(got, want), f"{shape} {step_kernel}: {np.count_nonzero(got != want)} sampled outputs differ (one call)"


@pytest.mark.parametrize("shape", [(4, 28, 28, 128, 128, 3), (8, 56, 56, 64, 64, 1), (8, 14, 14, 36, 100, 3), (2, 56, 56, 96, 72, 1)])
def test_full_output_binary32_table(shape):
    """Binary32 tables on layers that AUTO takes to the matrix cores by itself: every output, scaled and not, bit for bit."""
    import torch
    from paper_2304_09049_amd import binding as dg
    B, H, W, Cin, Cout, k = shape
    lw, la = np.array([-1.27, -0.32, 0.3217, 1.19], np.float32), np.array([0.05, 0.451, 0.98, 1.78], np.float32)
    lut, table = dg.dg_build_lut_f32(lw, la), oracle.build_lut_f32(lw, la)
    c = wl.small_conv(B, H, W, Cin, Cout, k, k, (1, 1), (k // 2, k // 2), seed=Cin, scale=True)
    desc = dg.conv_desc(B, H, W, Cin, Cout, k, k, (1, 1), (k // 2, k // 2))
    assert dg.dg_conv_kernel_name(lut, desc) == "onehot_mfma_f32"
    Xc, scale = torch.from_numpy(c.Ac).cuda(), torch.from_numpy(c.scale).cuda()
    Wp = dg.dg_pack_weights(torch.from_numpy(c.Wc).cuda(), Cout, k * k * Cin)
    Xp = dg.dg_pack_activations(Xc, B * H * W, Cin)
    want = oracle.conv2d_table_f32(c.Wc, c.Ac, table, stride=(1, 1), pad=(k // 2, k // 2))
    assert np.array_equal(dg.dg_conv2d_lut(lut, Wp, Xp, desc).cpu().numpy(), want)
    got = dg.dg_conv2d_lut_codes(lut, Wp, Xc, desc, work=torch.empty_like(Xp), scale=scale).cpu().numpy()
    assert np.array_equal(got, want * c.scale[None, None, None, :])


@pytest.mark.parametrize("bits,shape,kernel", [(4, (8, 28, 128, 128, 3), "onehot_smfmac_4as2_staged_32x64_k4"),
                                               (4, (16, 56, 256, 256, 3), "onehot_smfmac_4as2_staged_32x224"),
                                               (3, (8, 28, 128, 512, 1), "onehot_smfmac_4as2_ws_32xK"),
                                               (3, (2, 14, 128, 200, 3), "onehot_smfmac_4as2_splitk_s"),
                                               (4, (16, 56, 80, 128, 3), "onehot_smfmac_4as2_64x64")])
def test_sampled_output_two_lookups(bits, shape, kernel):
    """3- and 4-bit codes as two 2-bit lookups at full size, in AUTO's plans: packed and from codes, against sampled outputs."""
    import torch
    from paper_2304_09049_amd import binding as dg
    B, H, Cin, Cout, k = shape
    lw, la = list(range(-(1 << bits) // 2, (1 << bits) // 2)), list(range(1, (1 << bits) + 1)) if bits == 3 else list(range(16))
    lut = dg.dg_build_lut_bits(bits, lw, la, dg.DG_LUT_I8)
    desc = dg.conv_desc(B, H, H, Cin, Cout, k, k, (1, 1), (k // 2, k // 2))
    name = dg.dg_conv_kernel_name(lut, desc)
    assert name.startswith(kernel), name
    rng = np.random.default_rng(Cin + Cout)
    Wc, Xc = wl.draw_codes(rng, (Cout, k, k, Cin), nlev=1 << bits), wl.draw_codes(rng, (B, H, H, Cin), nlev=1 << bits)
    w = wl._conv("layer", B, H, H, Cin, Cout, k, k, (1, 1), (k // 2, k // 2))
    pos = _border_heavy_positions(w, rng, int(min(60000, 2e8 // w.K)))
    want = oracle.conv2d_sampled(Wc, Xc, lw, la, pos, stride=(1, 1), pad=(k // 2, k // 2))
    codes = torch.from_numpy(Xc).cuda()
    Wp = dg.dg_pack_codes_bits(torch.from_numpy(Wc).cuda(), Cout, k * k * Cin, bits)
    Xp = dg.dg_pack_codes_bits(codes, B * H * H, Cin, bits)
    assert np.array_equal(dg.dg_conv2d_lut(lut, Wp, Xp, desc).cpu().numpy().reshape(-1)[pos], want)
    got = dg.dg_conv2d_lut_codes(lut, Wp, codes, desc, work=torch.empty_like(Xp)).cpu().numpy()
    assert np.array_equal(got.reshape(-1)[pos], want)
