"""The native marshalling module's checks, and the planner's memo (neither needs a GPU)."""
import os
import subprocess
import sys

import numpy as np
import pytest
import torch

from paper_2304_09049_amd import binding as dg

SHAPES = """
import random, sys
from paper_2304_09049_amd import binding as dg
lut = dg.dg_build_lut((-2, -1, 0, 1), (0, 1, 2, 3))
wide = dg.dg_build_lut((-128, -1, 0, 1), (0, 1, 2, 127), dg.DG_LUT_I16)
rng = random.Random(7)
shapes = [(rng.choice((1, 8, 32)), s, s, 32 * rng.randint(1, 16), 8 * rng.randint(1, 64), k, k, (1, 1), (k // 2, k // 2))
          for s in (7, 14, 28, 56) for k in (1, 3) for _ in range(20)]
t3, t4 = (dg.dg_build_lut_bits(b, list(range(-(1 << b) // 2, (1 << b) // 2)), list(range(1 << b))) for b in (3, 4))
uneven = dg.dg_build_lut_bits(4, list(range(-8, 6)) + [7, 6], list(range(14)) + [15, 14])
for _ in range(2):                                   # 160 shapes, so that the second time round finds some plans kept and most replaced
    for s in shapes:
        for t in (lut, wide, t3, t4, uneven):
            d = dg.conv_desc(*s)
            print(dg.dg_conv_kernel_name(t, d), dg.dg_conv_codes_kernel_name(t, d), dg.dg_conv_kernel_name(t, d, "onehot_mfma"),
                  dg.dg_gemm_kernel_name(t, s[4], s[0] * s[1] * s[2], s[3]))
"""

# Small problems of every code width, one and two planes, GEMMs and convolutions, each three times in another order: most of their
# plans are replaced between two of its calls.  The outputs of all three are the oracle's.
PARITY = """
import random, sys
import numpy as np, torch
import oracle
from paper_2304_09049_amd import binding as dg
from paper_2304_09049_amd import workloads as wl
rng, gen = random.Random(11), np.random.default_rng(11)
levels = {2: ((-2, -1, 0, 1), (0, 1, 2, 3)), 22: ((-128, -1, 5, 127), (1, -3, 127, 2)), 3: (list(range(-4, 4)), list(range(1, 9))),
          4: (list(range(-8, 8)), list(range(16))), 44: (list(range(-8, 6)) + [7, 6], list(range(14)) + [15, 14])}
tables = {k: dg.dg_build_lut_bits(k % 10, list(w), list(a), dg.DG_LUT_I16) for k, (w, a) in levels.items()}
calls = []
for i in range(150):
    kind = rng.choice(list(levels))
    bits, (lw, la), lut = kind % 10, levels[kind], tables[kind]
    cin, cout = 32 * rng.randint(1, 8), rng.randint(1, 100)
    if i % 3:
        k, H, W, B = rng.choice((1, 3)), rng.randint(3, 12), rng.randint(3, 12), rng.randint(1, 3)
        w, x = wl.draw_codes(gen, (cout, k, k, cin), nlev=1 << bits), wl.draw_codes(gen, (B, H, W, cin), nlev=1 << bits)
        want = oracle.conv2d(w, x, lw, la, stride=(1, 1), pad=(k // 2, k // 2))
        desc, rows, K = dg.conv_desc(B, H, W, cin, cout, k, k, (1, 1), (k // 2, k // 2)), B * H * W, k * k * cin
    else:
        rows, K = rng.randint(1, 300), cin
        w, x = wl.draw_codes(gen, (cout, K), nlev=1 << bits), wl.draw_codes(gen, (rows, K), nlev=1 << bits)
        want, desc = oracle.gemm(w, x, lw, la), None
    pack = lambda c, r, n: dg.dg_pack_codes_bits(torch.from_numpy(c).cuda(), r, n, bits)
    calls.append((lut, desc, pack(w, cout, K), pack(x, rows, cin), torch.from_numpy(x).cuda(), cout, rows, K, want))
for time in range(3):
    for (lut, desc, wp, xp, codes, cout, rows, K, want) in rng.sample(calls, len(calls)):
        work = torch.empty_like(xp)
        if desc is not None:
            got = dg.dg_conv2d_lut(lut, wp, xp, desc), dg.dg_conv2d_lut_codes(lut, wp, codes, desc, work=work)
        else:
            got = dg.dg_gemm_lut(lut, wp, xp, cout, rows, K), dg.dg_gemm_lut_codes(lut, wp, codes, cout, rows, K, work=work)
        for g in got:
            assert np.array_equal(g.cpu().numpy(), want), (lut.bits, cout, rows, K)
print("the oracle's")
"""


def _names(overrides):
    env = {k: v for k, v in os.environ.items() if not k.startswith("DG_")}
    env["DG_TEST_OVERRIDES"] = overrides             # "1": every plan is made anew
    out = subprocess.run([sys.executable, "-c", SHAPES], env=env, capture_output=True, text=True, check=True,
                         cwd=os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
    return out.stdout.splitlines()


def test_remembered_plans_are_the_plans():
    fresh, kept = _names("1"), _names("0")
    assert len(fresh) == 1600 and fresh[:800] == fresh[800:]
    assert kept == fresh


@pytest.mark.gpu
def test_remembered_plans_give_the_oracles_outputs():
    """(In a process of its own, as the other tests run with overrides, under which no plan is remembered.)"""
    env = {k: v for k, v in os.environ.items() if not k.startswith("DG_")}
    out = subprocess.run([sys.executable, "-c", PARITY], env=env, capture_output=True, text=True,
                         cwd=os.path.dirname(os.path.dirname(os.path.abspath(__file__))), timeout=100)
    assert out.returncode == 0 and out.stdout == "the oracle's\n", out.stderr[-2000:]


def test_native_checks():
    lut = dg.dg_build_lut((-2, -1, 0, 1), (0, 1, 2, 3))
    host = torch.zeros(64, dtype=torch.uint8)
    desc = dg.conv_desc(1, 2, 2, 16, 4, 1, 1)
    for call in (lambda: dg.dg_pack_activations(host, 4, 16, out=host), lambda: dg.dg_pack_weights(host, 4, 16, out=host),
                 lambda: dg.dg_pack_codes_bits(host, 4, 16, 3, out=host), lambda: dg.dg_dequantize(host, 4, 16, host, out=host),
                 lambda: dg.dg_quantize_pack_activations(host, 4, 16, 1.0, 0.0, 0, out=host),
                 lambda: dg.dg_gemm_lut(lut, host, host, 4, 4, 16, out=host),
                 lambda: dg.dg_gemm_lut_codes(lut, host, host, 4, 4, 16, out=host),
                 lambda: dg.dg_conv2d_lut(lut, host, host, desc, out=host),
                 lambda: dg.dg_conv2d_lut_codes(lut, host, host, desc, out=host),
                 lambda: dg.dg_conv2d_lut_codes_static(lut, host, host, desc, host),
                 lambda: dg.dg_conv2d_lut_requant(lut, host, host, desc, host, 1.0, 0.0, 0, out=host)):
        with pytest.raises(ValueError, match="must live in device memory"):
            call()
    with pytest.raises(TypeError, match="must be a tensor"):
        dg.dg_pack_activations([1, 2], 4, 16, out=host)


BAD_TABLES = """
from paper_2304_09049_amd import binding as dg
native = dg._load_native()
class Stream:
    cuda_stream = 0
for table, error in ((-1, OverflowError), (1 << 70, OverflowError), ("table", TypeError), (None, TypeError)):
    for call in (lambda: native.gemm_lut(table, False, None, None, 1, 1, 16, None, 1, 1, None, 0, Stream),
                 lambda: native.gemm_lut_codes(table, False, None, None, 1, 1, 16, None, None, 1, 1, None, 0, Stream),
                 lambda: native.conv2d_lut(table, False, None, None, dg.conv_desc(1, 2, 2, 16, 4, 1, 1), None, None, 0, Stream),
                 lambda: native.conv2d_lut_codes(table, False, None, None, dg.conv_desc(1, 2, 2, 16, 4, 1, 1), None, None, None, 0, Stream),
                 lambda: native.conv2d_lut_codes_static(table, False, None, None, dg.conv_desc(1, 2, 2, 16, 4, 1, 1), None, None, 0, Stream),
                 lambda: native.conv2d_lut_requant(table, None, None, dg.conv_desc(1, 2, 2, 16, 4, 1, 1), None, 1.0, 0.0, 0, None, 0, Stream)):
        try:
            call()
        except error:
            continue
        raise SystemExit(f"{table!r} was taken for a table")
print("refused")
"""


def test_bad_table_addresses_raise():
    """A table that is no address is refused while the interpreter lock is held (in a process of its own: it ended there)."""
    out = subprocess.run([sys.executable, "-c", BAD_TABLES], capture_output=True, text=True,
                         cwd=os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
    assert out.returncode == 0 and out.stdout == "refused\n", (out.returncode, out.stderr[-2000:])


class StandIn:
    """No tensor, but it answers as a contiguous one on the GPU does.  (Its address is made up: nothing is launched.)"""

    def __init__(self, dtype=torch.uint8, count=1 << 20, is_cuda=True, contiguous=True):
        self.dtype, self.count, self.is_cuda, self.contiguous, self.device = dtype, count, is_cuda, contiguous, None

    def is_contiguous(self):
        return self.contiguous

    def data_ptr(self):
        return 0x1000

    def numel(self):
        return self.count


class Stream:
    cuda_stream = 0


def _refused(call, status):
    with pytest.raises(dg.DgError) as e:
        call()
    assert e.value.status == status


def test_objects_that_answer_as_tensors_and_tables():
    """Operands, tables and flags of other types than torch's and this package's own reach the library (which refuses these
    calls by their shape, 2, or their buffer's size, 4)."""
    x, f, i = StandIn(), StandIn(torch.float32), StandIn(torch.int32)
    lut = dg.dg_build_lut((-2, -1, 0, 1), (0, 1, 2, 3))
    desc = dg.conv_desc(1, 2, 2, 15, 4, 1, 1)
    _refused(lambda: dg.dg_pack_activations(x, 4, 15, out=x, stream=Stream), 2)
    _refused(lambda: dg.dg_pack_weights(x, 4, 16, out=StandIn(count=15), stream=Stream), 4)
    _refused(lambda: dg.dg_pack_codes_bits(x, 4, 16, 3, out=StandIn(count=31), stream=Stream), 4)
    _refused(lambda: dg.dg_quantize_pack_activations(f, 4, 16, 1.0, 0.0, 0, out=StandIn(count=15), stream=Stream), 4)
    _refused(lambda: dg.dg_dequantize(i, 0, 4, f, out=f, stream=Stream), 2)

    class Table:
        is_f32 = False

        def __init__(self, handle):
            self.handle = handle

    for table in (lut, Table(lut.handle), Table(lut.handle.value)):
        _refused(lambda: dg.dg_gemm_lut(table, x, x, 4, 4, 15, out=i, stream=Stream), 2)
        _refused(lambda: dg.dg_gemm_lut_codes(table, x, x, 4, 4, 15, work=x, out=i, stream=Stream), 2)
        _refused(lambda: dg.dg_conv2d_lut(table, x, x, desc, out=f, scale=f, stream=Stream), 2)
        _refused(lambda: dg.dg_conv2d_lut_codes(table, x, x, desc, work=x, out=i, stream=Stream), 2)
        _refused(lambda: dg.dg_conv2d_lut_codes_static(table, x, x, dg.conv_desc(64, 1024, 1024, 16, 4, 1, 1), i, stream=Stream), 4)
        _refused(lambda: dg.dg_conv2d_lut_requant(table, x, x, desc, f, 1.0, 0.0, 0, out=x, stream=Stream), 2)
    _refused(lambda: dg.dg_gemm_lut(Table(None), x, x, 4, 4, 16, out=i, stream=Stream), 1)
    binary32 = dg.Lut((-1.0, 0.5, 1.0, 2.0), (0.0, 1.0, 2.0, 3.0), entry=np.int64(dg.DG_LUT_F32))       # (its is_f32: numpy's True)
    _refused(lambda: dg.dg_gemm_lut(binary32, x, x, 4, 4, 15, out=f, stream=Stream), 2)
    with pytest.raises(ValueError, match="out must have dtype torch.float32, got torch.int32"):
        dg.dg_gemm_lut(binary32, x, x, 4, 4, 15, out=i, stream=Stream)
    for bad, match in ((StandIn(is_cuda=False), "live in device memory"), (StandIn(contiguous=False), "be contiguous"), (f, "have dtype")):
        with pytest.raises(ValueError, match="codes must " + match):
            dg.dg_pack_activations(bad, 4, 16, out=x, stream=Stream)
    for no_table in ("table", object()):
        with pytest.raises((TypeError, AttributeError)):
            dg.dg_gemm_lut(no_table, x, x, 4, 4, 15, out=i, stream=Stream)

    class Wider(dg.ConvDesc):
        pass

    _refused(lambda: dg.dg_conv2d_lut(lut, x, x, Wider(1, 2, 2, 15, 4, 1, 1, 1, 1, 0, 0), out=i, stream=Stream), 2)
    for no_desc in (bytes(desc), bytearray(desc), np.zeros(11, np.int32), (1, 2, 2, 15, 4, 1, 1, 1, 1, 0, 0)):
        with pytest.raises(TypeError, match="ConvDesc"):
            dg.dg_conv2d_lut(lut, x, x, no_desc, out=i, stream=Stream)


@pytest.mark.gpu
def test_native_checks_on_device_tensors():
    codes = torch.zeros(64, dtype=torch.uint8, device="cuda")
    lut = dg.dg_build_lut((-2, -1, 0, 1), (0, 1, 2, 3))
    with pytest.raises(ValueError, match="codes must have dtype torch.uint8, got torch.float16"):
        dg.dg_pack_activations(codes.half(), 4, 16)
    with pytest.raises(ValueError, match="codes must be contiguous"):
        dg.dg_pack_activations(codes.reshape(8, 8).t(), 4, 16)
    with pytest.raises(TypeError, match="ConvDesc"):
        dg.dg_conv2d_lut(lut, codes, codes, b"1234", out=codes.to(torch.int32))
    with pytest.raises(ValueError, match="out must have dtype torch.float32, got torch.int32"):
        dg.dg_gemm_lut(lut, codes, codes, 4, 4, 16, out=torch.zeros(16, dtype=torch.int32, device="cuda"),
                       scale=torch.ones(4, device="cuda"))
    side = torch.cuda.Stream()                       # a stream of the caller's, and torch's current one
    codes = torch.randint(0, 4, (64,), dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    a = dg.dg_pack_activations(codes, 4, 16, stream=side)
    with torch.cuda.stream(side):
        b = dg.dg_pack_activations(codes, 4, 16)
    torch.cuda.synchronize()
    assert torch.equal(a, b) and torch.equal(a, dg.dg_pack_activations(codes, 4, 16))
