"""Packing of 3- and 4-bit codes, 16 to a lane and the pairs that are left: byte for byte the oracle's, bits above a code's dropped,
at any address."""
import numpy as np
import pytest
import torch

import oracle
from paper_2304_09049_amd import binding as dg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits", [3, 4])
@pytest.mark.parametrize("rows,K", [(1, 2), (1, 14), (3, 10), (1, 16), (5, 18), (7, 64), (33, 130), (257, 4112), (1500, 2050)])
@pytest.mark.parametrize("shift_in,shift_out", [(0, 0), (2, 0), (0, 1), (1, 3)])
def test_pack_slots(bits, rows, K, shift_in, shift_out):
    rng = np.random.default_rng(rows + K)
    dirty = rng.integers(0, 256, size=(rows, K), dtype=np.uint8)
    codes = torch.empty(rows * K + shift_in, dtype=torch.uint8, device="cuda")[shift_in:].copy_(torch.from_numpy(dirty).flatten())
    whole = torch.full((rows * K // 2 + shift_out + 16,), 0xA5, dtype=torch.uint8, device="cuda")
    out = whole[shift_out:shift_out + rows * K // 2]
    dg.dg_pack_codes_bits(codes, rows, K, bits, out=out)
    assert np.array_equal(out.cpu().numpy().reshape(rows, K // 2), oracle.pack_codes(dirty & ((1 << bits) - 1), bits))
    assert (whole[:shift_out] == 0xA5).all() and (whole[shift_out + rows * K // 2:] == 0xA5).all()
