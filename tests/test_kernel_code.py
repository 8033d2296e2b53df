"""Kernels' machine code, compiled here: what the staged kernel's loads rely on, the registers that its narrow tiles may take, how the kernel
for ragged channel counts reads its table, and that no main loop of the kernel for products of levels reloads from scratch."""
import os
import re
import subprocess

import pytest

from paper_2304_09049_amd.build import CSRC, HIPCC_FLAGS


def compile_forms(tmp_path, forms, *flags, header="dg_sparse_staged_kernel.h", kernel="smfmac_staged_kernel", arguments="Args"):
    """The listing of a kernel's instantiations (the staged kernel's: <WM, WN, SKW, TURNS, HALF, NIB, TWO, SHORT>)."""
    source = tmp_path / "forms.hip"
    source.write_text(f'#include "{header}"\n' +
                      "".join(f"template __global__ void dgoh::{kernel}<{f}>(dgoh::{arguments});\n" for f in forms))
    return compile_listing(tmp_path, source, *flags)


def compile_listing(tmp_path, source, *flags):
    listing = tmp_path / "forms.s"
    common = [f for f in HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *common, *flags, "--cuda-device-only", "-S", str(source), "-o", str(listing)],
                   check=True, stderr=subprocess.DEVNULL)
    return listing.read_text()


def test_no_staged_load_has_a_scalar_offset(tmp_path):
    """The hardware holds a buffer load's LANE offset against the buffer's size, and takes a scalar offset off that size in 32 bits, so
    a load that is switched off (past the end of K) through its scalar offset is not outside at all."""
    text = compile_forms(tmp_path, ["1, 2, 4, false, false, false, false", "1, 2, 1, false, true, false, false",       # whole runs, half runs
                                    "1, 4, 4, true, false, true, false", "2, 4, 2, false, false, false, true"],        # 4-bit slots, two planes
                         "-O1")
    offsets = re.findall(r"buffer_load_dwordx4 v\d+, s\[\d+:\d+\], (\S+) offen lds", text)
    assert len(offsets) >= 4 * 3 * 2 and set(offsets) == {"0"}, set(offsets)


# (512 registers per SIMD lane, handed out by eights: 128 for four wavefronts, 168 for three)
@pytest.mark.parametrize("most,forms", [(128, [f"1, 2, {s}, {nib}, false" for s in ("1, false, false", "1, false, true", "2, false, false", "2, true, false",
                                                                                     "4, false, false", "4, true, false") for nib in ("false", "true")]),
                                        (168, ["2, 2, 4, true, false, false, true", "1, 4, 1, false, false, false, false, true"])])
def test_tiles_leave_room_for_the_next_workgroups(tmp_path, most, forms):
    """Layers of up to 1024 narrow tiles that four wavefronts share are all resident at once -- if a SIMD holds four of them (two planes without a
    filter window, and unshared 32 x 128 tiles: three) -- and run in two rounds otherwise."""
    text = compile_forms(tmp_path, forms)
    registers = [int(n) for n in re.findall(r"\.vgpr_count:\s+(\d+)", text)]
    assert len(registers) == len(forms) and max(registers) <= most, registers
    assert set(re.findall(r"\.private_segment_fixed_size:\s+(\d+)", text)) == {"0"}
    assert max(int(n) for n in re.findall(r"\.group_segment_fixed_size:\s+(\d+)", text)) * (512 // most) <= 160 * 1024


@pytest.fixture(scope="module")
def ragged_listing(tmp_path_factory):
    return compile_forms(tmp_path_factory.mktemp("ragged"), [], header="dg_sparse_ragged_kernel.h")        # (its launches instantiate every form)


def test_ragged_table_comes_with_the_scalar_arguments(ragged_listing):
    """Read from the arguments lane by lane, the table's rows were two vector loads that every launch waited for."""
    text = ragged_listing
    kernels = re.findall(r"^(_ZN4dgoh20smfmac_ragged_kernelILi(\d)ELi(\d)ELi(\d)\S+):(.*?)s_barrier", text, re.M | re.S)
    assert len(kernels) == 3 * 4 * 2
    for name, wm, wn, ch, start in kernels:
        # single words before the barrier: a scale per block of channels, and operands of one word (packed activations too)
        words = int(wm) + (2 * int(wm) + int(wn) if ch == "1" else 0)
        assert len(re.findall(r"global_load_dword ", start)) <= words, name


def test_ragged_wavefronts_eight_to_a_simd(ragged_listing):
    """A workgroup of 13 to 16 wavefronts has a second one beside it on a compute unit only if a SIMD holds eight of them: 64 vector registers, and
    80 scalar ones (of 800, handed out by sixteens; measured: at 82 the second workgroup waits for the first).  No form spills, and none waits for loads
    between its stores (a wait for one that was never used is a wait for every store before)."""
    text = ragged_listing
    kernels = re.findall(r"^(_ZN4dgoh20smfmac_ragged_kernelILi(\d)ELi(\d)ELi(\d)ELb(\d)\S+):(.*?)^\.Lfunc_end", text, re.M | re.S)
    notes = {name: (int(scalars), int(vectors), int(scratch)) for scratch, scalars, name, vectors in re.findall(
        r"\.private_segment_fixed_size: (\d+)\s+\.sgpr_count:\s+(\d+).*?\.symbol:\s+(\S+)\.kd.*?\.vgpr_count:\s+(\d+)", text, re.S)}
    assert len(kernels) == len(notes) == 3 * 4 * 2
    for name, wm, wn, ch, raw, code in kernels:
        scalars, vectors, scratch = notes[name]
        assert scratch == 0, name
        if wm == wn == "1":
            assert scalars <= 80 and vectors <= (64 if ch == "1" else 512), (name, scalars, vectors)
        assert code.count("vmcnt(") <= 16, (name, code.count("vmcnt("))


def test_twopower_loops_keep_their_registers(tmp_path):
    """The tiles of 128 channels take all 256 registers.  A reload from scratch in the main loop waits for every load before it: for the next run's
    pixels and weights, which are to arrive while this run is multiplied."""
    text = compile_listing(tmp_path, os.path.join(CSRC, "dg_twopower_kernel.hip"))
    kernels = re.findall(r"^(\S*twopower_kernelILi\d\S+):(.*?)^\.Lfunc_end", text, re.M | re.S)
    assert len(kernels) == 4 * 2
    for name, code in kernels:
        loops = [body for _, body in re.findall(r"^(\.LBB\d+_\d+):[^\n]*Inner Loop(.*?)s_cbranch_\w+ \1$", code, re.M | re.S)]
        mains = [body for body in loops if "s_barrier" in body and body.count("v_mfma") >= 16]
        assert len(mains) == 1, name
        assert "scratch_" not in mains[0], name


def test_onebit_loops_start_their_loads_as_measured(tmp_path):
    """The next run's loads start before this run's words are read from LDS where a run waits for nothing else: narrow tiles whose outputs' rows are
    pixels, and K shared by two without a window or beyond the caches.  In the other forms the loads' addresses would hold up the matrix instructions."""
    text = compile_listing(tmp_path, os.path.join(CSRC, "dg_onebit_kernel.hip"))
    kernels = re.findall(r"^\S*onebit_kernelILi(\d)ELi(\d)ELb(\d)ELb(\d)ELb(\d)E\S*:(.*?)^\.Lfunc_end", text, re.M | re.S)
    assert len(kernels) == 3 * 3 + 4
    for wn, ks, taps, tr, first, code in kernels:
        loops = [body for _, body in re.findall(r"^(\.LBB\d+_\d+):[^\n]*Inner Loop(.*?)s_cbranch_\w+ \1$", code, re.M | re.S)]
        mains = [body[body.index("s_barrier"):] for body in loops if "s_barrier" in body and body.count("v_mfma") >= 16]
        assert len(mains) == (2 if wn == "2" else 1)
        for body in mains:
            narrow = body.count("v_mfma") == 16
            reads_first = body.index("ds_read") < body.index("buffer_load")
            want = not narrow or (first == "1" and taps == "1" if ks == "2" else tr == "0")
            assert reads_first == want, (wn, ks, taps, tr, first, body.count("v_mfma"))
