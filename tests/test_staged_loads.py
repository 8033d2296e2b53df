"""The staged kernel's loads by their machine code: the hardware holds a buffer load's LANE offset against the buffer's size, and takes a
scalar offset off that size in 32 bits, so a load that is switched off (past the end of K) through its scalar offset is not
outside at all.  No load may have one."""
import os
import re
import subprocess

from paper_2304_09049_amd.build import HIPCC_FLAGS

FORMS = ["1, 2, 4, false, false, false, false", "1, 2, 1, false, true, false, false",       # whole runs, half runs
         "1, 4, 4, true, false, true, false", "2, 4, 2, false, false, false, true"]         # 4-bit slots, two planes


def test_no_staged_load_has_a_scalar_offset(tmp_path):
    source, listing = tmp_path / "forms.hip", tmp_path / "forms.s"
    source.write_text('#include "dg_sparse_staged_kernel.h"\n' +
                      "".join(f"template __global__ void dgoh::smfmac_staged_kernel<{f}>(dgoh::Args);\n" for f in FORMS))
    flags = [f for f in HIPCC_FLAGS if f not in ("-O3", "-shared", "-fPIC")]
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-O1", *flags, "--cuda-device-only", "-S", str(source), "-o", str(listing)],
                   check=True, stderr=subprocess.DEVNULL)
    offsets = re.findall(r"buffer_load_dwordx4 v\d+, s\[\d+:\d+\], (\S+) offen lds", listing.read_text())
    assert len(offsets) >= 4 * 3 * 2 and set(offsets) == {"0"}, set(offsets)
