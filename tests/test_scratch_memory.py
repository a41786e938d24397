"""What the compiler made of the kernels (the objects that the library is linked from; no GPU): scratch memory in a hot loop is a trip
to device memory that no source line shows."""
import glob
import os
import re
import subprocess

import pytest

LLVM = "/opt/rocm/llvm/bin/"


def scratch_bytes(obj, tmp):
    """kernel -> bytes of scratch memory per lane"""
    fat, code = str(tmp / "fat"), str(tmp / "code")
    subprocess.run([LLVM + "llvm-objcopy", "--dump-section", ".hip_fatbin=" + fat, obj, str(tmp / "rest.o")], check=True)
    subprocess.run([LLVM + "clang-offload-bundler", "--unbundle", "--type=o", "--targets=hipv4-amdgcn-amd-amdhsa--gfx950", "--input=" + fat, "--output=" + code],
                   check=True)
    notes = subprocess.run([LLVM + "llvm-readelf", "--notes", code], check=True, capture_output=True, text=True).stdout
    found = {}
    for kernel in notes.split("- .agpr_count")[1:]:
        found[re.search(r"\.name: +(\S+)", kernel).group(1)] = int(re.search(r"\.private_segment_fixed_size: +(\d+)", kernel).group(1))
    return found


@pytest.mark.skipif(not os.path.exists(LLVM + "clang-offload-bundler"), reason="needs ROCm's LLVM tools")
def test_scans_by_bounds_and_by_pairs_keep_nothing_in_scratch_memory(pqlib_path, tmp_path):
    from paper_2408_09992_amd import build
    objects = sorted(glob.glob(os.path.join(build.OBJ, "inst_filter_*.o")) + glob.glob(os.path.join(build.OBJ, "inst_scan_pair_*.o")) +
                     glob.glob(os.path.join(build.OBJ, "inst_scan_subset_pair.o")))
    if not objects:
        pytest.skip("the library was built elsewhere")
    found = {}
    for obj in objects:
        found.update(scratch_bytes(obj, tmp_path))
    assert len(found) > 100
    assert not {k: v for k, v in found.items() if v != 0}
