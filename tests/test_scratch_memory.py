"""What the compiler made of the kernels (the objects that the library is linked from; no GPU): scratch memory in a hot loop is a trip
to device memory that no source line shows."""
import glob
import os
import re
import subprocess

import pytest

LLVM = "/opt/rocm/llvm/bin/"


def compiled(obj, tmp):
    """kernel -> (bytes of scratch memory per lane, vector registers)"""
    fat, code = str(tmp / "fat"), str(tmp / "code")
    subprocess.run([LLVM + "llvm-objcopy", "--dump-section", ".hip_fatbin=" + fat, obj, str(tmp / "rest.o")], check=True)
    subprocess.run([LLVM + "clang-offload-bundler", "--unbundle", "--type=o", "--targets=hipv4-amdgcn-amd-amdhsa--gfx950", "--input=" + fat, "--output=" + code],
                   check=True)
    notes = subprocess.run([LLVM + "llvm-readelf", "--notes", code], check=True, capture_output=True, text=True).stdout
    found = {}
    for kernel in notes.split("- .agpr_count")[1:]:
        found[re.search(r"\.name: +(\S+)", kernel).group(1)] = tuple(int(re.search(rf"\.{field}: +(\d+)", kernel).group(1)) for field in ("private_segment_fixed_size", "vgpr_count"))
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
        found.update(compiled(obj, tmp_path))
    assert len(found) > 100
    assert not {k: v for k, v in found.items() if v[0] != 0}


@pytest.mark.skipif(not os.path.exists(LLVM + "clang-offload-bundler"), reason="needs ROCm's LLVM tools")
def test_scan_by_one_byte_bounds_keeps_nothing_in_scratch_memory(pqlib_path, tmp_path):
    from paper_2408_09992_amd import build
    obj = os.path.join(build.OBJ, "inst_scan_bytes.o")
    if not os.path.exists(obj):
        pytest.skip("the library was built elsewhere")
    found = compiled(obj, tmp_path)
    assert len(found) == 9 and not {k: v for k, v in found.items() if v[0] != 0}


@pytest.mark.skipif(not os.path.exists(LLVM + "clang-offload-bundler"), reason="needs ROCm's LLVM tools")
def test_kernels_by_pairs_leave_room_for_two_workgroups(pqlib_path, tmp_path):
    # eight waves each on four SIMDs of 512 registers: 128 at most.  (With 129, 28,058 items, m = 4, 496 queries take 20.2 us instead of 15.8; with 132 a list of 13,498
    # candidates, m = 16, 899 queries 67 instead of 45.)  What holds more vectors to a thread has never had room for two.
    from paper_2408_09992_amd import build
    two = {"scan_pair_kernelILi4ELi%dELi512ELi1E": range(1, 8), "scan_pair_kernelILi8ELi%dELi512ELi1E": (1, 2, 3, 4, 5, 6, 7, 8, 12),
           "scan_pair_kernelILi16ELi%dELi512ELi1E": (1, 2, 3, 4, 5, 6, 7, 8, 12, 16, 20, 24), "scan_pair_kernelILi32ELi%dELi512ELi1E": (1, 2, 3, 4, 8, 12, 16, 20),
           "scan_pair_kernelILi4ELi%dELi512ELi2E": (1, 2, 3, 4, 5, 6, 7, 8, 12), "scan_pair_kernelILi8ELi%dELi512ELi2E": (1, 2, 3, 4, 5, 6, 7, 8, 12, 16, 20, 24),
           "scan_pair_kernelILi16ELi%dELi512ELi2E": (1, 2, 3, 4, 8, 12, 16, 20, 24), "scan_subset_pair_kernelILi4ELi%dELi512E": (1, 2, 3, 4),
           "scan_subset_pair_kernelILi8ELi%dELi512E": (1, 2, 3, 4, 6, 8), "scan_subset_pair_kernelILi16ELi%dELi512E": (1, 2, 3, 4, 6, 8, 12, 16)}
    objects = glob.glob(os.path.join(build.OBJ, "inst_scan_pair_*.o")) + glob.glob(os.path.join(build.OBJ, "inst_scan_subset_pair.o"))
    if not objects:
        pytest.skip("the library was built elsewhere")
    found = {}
    for obj in objects:
        found.update(compiled(obj, tmp_path))
    for kernel, units in two.items():
        for u in units:
            registers = [v[1] for k, v in found.items() if kernel % u in k]
            assert len(registers) == 1 and registers[0] <= 128, (kernel % u, registers)
