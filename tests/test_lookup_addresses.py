"""Addresses that kernels form from sub-ids, computed by the kernels' own host-callable functions in a small host program (no GPU):
a sub-id of 16 bits may lie beyond the alphabet, and no lookup in device memory may leave its table then."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"

FAR_ROWS = r"""
#define PQ_INSTANCE_TU
#include "kernels.hpp"
#include <cstdio>
#include <initializer_list>
using namespace pqk;
int main() {
    long long checked = 0;
    for (uint32_t m : {4u, 8u, 16u}) {
        const uint32_t splits = filter_far_splits((int)m, 4, false, 2), queries = 32, part = 16;   // a lane reads 16 of a row's 32 bytes
        for (uint32_t b : {1u, 2u, 257u, 300u, 1024u, 2047u, 2048u})
            for (uint32_t v = 0; v < splits; ++v)
                for (uint32_t id = 0; id < 65536; ++id)
                    for (uint32_t first = 0; first < queries; first += part, ++checked) {
                        const unsigned long long at = filter_far_at(v, id, b, queries, first), end = (unsigned long long)splits * b * queries;
                        const unsigned long long row = (unsigned long long)v * b + (id < b ? id : b - 1);
                        if (at + part > end || at != row * queries + first || at % part != 0) {
                            std::printf("m %u b %u split %u sub-id %u: byte %llu of %llu\n", m, b, v, id, at, end);
                            return 1;
                        }
                    }
    }
    std::printf("checked %lld\n", checked);
    return checked > 0 ? 0 : 1;
}
"""


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
def test_rows_in_device_memory_are_never_left(tmp_path):
    source, exe = tmp_path / "far_rows.hip", tmp_path / "far_rows"
    source.write_text(FAR_ROWS)
    build = subprocess.run([HIPCC, "--offload-arch=gfx950", "--cuda-host-only", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "include"), "-I",
                            os.path.join(ROOT, "paper_2408_09992_amd", "csrc"), str(source), "-o", str(exe)], capture_output=True, text=True)
    assert build.returncode == 0, build.stderr
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert run.returncode == 0, run.stdout + run.stderr
