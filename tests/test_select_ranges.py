"""The scores that each block of the top-k selection reads: the blocks' ranges lie
end to end and cover every score once, for any number of scores below 2^32 (the
kernels' own function, compiled for the CPU)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = r"""
#include <hip/hip_runtime.h>
#include <stdio.h>
#include <stdlib.h>
#include "ROOT/paper_2205_15311_amd/csrc/jatam_internal.hpp"
int main(int argc, char** argv)
{
    for (int i = 1; i + 1 < argc; i += 2) {
        const uint32_t n = (uint32_t)strtoull(argv[i], nullptr, 10);
        const uint32_t blocks = (uint32_t)strtoul(argv[i + 1], nullptr, 10);
        uint64_t at = 0;
        for (uint32_t b = 0; b < blocks; ++b) {
            const jatam::SelectRange r = jatam::select_range(n, blocks, b);
            if (r.count != 0 && (r.first != at || (r.first & 255u) != 0u))
                return printf("n %u blocks %u block %u starts at %u\n", n, blocks, b, r.first), 1;
            at += r.count;
        }
        if (at != n)
            return printf("n %u blocks %u cover %llu\n", n, blocks, (unsigned long long)at), 1;
    }
    return 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    folder = tmp_path_factory.mktemp("select")
    source, exe = folder / "ranges.cpp", folder / "ranges"
    source.write_text(SOURCE.replace("ROOT", ROOT))
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__",
                    "-I" + os.path.join(rocm, "include"), "-o", str(exe), str(source)], check=True,
                   capture_output=True, text=True)
    return str(exe)


@pytest.mark.parametrize("n", [1, 255, 256, 257, 1024, 1025, 131_072, 8_388_608, 8_388_609,
                               (1 << 31) + 1, (1 << 32) - 262_145, (1 << 32) - 262_144,
                               (1 << 32) - 257, (1 << 32) - 1])
def test_ranges_cover_every_score_once(program, n):
    args = []
    for blocks in (1, 2, 127, 128, 129, 1023, 1024):
        args += [str(n), str(blocks)]
    res = subprocess.run([program] + args, capture_output=True, text=True)
    assert res.returncode == 0, res.stdout
