"""The number of workgroups of a kernel that a compute unit holds is asked for every kernel by itself, also for kernels of
one signature (host code alone, with an occupancy query that answers by the kernel it is asked about)."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2303_13775_amd", "csrc")

PROGRAM = r"""
#include <cstddef>
#include <cstdio>
enum { hipSuccess = 0 };
static void first(int) {}
static void second(int) {}
static void unknown(int) {}
static int asked = 0;
static int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *nb, void (*kernel)(int), int, size_t) {
    ++asked;
    *nb = kernel == first ? 6 : kernel == second ? 3 : 0;
    return hipSuccess;
}
#include "resident.h"
int main() {
    const int a = resident_blocks<first>(), b = resident_blocks<second>(), c = resident_blocks<unknown>();
    const int again = resident_blocks<first>();
    std::printf("%d %d %d %d %d\n", a, b, c, again, asked);
}
"""


def test_kernels_of_one_signature_have_answers_of_their_own(tmp_path):
    src, exe = tmp_path / "resident.cpp", tmp_path / "resident"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split()
    assert [int(x) for x in out] == [6, 3, 4, 6, 3]     # (a failed query counts as four; no query is repeated)
