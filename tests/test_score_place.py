"""Which part of which row a workgroup of the block scores has: every part once, and where the last parts have nothing to do, what there is to
do spread over the chip.  On the CPU."""
import os
import subprocess

import pytest

from paper_2509_04377_amd import build

CHECK = r"""
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "%s/pe_place.h"
// argv: rows, parts, heads that turn together; prints, for every number of parts with work, the most that eight XCDs of four shader
// engines, taken in turn, get
int main(int argc, char** argv) {
  const uint32_t rows = atoi(argv[1]), parts = atoi(argv[2]), heads = atoi(argv[3]);
  std::vector<uint32_t> part((size_t)rows * parts);
  for (uint32_t b = 0; b < rows * parts; ++b) {
    const uint32_t row = b / parts;
    part[b] = pe::score_part(b, row, parts, row / heads);
    if (part[b] >= parts || (parts %% 2 == 1 && part[b] != b %% parts)) return 1;
  }
  for (uint32_t row = 0; row < rows; ++row) {
    std::vector<int> seen(parts);
    for (uint32_t i = 0; i < parts; ++i)
      if (seen[part[row * parts + i]]++) return 2;
  }
  for (uint32_t used = 1; used <= parts; ++used) {
    uint32_t on[32] = {0}, most = 0;
    for (uint32_t b = 0; b < rows * parts; ++b) on[b %% 32] += part[b] < used;
    for (uint32_t n : on) most = n > most ? n : most;
    printf("%%u ", most);
  }
  return 0;
}
"""


@pytest.fixture(scope="module")
def most_work(tmp_path_factory):
    d = tmp_path_factory.mktemp("score_place")
    src, exe = d / "place.hip", d / "place"
    src.write_text(CHECK % build.CSRC)
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.run([hipcc] + build.FLAGS + [str(src), "-o", str(exe)], check=True, stderr=subprocess.DEVNULL)

    def run(*args):
        out = subprocess.run([str(exe)] + [str(a) for a in args], check=True, capture_output=True, text=True).stdout
        return [int(x) for x in out.split()]
    return run


@pytest.mark.parametrize("heads", [1, 8])
@pytest.mark.parametrize("rows,parts", [(7776, 2), (2560, 4), (1024, 6), (768, 20), (4096, 8), (1024, 64), (777, 3), (768, 27), (40, 1)])
def test_parts_of_rows_over_the_chip(most_work, rows, parts, heads):
    """Parts beside one another, one a row with work, are a multiple of 32 apart at worst: one engine in 32 has all of it.  The bound is what
    numbers at random keep within (six standard deviations of rows * used / 32 each, heads at a time)."""
    for used, most in enumerate(most_work(rows, parts, heads), 1):
        mean = rows * used / 32
        if parts % 2 == 0 or used == parts:
            assert most <= mean + 6 * (mean * heads) ** 0.5 + 1, used
