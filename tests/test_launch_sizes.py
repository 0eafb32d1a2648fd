"""Launch sizes on the CPU: kernels with several threads per cell, list or work
unit stay below the 2^32 work-items of a dispatch at every accepted size."""
import os
import subprocess

import pytest

from conftest import ROOT

CSRC = os.path.join(ROOT, "paper_1809_09930_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "sj_launch.hpp"

int main(int argc, char **argv) {
  const uint64_t n = strtoull(argv[1], nullptr, 10);
  const uint32_t threads = (uint32_t)strtoul(argv[2], nullptr, 10);
  const uint64_t strided = (uint64_t)sj::stride_blocks(n * threads) * sj::kLaunchBlock;
  if (strided >= 1ull << 32 || (n && !strided)) return 1;
  uint64_t next = 0;
  int ok = 1;
  sj::for_unit_launches(n, threads, [&](uint64_t u, uint64_t m) {
    // whole workgroups of up to 512 threads, the units in order and each once
    ok = ok && u == next && m > 0 && m <= n - u;
    ok = ok && (m * threads + 511) / 512 * 512 < 1ull << 32;
    next = u + m;
  });
  return ok && next == n ? 0 : 2;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("launch")
    src, exe = d / "launch.cpp", d / "launch"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-I" + CSRC, "-o", str(exe), str(src)], check=True)
    return str(exe)


@pytest.mark.parametrize("threads", [8, 64, 128, 256, 512])
@pytest.mark.parametrize("n", [0, 1, 2 ** 23 + 1, 2 ** 25, 2 ** 26 - 1, 2 ** 26, 2 ** 29, 2 ** 32 - 1])
def test_below_a_dispatch(program, n, threads):
    assert subprocess.run([program, str(n), str(threads)]).returncode == 0
