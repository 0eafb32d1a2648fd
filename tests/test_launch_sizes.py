"""Launch sizes and list positions on the CPU: kernels with several threads per
cell, list or work unit stay below the 2^32 work-items of a dispatch at every
accepted size, and their steps over lists that end near 2^32 entries stay inside
them."""
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


# A wave's walk over 64 / G lists, in the kernels' form: every entry once and no other.
LISTS = r"""
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "sj_launch.hpp"

int main(int argc, char **argv) {
  const uint32_t G = (uint32_t)strtoul(argv[1], nullptr, 10);
  std::vector<uint32_t> off;  // starts of the lists, then the end
  for (int i = 2; i < argc; ++i) off.push_back((uint32_t)strtoull(argv[i], nullptr, 10));
  const size_t lists = off.size() - 1;
  if (lists > 64 / G) return 3;
  std::vector<uint64_t> seen(lists, 0);
  for (uint32_t t = 0;; ++t) {
    bool any = false;
    for (size_t a = 0; a < lists; ++a) any = any || t < sj::list_steps(off[a], off[a + 1], G);
    if (!any) break;
    for (size_t a = 0; a < lists; ++a)
      for (uint32_t l = 0; l < G; ++l) {
        uint32_t i;
        if (!sj::list_entry(off[a], off[a + 1], t, G, l, &i)) continue;
        if (i != off[a] + seen[a] || i >= off[a + 1]) return 1;  // (lanes take them in order)
        ++seen[a];
      }
  }
  for (size_t a = 0; a < lists; ++a)
    if (seen[a] != off[a + 1] - off[a]) return 2;
  return 0;
}
"""


def _compile(tmp_path_factory, name, text):
    d = tmp_path_factory.mktemp(name)
    src, exe = d / (name + ".cpp"), d / name
    src.write_text(text)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-I" + CSRC, "-o", str(exe), str(src)], check=True)
    return str(exe)


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    return _compile(tmp_path_factory, "launch", PROGRAM)


@pytest.fixture(scope="module")
def lists(tmp_path_factory):
    return _compile(tmp_path_factory, "lists", LISTS)


@pytest.mark.parametrize("threads", [8, 64, 128, 256, 512])
@pytest.mark.parametrize("n", [0, 1, 2 ** 23 + 1, 2 ** 25, 2 ** 26 - 1, 2 ** 26, 2 ** 29, 2 ** 32 - 1])
def test_below_a_dispatch(program, n, threads):
    assert subprocess.run([program, str(n), str(threads)]).returncode == 0


@pytest.mark.parametrize("G", [8, 64])
@pytest.mark.parametrize("offsets", [
    [0, 0], [0, 1], [5, 69, 69, 200], [2 ** 32 - 3, 2 ** 32 - 1], [2 ** 32 - 65, 2 ** 32 - 2],
    # a short list that ends at the last entry beside a long one
    [2 ** 32 - 5003, 2 ** 32 - 3, 2 ** 32 - 1], [2 ** 32 - 400, 2 ** 32 - 399, 2 ** 32 - 1]])
def test_lists_at_the_end_of_32_bits(lists, G, offsets):
    offsets = offsets[-(64 // G + 1):]
    assert subprocess.run([lists, str(G)] + [str(x) for x in offsets], timeout=20).returncode == 0
