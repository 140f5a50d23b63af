"""The list that the survivors of all queries share (csrc/survivors.hpp): every entry that is read has been written, in
whatever order the workgroups take their places.  Compiled for the host; the loop below is ms_list_kernel's."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2401_08281_amd", "csrc")

PROGRAM = r"""
#include <algorithm>
#include <cstdio>
#include <random>
#include <vector>
#include "survivors.hpp"

static int check(const std::vector<unsigned>& mine, unsigned cap, std::mt19937& rng) {
  const size_t nq = mine.size(), blocks = (nq + 15) / 16;
  std::vector<size_t> order(blocks);
  for (size_t b = 0; b < blocks; ++b) order[b] = b;
  std::shuffle(order.begin(), order.end(), rng);
  std::vector<int> writes(cap, 0);
  std::vector<char> again(nq, 0);
  unsigned count = 0, unwritten = 0, starts_inside = 0;
  for (size_t b : order) {
    unsigned base = count, t = 0;
    for (size_t w = 0; w < 16 && b * 16 + w < nq; ++w) {
      const unsigned n = mine[b * 16 + w], at = base + t;
      t += n;
      const SurvivorPlace p = survivor_place(at, n, cap);
      if (p.unwritten) { unwritten = p.unwritten; ++starts_inside; }
      if (p.full) { again[b * 16 + w] = 1; continue; }
      for (unsigned i = 0; i < n; ++i) { if (at + i >= cap) return 1; ++writes[at + i]; }
    }
    count = base + t;
  }
  const unsigned total = survivors_written(count, cap, unwritten);
  if (starts_inside > 1 || total > cap) return 2;
  for (unsigned i = 0; i < cap; ++i) if (writes[i] != (i < total ? 1 : 0)) return 3;
  unsigned kept = 0;
  for (size_t q = 0; q < nq; ++q) if (!again[q]) kept += mine[q];
  if (kept != total) return 4;
  if (count <= cap && kept != count) return 5;      // what fits is kept
  return 0;
}

int main() {
  std::mt19937 rng(5);
  int bad = 0, runs = 0;
  auto run = [&](const std::vector<unsigned>& mine, unsigned cap) {
    const int r = check(mine, cap, rng);
    ++runs;
    if (r) { std::printf("failed: code %d, %zu queries, room for %u\n", r, mine.size(), cap); ++bad; }
  };
  for (unsigned nq : {1u, 15u, 16u, 17u, 333u})
    for (unsigned each : {0u, 1u, 168u, 500u, 4096u})
      for (long off : {-1000000L, -1L, 0L, 1L, 7L}) {       // one survivor too many, exactly full, one place left, ...
        const long cap = off == -1000000L ? (long)nq * each / 3 : (long)nq * each + off;
        if (cap >= 0) run(std::vector<unsigned>(nq, each), (unsigned)cap);
      }
  for (int i = 0; i < 2000; ++i) {
    std::vector<unsigned> mine(1 + rng() % 200);
    unsigned sum = 0;
    for (unsigned& m : mine) { m = rng() % 4 ? rng() % 40 : 0; sum += m; }
    run(mine, rng() % (sum + 20));
    run(mine, sum);
    if (sum) run(mine, sum - 1);
  }
  std::printf("%d runs, %d failed\n", runs, bad);
  return bad != 0;
}
"""


def test_every_survivor_that_is_read_was_written(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    src, exe = tmp_path / "places.cpp", str(tmp_path / "places")
    src.write_text(PROGRAM)
    subprocess.run([gxx, "-std=c++17", "-O1", "-Wall", "-Werror", "-I", CSRC, str(src), "-o", exe], check=True)
    run = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=60)
    assert run.returncode == 0, run.stdout[-2000:]
