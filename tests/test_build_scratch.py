"""The temporaries of a plan build (Scratch in csrc/internal.h), taken from a
simulated device of limited memory: compiled and run on the host."""
import shutil
import subprocess
from pathlib import Path

import pytest

ROOT = Path(__file__).resolve().parent.parent
GXX = shutil.which("g++")

SOURCE = r"""
#include <cstdio>
#include <map>
#include "paper_2511_15269_amd/csrc/internal.h"

// a device that hands out `room` bytes
static size_t room = 0, used = 0, peak = 0, calls = 0;
static std::map<void*, size_t> live;
static char* next = (char*)(1 << 20);

namespace fmm {
void* dev_alloc(fmm_plan*, size_t bytes) {
  if (used + bytes > room) throw Error{FMM_ENOMEM, "full"};
  used += bytes;
  if (used > peak) peak = used;
  ++calls;
  void* p = next;
  next += (bytes + 511) / 256 * 256;
  live[p] = bytes;
  return p;
}
void dev_free(fmm_plan*, void* p) {
  used -= live.at(p);
  live.erase(p);
}
}  // namespace fmm

static const size_t MB = (size_t)1 << 20;

// requests of `sizes` under `expect` in a device of `r` bytes: whether they
// fit; pieces must not overlap
static bool fits(size_t r, size_t expect, const std::vector<size_t>& sizes) {
  fmm_plan pl;
  room = r;
  used = peak = calls = 0;
  std::map<char*, size_t> piece;
  try {
    fmm::Scratch sc(&pl, expect);
    for (size_t b : sizes) {
      char* p = (char*)sc.get(b);
      if (!p) {
        std::puts("NULL");
        return false;
      }
      auto it = piece.lower_bound(p);
      if (it != piece.end() && p + b > it->first) std::puts("OVERLAP");
      if (it != piece.begin() && std::prev(it)->first + std::prev(it)->second > p)
        std::puts("OVERLAP");
      piece[p] = b;
    }
  } catch (const fmm::Error&) {
    if (used != 0 || !live.empty()) std::puts("LEAK");
    return false;
  }
  if (used != 0 || !live.empty()) std::puts("LEAK");
  return true;
}

int main() {
  // requests of about a whole block, whatever the remainder by 256
  bool all = true;
  for (size_t e : {(size_t)0, (size_t)160 * 12345, (size_t)160 * 777})
    for (size_t less : {0, 1, 100, 255, 256, 300})
      all = all && fits((size_t)1 << 50, e, {4 * MB + e - less, 5});
  std::printf("whole block: %d\n", (int)all);
  // lists of a level march: ten arrays a level, the last levels the largest,
  // three times what was expected in all
  std::vector<size_t> march;
  for (size_t level = 1; level <= 10; ++level)
    for (int k = 0; k < 10; ++k) march.push_back(((size_t)3 << level) * MB / 16 + 4);
  auto sum = [](const std::vector<size_t>& v) {
    size_t s = 0;
    for (size_t b : v) s += (b + 255) / 256 * 256;
    return s;
  };
  for (size_t f : {(size_t)1, (size_t)16, (size_t)256}) {
    std::vector<size_t> v;
    for (size_t b : march) v.push_back(b * f);
    const size_t need = sum(v);
    std::printf("march %zu: %d", need / MB, (int)fits(need + need / 8 + 64 * MB, need / 3, v));
    fits((size_t)1 << 50, need / 3, v);
    std::printf(" peak %zu calls %zu\n", peak / MB, calls);
  }
  // a build whose expected block is larger than what it needs, and larger than
  // the device
  std::printf("over: %d", (int)fits(100 * MB, 800 * MB, {30 * MB, 30 * MB, 30 * MB}));
  std::printf(" %d", (int)fits(1000 * MB, 40000 * MB, {300 * MB, 300 * MB, 300 * MB}));
  // small requests right after an expected block that does not fit
  std::printf(" %d\n", (int)fits(3 * MB, 800 * MB, {MB, 100, MB, 200}));
  // ordinary builds: one block where the expectation holds
  fits((size_t)1 << 50, 16 * MB, {5 * MB, 4 * MB, 3 * MB, 1 * MB, 100, 7});
  std::printf("ordinary calls %zu\n", calls);
  return 0;
}
"""


@pytest.mark.skipif(GXX is None, reason="no g++")
def test_build_temporaries_fit_where_their_sum_fits(tmp_path):
    src, exe = tmp_path / "scratch.cpp", tmp_path / "scratch"
    src.write_text(SOURCE)
    subprocess.run([GXX, "-std=c++17", "-O1", "-Wno-unused", "-D__HIP_PLATFORM_AMD__",
                    f"-I{ROOT}", "-I/opt/rocm/include", str(src), "-o", str(exe),
                    "-L/opt/rocm/lib", "-lamdhip64", "-Wl,-rpath,/opt/rocm/lib"],
                   check=True, capture_output=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout
    print(out)
    lines = out.splitlines()
    assert not {"OVERLAP", "LEAK", "NULL"} & set(lines)
    assert lines.pop(0) == "whole block: 1"
    for line, factor in zip(lines[:3], (1, 16, 256)):
        words = line.replace(":", "").split()
        need, ok, peak = int(words[1]), int(words[2]), int(words[4])
        # all temporaries that fit into 8/9 of the device are given
        assert ok == 1
        assert peak <= need * 9 / 8 + 64
        assert int(words[6]) <= 100
    assert lines[3] == "over: 1 1 1"
    assert lines[4] == "ordinary calls 1"
