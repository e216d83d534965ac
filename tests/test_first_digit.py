"""The first digit that pooling counts and selection reads (first_digit.h), over all keys, in a host program."""
import os
import shutil
import subprocess

import pytest

PROGRAM = r"""
#include <cstdio>
#define __host__
#define __device__
#include "first_digit.h"
using namespace speckv;
int main() {
  int before = 0;
  uint32_t seen[2048] = {0};
  // every change of digit is at a multiple of 2^18: both ends of each such run of keys
  for (uint64_t base = 0; base < (1ull << 32); base += 1u << 18) {
    const uint32_t ends[2] = {(uint32_t)base, (uint32_t)(base + (1u << 18) - 1)};
    for (uint32_t key : ends) {
      const int D = first_digit_of(key);
      if (D < before || D > 2047) { std::printf("key %08x: digit %d after %d\n", key, D, before); return 1; }
      before = D;
      seen[D] = 1;
      int open;
      const uint32_t prefix = key_prefix_of((uint32_t)D, &open);
      // a positive number, infinity or NaN is described by its digit, by at least as many bits as 2 of mantissa make
      if (key >= 0x80000000u) {
        if (open != 21 && open != 18) { std::printf("key %08x: %d bits open\n", key, open); return 1; }
        if (prefix >> open != key >> open || prefix << (32 - open) != 0) { std::printf("key %08x: prefix %08x\n", key, prefix); return 1; }
        const bool usual = key >= (0x80000000u | (98u << 23)) && key < (0x80000000u | (134u << 23));     // 2^-29 to 2^7
        if (usual != (open == 18)) { std::printf("key %08x: %d bits open\n", key, open); return 1; }
      } else if (open != 32) { std::printf("key %08x: %d bits open\n", key, open); return 1; }
    }
  }
  // a digit that stands for keys stands for none but those (the prefix leads back to it)
  for (uint32_t D = 0; D < 2048; ++D) {
    int open;
    const uint32_t prefix = key_prefix_of(D, &open);
    if (open == 32) { if (D > 0 && D <= (uint32_t)kLastDigit) return 1; continue; }
    if (!seen[D] || first_digit_of(prefix) != (int)D || first_digit_of(prefix + ((1u << open) - 1u)) != (int)D) { std::printf("digit %u\n", D); return 1; }
  }
  std::printf("digits ok\n");
  return 0;
}
"""


def test_first_digit_covers_every_score(repo_root, tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    src, exe = tmp_path / "digits.cpp", str(tmp_path / "digits")
    src.write_text(PROGRAM)
    subprocess.run([cxx, "-std=c++17", "-O2", "-Wall", "-Werror", "-I",
                    os.path.join(repo_root, "paper_2506_08373_amd", "csrc"), str(src), "-o", exe],
                   check=True, capture_output=True, text=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0 and "digits ok" in r.stdout, r.stdout
