"""The candidate lists' store (sph_listout.h), compiled for the host: every entry that a list counts has
been written to its slot, also where a target has more candidates than the list takes (the passes walk
those entries), and nothing is written past a slot's capacity."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2107_07315_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <cstring>
#include <map>
#include <random>
#include <vector>
#include <stdint.h>
#define __device__
#define __forceinline__ inline
struct uint4 { uint32_t x, y, z, w; };
static uint4 make_uint4(uint32_t x, uint32_t y, uint32_t z, uint32_t w) { return uint4{x, y, z, w}; }
static std::mt19937 rng(5);
// one lane of the wave: another lane may ask for room at any time
static uint64_t __ballot(bool v) { return v || rng() % 4 == 0; }
static uint32_t __builtin_amdgcn_perm(uint32_t a, uint32_t b, uint32_t sel) {   // bytes 0..3 of b, 4..7 of a
  const uint64_t v = ((uint64_t)a << 32) | b;
  uint32_t r = 0;
  for (int k = 0; k < 4; ++k) r |= (uint32_t)((v >> (8 * ((sel >> (8 * k)) & 0xff))) & 0xff) << (8 * k);
  return r;
}
#include "sph_listout.h"

template <int L>
static int one(int cap, int want, int dense) {
  const int cap_sl = ((cap + L - 1) / L + 7) / 8 * 8, capw = 3;   // cand_slot_capacity; the target is particle 1 of 3
  const int groups = cap_sl / 8;
  std::vector<uint16_t> buf((size_t)8 * groups * capw * L + 64, 0xffff);
  alignas(16) uint16_t ring[kRingRow];
  memset(ring, 0xee, sizeof(ring));
  ListOut<L> out;
  out.ring = ring;
  out.slot0 = reinterpret_cast<uint4*>(buf.data()) + L;
  out.gstride = (int64_t)capw * L;
  out.cap_sl = cap_sl;
  out.cnt = out.stored = 0;
  std::vector<int> entry;   // the local indices appended, in order
  int base = 0;
  while ((int)entry.size() < want) {
    uint32_t u0 = 0, u1 = 0, m0 = 0, m1 = 0;
    for (int b = 0; b < 64; ++b) {
      if ((int)(rng() % 8) >= dense) continue;
      (b < 32 ? u0 : u1) |= 1u << (b & 31);
      if (rng() % 4 == 0 || (int)entry.size() >= want) continue;   // a member of the union, not a hit of this target
      (b < 32 ? m0 : m1) |= 1u << (b & 31);
      const uint64_t u = u0 | (uint64_t)u1 << 32;
      entry.push_back(base + __builtin_popcountll(u) - 1);
    }
    out.append(m0, m1, u0, u1, base, 8191);
    base += __builtin_popcountll(u0 | (uint64_t)u1 << 32);
  }
  out.finish();
  if (out.cnt != (int)entry.size()) return printf("L %d cap %d: count %d of %d\n", L, cap, out.cnt, (int)entry.size()), 1;
  const int counted = out.cnt < cap ? out.cnt : cap;
  std::vector<char> used(buf.size(), 0);
  for (int k = 0; k < counted; ++k) {
    const int s = k % L, e = k / L;
    const size_t at = ((size_t)(e / 8) * capw * L + L + s) * 8 + e % 8;
    const int v = entry[k] < 8191 ? entry[k] : 8191;
    if (buf[at] != v) return printf("L %d cap %d, %d hits: entry %d is %d, not %d\n", L, cap, out.cnt, k, buf[at], v), 1;
  }
  for (int g = 0; g < groups; ++g)   // particles 0 and 2
    for (int p = 0; p < capw; p += 2)
      for (int i = 0; i < 8 * L; ++i)
        if (buf[((size_t)g * capw + p) * L * 8 + i] != 0xffff) return printf("L %d cap %d: another particle's list\n", L, cap), 1;
  for (size_t i = (size_t)8 * groups * capw * L; i < buf.size(); ++i)
    if (buf[i] != 0xffff) return printf("L %d cap %d: past the lists\n", L, cap), 1;
  return 0;
}

int main() {
  int bad = 0, n = 0;
  for (int cap : {2, 16, 24, 80, 88, 200, 1024})
    for (int d : {-33, -9, -1, 0, 1, 6, 31, 32, 33, 63, 64, 200})
      for (int dense = 1; dense <= 8; dense += 2) {
        if (cap + d < 0) continue;
        bad += one<1>(cap, cap + d, dense) + one<2>(cap, cap + d, dense) + one<4>(cap, cap + d, dense);
        n += 3;
      }
  printf("%d lists, %d wrong\n", n, bad);
  return bad ? 1 : 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_counted_entries_are_stored(tmp_path):
    src, exe = tmp_path / "lists.cpp", tmp_path / "lists"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, "-o", str(exe), str(src)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout[-2000:]
