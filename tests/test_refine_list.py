"""The cubes a refinement lists (the library's helpers, compiled here for the
host): exactly those outside the list keep their type under Eqs. (3)-(5), for
every type, previous type and set of near corners; a listed cube's eight bits
read from its four rows of corners or from a row's planes are its type, and
flipping them in the planes changes that cube alone."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1803_03949_amd", "csrc")

PROBE = r"""
#include <stdio.h>
#include "vm_internal.h"
using namespace vm;
int main() {
  long n = 0, bad = 0, listed = 0;
  for (uint32_t t = 0; t < 256; ++t) {
    const uint64_t cand = refine_candidates(t);
    for (int x = 0; x < 8; ++x) {
      // the cube among empty and among full ones
      for (uint32_t rest = 0; rest < 2; ++rest) {
        uint32_t lo = rest ? ~(0x01010101u << x) : 0u, hi = lo;
        lo |= planes_flip(t, x), hi |= planes_flip(t >> 4, x);
        const uint32_t want = refinable_cubes(lo, hi);
        bad += (want & ~(1u << x)) != 0;
        listed += want != 0;
        bad += planes_type(lo, hi, x) != t;
        bad += planes_type((uint64_t)hi << 32 | lo, x) != t;
        for (uint32_t f = 0; f < 256; f += 37) {
          const uint32_t l2 = lo ^ planes_flip(f, x), h2 = hi ^ planes_flip(f >> 4, x);
          for (int k = 0; k < 8; ++k)
            bad += planes_type(l2, h2, k) != (k == x ? t ^ f : planes_type(lo, hi, k));
        }
        // rows of corners with the cube's corners at bits s and s + 1
        for (uint32_t s = x; s <= 18u + x; s += 9) {
          const uint32_t pad = rest ? ~(3u << s) : 0u;
          const uint32_t r00 = pad | ((t & 1) | (t >> 1 & 1) << 1) << s;
          const uint32_t r10 = pad | ((t >> 3 & 1) | (t >> 2 & 1) << 1) << s;
          const uint32_t r01 = pad | ((t >> 4 & 1) | (t >> 5 & 1) << 1) << s;
          const uint32_t r11 = pad | ((t >> 7 & 1) | (t >> 6 & 1) << 1) << s;
          bad += corner_bits(r00, r10, r01, r11, s) != t;
        }
      }
    }
    const bool can = refinable_cubes(planes_flip(t, 3), planes_flip(t >> 4, 3)) != 0;
    bool some = false;
    for (uint32_t prev = 0; prev < 256; ++prev)
      for (uint32_t near8 = 0; near8 < 256; ++near8) {
        const uint32_t r = refine_type(t, prev, (refine_candidates(prev) >> 63) != 0, near8, cand);
        bad += r != t && !(can && near8);
        some |= r != t;
        ++n;
      }
    // a listed type with a regular one within three corners changes for some
    bad += can && (cand >> 32) && !some;
  }
  printf("%ld %ld %ld\n", n, listed, bad);
  return 0;
}
"""


def test_only_listed_cubes_change(tmp_path):
    src = tmp_path / "probe.hip"
    src.write_text(PROBE)
    exe = tmp_path / "probe"
    r = subprocess.run(["/opt/rocm/bin/hipcc", "--offload-arch=gfx950", "-O2", "-std=c++17",
                        "-I", os.path.join(ROOT, "include"), "-I", CSRC, str(src), "-o", str(exe)],
                       capture_output=True, text=True)
    if r.returncode != 0 and "not found" in r.stderr:
        pytest.skip("hipcc not available")
    assert r.returncode == 0, r.stderr[-2000:]
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    n, listed, bad = (int(x) for x in out.stdout.split())
    # 8 types (0, 255 and the six regular ones) are never listed
    assert n == 1 << 24 and listed == 248 * 16 and bad == 0
