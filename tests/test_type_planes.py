"""The library's bit-plane helpers (shared by its kernels, compiled here for
the host): a row's planes and types are each other's transpose, a cube has
triangles unless its type is 0 or 255, and the edges a row of cubes uses by
its types' corner bits are exactly those the marching-cubes table uses, for
every type at every place of a row and next to every type of the -x row."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1803_03949_amd", "csrc")

PROBE = r"""
#include <stdio.h>
#include "vm_internal.h"
#include "vm_tables.hip"
using namespace vm;
static uint8_t tri[256 * 16], uses[256 * 12];
// planes of a row of eight types
static void planes(const uint8_t* t, uint32_t& lo, uint32_t& hi) {
  lo = hi = 0;
  for (int k = 0; k < 8; ++k)
    for (int x = 0; x < 8; ++x) {
      const uint32_t b = (uint32_t)((t[x] >> k) & 1);
      (k < 4 ? lo : hi) |= b << (8 * (k & 3) + x);
    }
}
int main() {
  build_mc_tables(tri, uses);
  long bad = 0, rows = 0;
  uint32_t seed = 1;
  for (int round = 0; round < 1 << 18; ++round) {
    uint8_t t[8], back[8];
    for (int x = 0; x < 8; ++x) {
      // every type at every place, then random rows with many empty cubes
      seed = seed * 1664525u + 1013904223u;
      t[x] = round < 2048 ? (uint8_t)(x == (round & 7) ? round >> 3 : 0)
                          : ((seed >> 24) & 1 ? (uint8_t)(seed >> 16) : (seed >> 25) & 1 ? 255 : 0);
      back[x] = (uint8_t)(seed >> 8);
    }
    uint32_t lo, hi, xlo, xhi, next, diag, tl, th;
    planes(t, lo, hi);
    planes(back, xlo, xhi);
    tl = lo, th = hi;
    transpose8(tl, th);
    const uint32_t surf = surface_cubes(lo, hi);
    uint32_t want[3] = {0, 0, 0}, wn[4] = {0, 0, 0, 0}, wd = 0;
    for (int x = 0; x < 8; ++x) {
      bad += (((x < 4 ? tl : th) >> (8 * (x & 3))) & 255u) != t[x];
      bad += planes_type((uint64_t)hi << 32 | lo, x) != t[x];
      bad += ((surf >> x) & 1u) != (tri[t[x] * 16] != 0);
      const uint8_t* u = uses + 12 * t[x];
      const uint8_t* p = uses + 12 * (x > 0 ? t[x - 1] : back[7]);
      want[0] |= (uint32_t)(u[0] != 0) << x;
      want[1] |= (uint32_t)(u[3] || p[1]) << x;
      want[2] |= (uint32_t)(u[8] || p[9]) << x;
      wn[0] |= (uint32_t)(u[2] != 0) << x;          // (y + 1, z): x edges
      wn[1] |= (uint32_t)(u[11] || p[10]) << x;     // and z edges
      wn[2] |= (uint32_t)(u[4] != 0) << x;          // (y, z + 1): x edges
      wn[3] |= (uint32_t)(u[7] || p[5]) << x;       // and y edges
      wd |= (uint32_t)(u[6] != 0) << x;             // (y + 1, z + 1): x edges
    }
    transpose8(tl, th);
    bad += tl != lo || th != hi;
    const uint32_t own = row_edges(lo, hi, xlo, xhi, &next, &diag);
    bad += own != (want[0] | want[1] << 8 | want[2] << 16);
    bad += next != (wn[0] | wn[1] << 8 | wn[2] << 16 | wn[3] << 24);
    bad += diag != wd;
    ++rows;
  }
  printf("%ld %ld\n", rows, bad);
  return 0;
}
"""


def test_row_helpers_match_the_marching_cubes_table(tmp_path):
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
    rows, bad = (int(x) for x in out.stdout.split())
    assert rows == 1 << 18 and bad == 0
