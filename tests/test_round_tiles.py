"""Rows per tile of a screened round: small rounds make enough tiles, none more than fit."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SRC = r'''
#include <stdio.h>
#include <random>
#include <vector>
#include "host_limits.h"
using namespace sieve;
static int64_t tiles(const std::vector<int>& c, const std::vector<int>& len, int g, int chunk) {
  int64_t t = 0;
  for (size_t p = 0; p < c.size(); ++p)
    t += (int64_t)((c[p] + g - 1) / g) * ((len[p] + chunk - 1) / chunk);
  return t;
}
int main() {
  std::mt19937 r(7);
  int splits = 0;
  for (int it = 0; it < 20000; ++it) {
    const int nlist = 1 + (int)(r() % (it % 2 ? 40u : 900u)), g = (int[]){64, 112, 128}[r() % 3];
    std::vector<int> len(nlist), c(nlist, 0);
    int64_t n = 0, items = 0, mx = 0;
    for (int& x : len) {
      x = (int)(r() % (1u << (r() % 15)));
      n += x;
      if (x > mx) mx = x;
    }
    const int touched = 1 + (int)(r() % nlist);
    for (int p = 0; p < touched; ++p) {
      c[(size_t)((p * 7919ll) % nlist)] += 1 + (int)(r() % (1u << (r() % 10)));
    }
    for (int x : c) items += x;
    const int chunk0 = (int[]){1024, 2048, 4096, (int)((mx + 127) / 64 * 64)}[r() % 4];
    // the workspace's size: the bound of whole chunks and some more
    const int64_t cap = round_tile_bound(items, 64, chunk0, nlist, n, mx) + (r() % 3) * 100;
    const int chunk = screen_rows_per_tile(chunk0, 256, items, g, nlist, n, mx, cap);
    if (chunk > chunk0 || chunk < 64 || chunk % 64) return 1;
    if (tiles(c, len, g, chunk) > cap) return 2;
    if (tiles(c, len, g, chunk) > round_tile_bound(items, g, chunk, nlist, n, mx)) return 3;
    splits += chunk < chunk0;
  }
  if (splits < 1000) return 4;
  // few lists, few queries: about a tile per work-group, and none of 64 rows
  for (int nlist = 1; nlist <= 300; ++nlist)
    for (int len : {100, 312, 781, 1517, 2145, 9000})
      for (int chunk0 : {1024, 4096, 16384}) {
        const int chunk = screen_rows_per_tile(chunk0, 256, nlist * 100ll, 128, nlist,
                                               (int64_t)nlist * len, len, 1 << 20);
        const int64_t t = (int64_t)nlist * ((len + chunk - 1) / chunk);
        if (2 * t < 200 && chunk > 320 && len > 320) return 5;
        if (t > 256 && chunk < chunk0) return 9;  // one tile per work-group
        if (chunk < 128 && chunk < chunk0) return 6;
      }
  // a round that fills the chip keeps its chunk
  if (screen_rows_per_tile(2048, 512, 65536, 128, 1024, 1000000, 1300, 1 << 20) != 2048) return 8;
  puts("ok");
  return 0;
}
'''


def test_rows_per_tile(tmp_path):
    src = tmp_path / "tiles.cpp"
    src.write_text(SRC)
    exe = tmp_path / "tiles"
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-I",
                    os.path.join(ROOT, "paper_2608_03199_amd", "csrc"), str(src), "-o",
                    str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0 and out.stdout.strip() == "ok", out.returncode
