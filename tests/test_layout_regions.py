"""The workspace regions that hold several things at once have room for all of them: the float64 tail information and
level matrices behind the per-window records, the tree of a tile and the levels above the tiles. The layout header is compiled for
the host and asked for every size.
"""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2410_00627_amd", "csrc")

PROGRAM = r"""
#define __host__
#define __device__
#include "srtm_layout.h"
#include <cstdio>
#include <initializer_list>
using namespace srtm;
static long bad = 0, seen = 0;
static void need(bool ok, const char* what, int nx, long N, int esz) {
  ++seen;
  if (!ok && ++bad <= 10) std::printf("%s: nx %d N %ld, %d bytes\n", what, nx, N, esz);
}
static void check(int nx, int ny, long N, int esz) {
  const int nn = nx * nx, is = info_stride(nx), nlev = make_scan_plan(N).nlev, top = 63 - __builtin_clzll(N);
  const WorkLayout w = make_work_layout(nx, ny, 2, N, esz, true);
  need(w.carry + (size_t)N * is * esz <= w.btile_agg, "prior records", nx, N, esz);
  need(w.sfx + (size_t)N * is * esz <= w.stats, "information records", nx, N, esz);
  if (N > TILE) {
    need(w.sfx + tail_info_off(N, nx, esz) + sizeof(double) * is * (top + 1) <= w.stats, "tail information", nx, N, esz);
    if (esz == 4 && nx >= 2 && nx <= 4)
      need(w.carry + lev64_off(N, nx, esz) + sizeof(double) * 3 * nn * nlev <= w.btile_agg, "level matrices", nx, N, esz);
  }
  const WorkLayout f = make_work_layout(nx, ny, 2, N, esz, false);  // filter alone: the tree and the levels, no information
  if (N > TILE && esz == 4 && nx >= 2 && nx <= 4)
    need(f.carry + lev64_off(N, nx, esz) + sizeof(double) * 3 * nn * nlev <= f.stats, "level matrices, filter", nx, N, esz);
  const int64_t nf = N >> LOG_TILE;
  int q = 1;
  while (nf >> q) ++q;
  need(w.ftile_state + (size_t)tile_level_off(nf, q) * 2 * nx * esz <= w.utree, "levels above the tiles", nx, N, esz);
}
int main() {
  const int pairs[][2] = {{1, 1}, {2, 1}, {2, 2}, {3, 1}, {3, 2}, {4, 1}, {4, 2}, {6, 1}};
  for (int p = 1; p < LOG_TILE; ++p) {
    need(tree_off(p) + (TILE >> p) <= tree_off(p + 1), "levels of a tile overlap", 0, p, 0);
    need(tree_off(p + 1) <= TILE - 1, "no slot left for the flag", 0, p, 0);
  }
  for (auto& pr : pairs)
    for (int esz : {4, 8}) {
      for (long N = 1; N <= 4096; ++N) check(pr[0], pr[1], N, esz);
      for (int b = 12; b <= 26; ++b)
        for (long d = -2; d <= 2; ++d) check(pr[0], pr[1], (1L << b) + d > (1L << 26) ? 1L << 26 : (1L << b) + d, esz);
    }
  std::printf("%ld checks, %ld failed\n", seen, bad);
  return bad ? 1 : 0;
}
"""


def test_regions_have_room(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host compiler")
    src, exe = tmp_path / "regions.cpp", tmp_path / "regions"
    src.write_text(PROGRAM)
    r = subprocess.run([cxx, "-std=c++17", "-O1", "-I" + CSRC, str(src), "-o", str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
