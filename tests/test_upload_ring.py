"""The upload ring's bookkeeping (csrc/ring.hpp) in a CPU program: the bytes behind a
returned place stay as they are until at least half of the ring (3 / 4 is the library's
own bound) has been uploaded after it, whether they were copied or found again."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2311_08050_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <deque>
#include "ring.hpp"
using inla::UploadRing;
struct Live { size_t at, bytes, total; unsigned char v; };
int main(int argc, char **argv) {
  unsigned long long seed = strtoull(argv[1], nullptr, 10);
  auto rnd = [&](unsigned m) { seed = seed * 6364136223846793005ull + 1442695040888963407ull; return (unsigned)(seed >> 33) % m; };
  UploadRing R;
  R.size = 64 * 256;
  std::vector<char> host(R.size);
  std::deque<Live> live;
  size_t total = 0, found = 0, laps = 0;
  for (int step = 0; step < 20000; ++step) {
    // a few sizes and values, so that the same bytes come again; now and then a block
    // that is not kept
    const bool keep = rnd(3) != 0;
    const size_t bytes = 1 + 200 * rnd(keep ? 4 : 20), padded = (bytes + 255) / 256 * 256;
    const unsigned char v = (unsigned char)rnd(3);
    std::vector<char> src(bytes, (char)v);
    const void *stream = (const void *)(size_t)rnd(2);
    size_t at;
    if (keep && R.find(host.data(), src.data(), bytes, stream, at)) {
      ++found;
    } else {
      if (!R.fits(padded)) { R.start_over(); ++laps; }
      at = R.take(padded, bytes, stream, keep);
      if (at + bytes > R.size) { printf("out of range\n"); return 1; }
      for (size_t i = 0; i < bytes; ++i) host[at + i] = src[i];
      total += padded;
    }
    if (keep) live.push_back({at, bytes, total, v});
    while (!live.empty() && total - live.front().total > R.size / 2) live.pop_front();
    for (const Live &l : live)
      for (size_t i = 0; i < l.bytes; ++i)
        if (host[l.at + i] != (char)l.v) { printf("overwritten %zu bytes after it was handed out\n", total - l.total); return 1; }
  }
  printf("found %zu laps %zu\n", found, laps);
  return found > 1000 && laps > 50 ? 0 : 1;
}
"""


@pytest.mark.parametrize("seed", [1, 2, 3])
def test_places_outlive_half_a_ring(tmp_path, seed):
    cxx = shutil.which("g++") or shutil.which("c++")
    assert cxx, "a C++ compiler"
    src, exe = tmp_path / "ring.cpp", tmp_path / "ring"
    src.write_text(PROGRAM)
    subprocess.run([cxx, "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe), str(seed)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
