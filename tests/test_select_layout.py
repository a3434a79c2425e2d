"""The selection's workspace arithmetic (csrc/select_layout.h), compiled for the host: whatever the number of entries and
of keys per lane, the workgroups' segments end inside the region, and they stay large enough to be of use."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2509_09754_amd", "csrc")

SEGMENTS = r"""
#include <cstdio>
#include <initializer_list>
#include "select_layout.h"
using namespace lava;
int main() {
  long long checked = 0;
  for (int keys : {2, 4, 8, kMostKeys}) {
    // a region grows at multiples of 16384 entries, the number of workgroups at multiples of 1024 * keys: both neighbours of each
    for (long long step : {16384ll, 1024ll * keys})
      for (long long at = 0; at <= 512ll * 1024 * kMostKeys; at += step)
        for (long long total = at - 1; total <= at + 1; ++total) {
          if (total < 1) continue;
          const SelectWorkspace w = select_layout(total);
          const long long nb = workgroups_for(total, keys), seg = segment_words(keys, nb, w.blk_words);
          const bool inside = nb * seg <= (long long)w.blk_words && w.off_blk + 4 * w.blk_words <= w.bytes;
          if (!inside || seg > (long long)kSegWords * keys || seg < 32 * keys) {
            std::printf("total %lld keys %d: %lld segments of %lld words, %zu in the region\n", total, keys, nb, seg, w.blk_words);
            return 1;
          }
          ++checked;
        }
  }
  std::printf("%lld\n", checked);
  return 0;
}
"""


def run(source, tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++") or shutil.which("clang++")
    if cxx is None:
        pytest.skip("no host compiler")
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(source)
    subprocess.run([cxx, "-std=c++17", "-O2", "-Wall", "-Werror", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    return subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)


def test_segments_end_inside_the_region(tmp_path):
    res = run(SEGMENTS, tmp_path)
    assert res.returncode == 0, res.stdout
    assert int(res.stdout) > 5000


SPANS = r"""
#include <climits>
#include <cstdio>
#include <initializer_list>
#include "select_layout.h"
using namespace lava;
int main() {
  long long checked = 0;
  for (int span : {64 * 2, 64 * 4, 64 * 8, 64 * kMostKeys, 64 * 32})
    for (long long total : {1ll, span - 1ll, (long long)span, span + 1ll, (1ll << 30) + 5, INT_MAX - 2ll * span, (long long)INT_MAX - span,
                            INT_MAX - span + 1ll, INT_MAX - 64ll, INT_MAX - 1ll, (long long)INT_MAX})
      for (long long base : {0ll, (total - 1) / span * span, total / span * span, (total / span > 0 ? total / span - 1 : 0) * span}) {
        if (base > INT_MAX) continue;
        if (span_complete((int)base, span, (int)total) != (base + span <= total)) return 1;
        for (long long p : {0ll, base, base + 1, base + span - 1, base + span, total - 1, total, (long long)INT_MAX})
          if (p <= INT_MAX && in_span((int)p, (int)base, span) != (p >= base && p < base + span)) return 2;
        ++checked;
      }
  std::printf("%lld\n", checked);
  return 0;
}
"""


def test_spans_at_the_end_of_31_bits(tmp_path):
    """Where a wavefront's entries end is decided without forming an index beyond 2^31 - 1."""
    res = run(SPANS, tmp_path)
    assert res.returncode == 0 and int(res.stdout) > 100, (res.returncode, res.stdout)
