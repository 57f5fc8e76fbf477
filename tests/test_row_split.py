"""What the short-row kernels read of a row, from the header they take it from, compiled for the
host and walked over every offset within 16 bytes and every length (CPU only).

An fp32 row is read as its own entries, each exactly once; the ABI promises readable memory around
a row for bf16 alone, whose rows are read as the aligned 16-byte chunks that cover them."""
import subprocess

from paper_2605_12070_amd import build as B

PROGRAM = r"""
#include <cstdio>
#include <cstring>
#include "row_split.h"
using namespace dppo;

template <typename Tin>
int walk() {
  constexpr int E = 16 / (int)sizeof(Tin);
  alignas(16) static Tin buf[8192];
  static int seen[8192];
  for (int off = 0; off < E; ++off)
    for (int V = 1; V <= 6145; V += V < 600 ? 1 : 61) {
      const Tin* row = buf + E + off;
      const WaveSpan w = wave_span(row, V);
      std::memset(seen, 0, sizeof(seen));
      int low = V, high = 0;                     // entries of memory read, relative to the row
      const int n = w.bytes / (int)sizeof(Tin);
      if (n > 0) {
        low = w.first;
        high = w.first + n;
        if ((uintptr_t)(row + w.first) % 16 != 0 || w.bytes % 16 != 0) return 1;
      }
      for (int k = w.lo; k < w.hi; ++k) {
        const int e = w.first + k;
        if (k >= n || e < 0 || e >= V) return 2; // an entry of another row taken for this one's
        ++seen[e];
      }
      const RowSplit sp{w.first, w.bytes / 16, w.nedge};
      for (int i = 0; i < w.nedge; ++i) {
        const int e = sp.template entry<E>(i);
        if (e < 0 || e >= V) return 3;
        ++seen[e];
        low = e < low ? e : low;
        high = e + 1 > high ? e + 1 : high;
      }
      for (int e = 0; e < V; ++e)
        if (seen[e] != 1) return 4;
      if (sizeof(Tin) == 4 && (low < 0 || high > V)) return 5;
      if (sizeof(Tin) == 2 && (low <= -E || high >= V + E)) return 6;
      // an fp32 chunk is the row's as a whole or not at all
      if (sizeof(Tin) == 4 && (w.lo != 0 || w.hi != n || w.nedge > 2 * (E - 1))) return 7;
    }
  return 0;
}

int main() {
  std::printf("%d %d\n", walk<float>(), walk<uint16_t>());
  return 0;
}
"""


def test_short_rows_read_their_own_entries(tmp_path):
    src = tmp_path / "walk.hip"
    src.write_text(PROGRAM)
    exe = tmp_path / "walk"
    subprocess.run([B.hipcc(), *B.FLAGS, str(src), "-o", str(exe)], check=True, capture_output=True)
    assert subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split() == ["0", "0"]
