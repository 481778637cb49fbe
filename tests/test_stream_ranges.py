"""The arithmetic that deals the streaming GEMM's items to its workgroups, on
the CPU: the kernel's own function (range_from, which the host can call too)
in 32 and in 64 bits, against the definition."""
import os
import shutil
import subprocess

import pytest

from paper_2608_13057_amd import build

SRC = r"""
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>
#include "gemm_stream.h"
using namespace tempo::gemm;

static std::mt19937_64 rng(11);
static int ri(int lo, int hi) { return lo + (int)(rng() % (unsigned long long)(hi - lo + 1)); }
#define CHECK(c, ...) do { if (!(c)) { printf("line %d: ", __LINE__); printf(__VA_ARGS__); printf("\n"); exit(1); } } while (0)

template <int BM>
static void one(int S, int maxrows, int my_nb, int C, int whole, int wpx, bool define) {
  std::vector<int32_t> off(S + 1, 0), cnt(S, 0), sw(S + 1, 0);
  for (int s = 0; s < S; s++) {
    cnt[s] = ri(0, 3) ? ri(0, maxrows) : 0;
    const int nt = (cnt[s] + BM - 1) / BM;
    off[s + 1] = off[s] + nt * BM;
    sw[s + 1] = sw[s] + (nt ? (nt - 1) * tile_weight<BM>(BM) + tile_weight<BM>(cnt[s] - (nt - 1) * BM) : 0);
  }
  Geo g{};
  g.C = C;
  g.RC = whole ? C : 1;
  g.my_nb = my_nb;
  g.wpx = wpx;
  g.items = off[S] / BM * my_nb;
  auto first = [&](auto unit, auto T) {
    int n = 0;
    for (int s = 0; s < S; s++) n += unit * sw[s + 1] <= T;
    return n;
  };
  const long long unit = (long long)my_nb * (C / g.RC), total = unit * sw[S];
  const bool fits = total * wpx < (1ll << 31);
  // the weight before every range unit, for small cases
  std::vector<long long> pre;
  if (define) {
    pre.push_back(0);
    for (int s = 0; s < S; s++)
      for (int r = 0; r < cnt[s]; r += BM)
        for (long long u = 0; u < unit; u++) pre.push_back(pre.back() + tile_weight<BM>(std::min(BM, cnt[s] - r)));
    CHECK(pre.back() == total, "total");
  }
  int prev = 0;
  for (int j = 0; j <= wpx; j++) {
    const int q = range_from<BM, long long>(g, j, off.data(), cnt.data(), sw.data(), S, first);
    if (fits) {
      const int q32 = range_from<BM, int>(g, j, off.data(), cnt.data(), sw.data(), S, first);
      CHECK(q32 == q, "32 bits %d, 64 bits %d (S %d nb %d C %d wpx %d j %d)", q32, q, S, my_nb, C, wpx, j);
    }
    CHECK(q >= prev && q <= g.items * C && q % g.RC == 0, "order: %d after %d", q, prev);
    if (j == 0) CHECK(q == 0, "start %d", q);
    if (j == wpx) CHECK(q == g.items * C, "end %d of %d", q, g.items * C);
    if (define && j > 0 && j < wpx) {
      // the smallest unit whose weight prefix reaches j / wpx of the total
      const long long T = total * j / wpx;
      size_t n = 0;
      while (n + 1 < pre.size() && pre[n] < T) n++;
      CHECK(q == (int)n * g.RC, "definition: unit %zu, got %d / %d", n, q, g.RC);
    }
    prev = q;
  }
}

template <int BM>
static void all() {
  for (int k = 0; k < 3000; k++) {
    const int C = ri(1, 2);
    one<BM>(ri(1, 12), ri(1, 5 * BM), ri(1, 6), C, ri(0, 1), ri(1, 40), true);
  }
  for (int k = 0; k < 3000; k++) {  // products on both sides of 2^31
    const int S = ri(1, 256), wpx = ri(0, 1) ? 32 : 256;
    one<BM>(S, ri(1, 40 * BM), ri(1, 1 << ri(1, 12)), ri(1, 2), ri(0, 1), wpx, false);
  }
}

int main() {
  all<64>();
  all<128>();
  all<192>();
  all<256>();
  printf("ok\n");
  return 0;
}
"""


def test_range_arithmetic(tmp_path):
    """Ranges of 1 .. 256 slots (empty ones and ragged last tiles among them),
    by chunks and by whole items: they tile the items in order, each boundary
    is the one of the definition (small cases), and the 32-bit form, used where
    every product is below 2^31, gives what the 64-bit one does right up to
    there."""
    if not os.path.exists(build.HIPCC) and shutil.which("hipcc") is None:
        pytest.skip("hipcc not available")
    src = tmp_path / "ranges.hip"
    src.write_text(SRC)
    exe = tmp_path / "ranges"
    subprocess.run([build.HIPCC, "-O1", "-std=c++17", "--offload-arch=gfx950", "--offload-host-only", "-Wno-unused-result",
                    "-I", build.CSRC, str(src), "-o", str(exe)], check=True, capture_output=True, timeout=300)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout
