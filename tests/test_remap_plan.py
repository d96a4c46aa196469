"""How a layer's table and reference counts are dealt to workgroups (CPU only: the plan is plain C++): every item belongs to
exactly one share, and a share that starts past the last item is empty rather than negative, for every count of blocks."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2507_21433_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "rc_remap_plan.hpp"

static long empty_shares;
static void check(int64_t n, int64_t G, const char* what, int64_t L, int64_t RE) {
  const int length = (int)rc::share_length(n, G);
  int64_t next = 0;
  for (int64_t g = 0; g < G; ++g) {
    const int first = (int)(g * length), items = rc::share_items((int)n, first, length);
    if (items < 0 || items > length || (items > 0 && first != next) || (items == 0 && next != n)) {
      std::printf("%s: %lld layers, %lld entries, %lld items, share %lld: %d items at %d\n", what, (long long)L, (long long)RE,
                  (long long)n, (long long)g, items, first);
      std::exit(1);
    }
    empty_shares += items == 0;
    next += items;
  }
  if (next != n) std::exit(2);
}

int main() {
  const int64_t layers[] = {1, 2, 3, 8, 9, 16, 40, 64, 127, 128}, entries[] = {1, 288, 4096, 8191, 8192, 12289, 16384, 49152, 49664, 65536, 100000, 131072};
  for (int64_t L : layers)
    for (int64_t RE : entries) {
      const int64_t G = rc::chunks_per_layer(RE, L);
      if (G < 1) return 3;
      check(RE, G, "table", L, RE);
      if (L <= 64 && empty_shares) return 4;  // chunks of the table are long: none is empty
      const long before = empty_shares;
      for (int64_t NB = 0; NB < 4200; ++NB) check(NB, G, "counts", L, RE);
      check(50176, G, "counts", L, RE);
      if (RE == 131072 && L <= 8 && empty_shares == before) return 5;  // the range that has empty shares is in the test
      empty_shares = 0;
    }
  return 0;
}
"""


def test_shares_cover_a_layer_once(tmp_path):
    src, exe = tmp_path / "plan.cpp", str(tmp_path / "plan")
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-Wall", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-I", CSRC,
                           "-o", exe, str(src)])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, f"{r.returncode}: {r.stdout}{r.stderr}"
