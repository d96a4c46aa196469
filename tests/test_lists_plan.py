"""How lists of candidates are dealt to waves (CPU only: the plan is plain C++): every candidate belongs to exactly one wave, every
list to one workgroup's waves, and no call is sent to a launch of 2^32 threads, which cannot be made."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2507_21433_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include "rc_lists_plan.hpp"

int main() {
  const int64_t layers[] = {1, 2, 7, 48, 64, 1024, 65535}, queries[] = {1, 60, 255, 449, 1024, 4096, 65535},
                cands[] = {1, 2, 4, 5, 12, 16, 17, 24, 33, 100, 4095, 4096, 65536, (1 << 20) - 1, 1 << 20, (1 << 20) + 1},
                pools[] = {1, 100, 4096, 400000};
  long taken = 0, too_many = 0;
  for (int64_t L : layers)
    for (int64_t Q : queries)
      for (int64_t C : cands)
        for (int64_t P : pools) {
          const rc::WideLists w = rc::wide_lists(C);
          if (w.parts < 1 || w.per < 1 || w.per > 2 * w.slots || w.slots > 8 || (int64_t)w.per * (w.parts - 1) >= C || (int64_t)w.per * w.parts < C) {
            std::printf("lists of %lld: %d waves of %d\n", (long long)C, w.parts, w.per);
            return 1;
          }
          if (L * Q * w.parts >= 1 << 26) ++too_many;
          if (!rc::wide_wins(L * Q, Q, C, P, 4096)) continue;
          ++taken;
          for (int alike = 0; alike < 2; ++alike) {
            const rc::WidePlan p = rc::wide_plan(Q, C, P, L, alike);
            const int64_t grid = rc::wide_grid(p.items, p.per_xcd);
            if (grid * p.waves * 64 >= 1LL << 32 || grid < p.items || p.wgs_z * p.waves < Q * w.parts || (p.wgs_z - 1) * p.waves >= Q * w.parts ||
                p.items != L * p.wgs_z) {
              std::printf("%lld layers, %lld lists of %lld: %lld workgroups of %d waves\n", (long long)L, (long long)Q, (long long)C,
                          (long long)grid, p.waves);
              return 2;
            }
          }
        }
  return taken > 100 && too_many > 10 ? 0 : 3;
}
"""


def test_lists_are_dealt_out_once_and_fit_a_launch(tmp_path):
    src, exe = tmp_path / "plan.cpp", str(tmp_path / "plan")
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-Wall", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-I", CSRC,
                           "-o", exe, str(src)])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, f"{r.returncode}: {r.stdout}{r.stderr}"
