"""Rules of rip_launch_policy.h for short launches and groups above eight,
built and run on the CPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <initializer_list>
#include "rip_launch_policy.h"
using namespace rip::policy;
int bad = 0;
#define CHECK(x) do { if (!(x)) { std::printf("failed: %s\n", #x); ++bad; } } while (0)
int main() {
  for (int k = kMaxK + 1; k <= 256; ++k)
    for (int64_t work : {1, 255, 256, 257, 513, 2048, 4096, 4097, 16384, 16385, 1 << 20})
      for (int mom = 0; mom < 2; ++mom) {
        for (int form = 0; form < 4; ++form) {
          const bool bf16 = form & 1, updates = form & 2;
          const WidePlan p = wide_plan(k, work, bf16, mom, updates);
          CHECK(p.waves >= 1 && p.waves <= kWideWaves);
          CHECK(p.per_cu >= 1 && p.per_cu * p.waves <= 32);
          CHECK(p.per_cu == 1 || p.per_cu % 2 == 0);
          CHECK(most_blocks(p.waves) >= 1 && most_blocks(p.waves) * p.waves * 64 <= 1ll << 31);
          for (int j = 1; j <= k; ++j) {  // every unit of the launch
            const int c = wide_share(j, p.waves);
            CHECK(c >= 1 && c <= kWideC);
            const int rounds = (j + kWideC * p.waves - 1) / (kWideC * p.waves);
            CHECK(c * p.waves * rounds >= j);
          }
          // where workgroups share a CU the registers hold two of them (16 waves
          // in the largest variant), and all of them where three waves will do;
          // long launches count on no more
          const int64_t all = (work + 2 * kCus - 1) / (2 * kCus) * 2;
          CHECK(work <= kCus || p.waves <= 8 || (mom && k > 64));
          if (work > kCus && k > 16 && k <= 64 && all * 3 <= wide_resident(bf16, mom))
            CHECK(all * p.waves <= wide_resident(bf16, mom));
          CHECK(work <= 4 * kLongWide || p.waves * p.per_cu <= 16);
          CHECK(work <= kLongWide || !mom || p.waves * p.per_cu <= 16);
        }
      }
  // a group with momentum of which up to a fifth of the members update streams
  // like one that averages and takes that plan; 25 to 32 members of which some
  // update, that of short launches
  for (int k = kMaxK + 1; k <= 256; ++k)
    for (int64_t work : {16 * kCus + 1, 64 * kCus + 1, 256 * kCus + 1, 1 << 20})
      for (int bf16 = 0; bf16 < 2; ++bf16) {
        const WidePlan q = wide_plan(k, work, bf16, false, 0.0);
        for (int act = 0; act <= k; ++act) {
          const double share = (double)act / k;
          const WidePlan p = wide_plan(k, work, bf16, true, share);
          CHECK(p.waves >= 1 && p.per_cu >= 1 && p.waves * p.per_cu <= 16);
          if (act * 5 <= k) CHECK(p.waves == q.waves && p.per_cu == q.per_cu);
          if (k > 24 && k <= 32 && act * 5 > k && act * 4 <= k * 3) CHECK(p.waves == (k + 3) / 4);
        }
      }
  // short launches: all workgroups at once up to 16 per CU whatever the units
  // prefer and whatever they store, and never a higher cap for a longer launch
  for (int cap = 2; cap <= 12; cap += 2)
    for (int bf16_mom = 0; bf16_mom < 2; ++bf16_mom) {
      int last = kAllWaves;
      for (int64_t work = 1; work <= 100 * kCus; work += work < 2600 ? 1 : 17) {
        const int c = short_cap(cap, work, bf16_mom);
        CHECK(c >= cap && c <= last);
        CHECK(work > 16 * kCus || c == kAllWaves);
        CHECK(work <= 16 * kCus || c == cap || (cap >= 8 && cap <= 10 && c == kShortWaves));
        CHECK(work <= 80 * kCus || c == cap);
        last = c;
      }
    }
  CHECK(short_cap(10, 40 * kCus, true) == 12 && short_cap(10, 60 * kCus, true) == 10);
  CHECK(short_cap(10, 60 * kCus, false) == 12);
  CHECK(short_cap(10, 100 * kCus, false, true) == 12 && short_cap(10, 230 * kCus, false, true) == 10);
  CHECK(short_cap(10, 100 * kCus, false, false) == 10);
  // separate tensors: more waves where flat replicas lost them, never fewer
  for (int mom = 0; mom < 2; ++mom)
    for (int k = 1; k <= kMaxK; ++k)
      for (int act = 0; act <= k; ++act) {
        const int32_t ks[] = {k, k}, as[] = {act, k};
        CHECK(launch_waves(ks, as, 2, mom, true) >= launch_waves(ks, as, 2, mom));
      }
  {
    const int32_t one[] = {1}, two[] = {2}, three[] = {3}, seven[] = {7}, none[] = {0};
    CHECK(launch_waves(one, one, 1, false, true) == 12);
    CHECK(launch_waves(two, none, 1, false, true) == 14);
    CHECK(launch_waves(three, none, 1, false, true) == 10);
    CHECK(launch_waves(seven, none, 1, false, true) == 8);
  }
  // a short step stays one launch, whatever its units prefer
  {
    const int32_t k[] = {8, 2, 1, 1};
    for (int mom = 0; mom < 2; ++mom) {
      CHECK(step_bytes(k, k, 4, mom, 4000) == 12 * (mom ? 20000.0 : 12000.0));
      CHECK(!long_enough_to_split(step_bytes(k, k, 4, mom, 4 * 1200000)));
      CHECK(long_enough_to_split(step_bytes(k, k, 4, mom, 4 * 8000000)));
    }
    const int32_t none[] = {0, 0, 0, 0};
    CHECK(step_bytes(k, none, 4, false, 1000) == 24000);
  }
  std::printf(bad ? "%d failed\n" : "ok\n", bad);
  return bad != 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_short_launches_and_wide_plans(tmp_path):
    src, exe = tmp_path / "p.cpp", tmp_path / "p"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-I",
                    os.path.join(ROOT, "paper_1909_08029_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True, timeout=120)
    res = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0, res.stdout
