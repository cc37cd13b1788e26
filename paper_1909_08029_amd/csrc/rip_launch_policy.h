// Residency cap of one fused-kernel launch (resident waves per CU, enforced
// by the host with an LDS reservation), chosen from the units the launch
// runs.  Plain host code with no HIP dependency, so it is tested on its own.
#pragma once

#include <cmath>
#include <cstdint>

namespace rip {
namespace policy {

constexpr int kMaxK = 8;   // largest group size with a specialized kernel path
constexpr int kCus = 256;  // compute units of an MI355X

// Resident waves per CU at which each unit shape sustained the most HBM
// bandwidth on MI355X, by group size k (1 to kMaxK; larger groups have a kernel
// of their own and take wide_plan below), for units whose members all update
// (plain SGD, momentum) and for units that only average.  Measured with bench.py
// --sweep-caps (32 fp32 replicas of 25.6M parameters, every unit of one size,
// even caps of 2-16 waves/CU, one process per shape; two sessions on different
// machines agreed) and again in replayed graphs on 14-16 replicas of 16.8M.
// With the kernel's shorter way to a wave's first load some shapes peak two
// waves lower than before (replicas of 25.6M, before -> after: lone updates 781
// -> 773 us at 12 -> 10, groups of seven 1380 -> 1333 at 8 -> 6, with momentum
// 1747 -> 1716 and groups of six 1475 -> 1464 at 6 -> 4; averaging only, triples
// 583 -> 572 at 10 -> 8).  A lane keeps one 16-byte load in flight per slot of
// every stream it reads (w, plus g and v when the member updates), so units that
// read more streams peak with fewer resident waves; beyond that, more waves add
// outstanding requests without adding bandwidth (GB/s, plain SGD group of eight
// at 6 / 8 / 10 waves: 6246 / 5937 / 5892; momentum group of three at 4 / 6 / 8:
// 4697 / 5154 / 6028).  Where two caps measured within 1%, the table takes the
// one that also suited the mixed launches of the paper's schedules.  Odd caps
// measured the same as the even cap below them (the LDS reservation appears to
// be granted per half of a CU's LDS), so only even caps are used.  bf16 units (8
// replicas of 1.3G parameters) peaked at the same caps within 2%, except
// averaging-only groups of eight, which ran 5% faster at 6 than at 8 (fp32:
// equal).
constexpr int kWavesSgd[kMaxK + 1] = {0, 10, 10, 8, 10, 8, 8, 6, 6};
constexpr int kWavesMom[kMaxK + 1] = {0, 10, 10, 10, 8, 6, 4, 4, 4};
constexpr int kWavesAvg[kMaxK + 1] = {0, 12, 12, 8, 12, 10, 8, 6, 6};
// Handles of several segments (separate layer tensors) need more waves for some
// shapes: a wave first finds its segment, a chain of scalar loads that flat
// replicas don't have, and lanes of a tensor's last tile have nothing to load.
// On the layer tensors of networks of 1M to 90M elements (44 to 70 handles of
// 6 to 161 tensors each; time above the best cap, flat entry -> this one): lone
// updates 2.9% -> 0.2, averaging only, pairs 2.7 -> 0.5, triples 1.6 -> 0.5,
// groups of seven 7.9 -> 0.0 (flat: 0.2 -> 1.1, 0.0 -> 2.7, 0.1 -> 1.4 and 0.1
// -> 2.2).
constexpr int seg_waves_sgd(int k) { return k == 1 ? 12 : kWavesSgd[k]; }
constexpr int seg_waves_avg(int k) {
  return k == 2 ? 14 : k == 3 ? 10 : k == 7 ? 8 : kWavesAvg[k];
}

// The cap used when a launch has no units (nothing is launched then).
constexpr int kWavesDefault = 8;

// Preferred cap of one unit of k members of which `act` update this step:
// the averaging-only and all-updating preferences, interpolated by the share
// of updating members.  `segs`: the handle has several segments.
inline double unit_waves(int32_t k, int32_t act, bool mom, bool segs = false) {
  const double f = (double)act / (double)k;
  const int sgd = segs ? seg_waves_sgd(k) : kWavesSgd[k];
  const int avg = segs ? seg_waves_avg(k) : kWavesAvg[k];
  return f * (mom ? kWavesMom[k] : sgd) + (1.0 - f) * avg;
}

// Cap of a launch running `units` units (unit u: k[u] members, act[u] of them
// updating; mom: the launch applies momentum).  The units' preferences are
// averaged, weighted by the bytes each moves (an updating member moves w, g
// and v; an averaging one w), and the mean is rounded up to an even cap: a cap
// below a shape's preference cost more (SGD groups of 2-4 at 8 waves: -3%)
// than one above it (groups of 5-8 at 10: -1%).
inline int launch_waves(const int32_t* k, const int32_t* act, int32_t units, bool mom,
                        bool segs = false) {
  double num = 0.0, den = 0.0;
  for (int32_t u = 0; u < units; ++u) {
    const double bytes = act[u] * (mom ? 5.0 : 3.0) + (k[u] - act[u]) * 2.0;
    num += unit_waves(k[u], act[u], mom, segs) * bytes;
    den += bytes;
  }
  if (den == 0.0) return kWavesDefault;
  return 2 * (int)std::ceil(num / den / 2.0 - 1e-6);
}

// A launch of at most this many one-slot tiles (four waves per CU) takes
// one-slot tiles for every unit: more waves, each with fewer loads and less
// code to fetch, finish sooner while the chip is not full.  (8 fp32 replicas
// of 10,007 in pairs: 2.5 us with two slots, 2.0 with one; with momentum 3.0
// and 2.2; lone bf16 updates with momentum 3.1 with four slots, 2.3 with one.
// Pairs of 80,007, 1252 tiles: 3.5 and 3.8; of 160,007, 2500 tiles: 4.4, 5.1.)
constexpr int kOneSlotWork = 1024;

// The cap of a launch of `work` workgroups (one wave each) whose units prefer
// `cap`.  The preferences are those of long launches; a short one is bound by
// how its waves fall into rounds.  Up to 16 per CU, which the registers of
// every variant of the kernel allow, all of them start at once.  (1182 random
// launches of 3 to 16 workgroups per CU, groups of 1 to 8, both types, each
// timed at caps of 4 to 20; mean over the launches of the time above the best
// cap of each: at the preference 4.4%, at 12 1.7%, at 16 0.6%, at 20 0.6%.
// Groups of eight with momentum of 196,608 11.5 us at the preference, 9.4 at
// 16; pairs of 753,664 bf16 with it, 12 per CU, 11.3 at 10, 10.5 at 14.)
// Beyond, launches that prefer 8 take 12 up to 24 per CU (83 launches: 1.9%
// above the best at 8, 1.6 at 12; 16 replicas of 304,327 in 59 tensors, groups
// of four with momentum, 17.3 us and 16.9), and launches that prefer 10 take
// 12 up to 80 per CU, or 48 for bf16 with momentum (524 launches of 16 to 80:
// 2.1% above the best at 10, 1.2 at 12, 2.2 at 16; lone updates of 2.6M 39.0 us
// and 37.9; bf16 with momentum up to 48: 2.0% and 0.7, from 48 to 80 1.1 and
// 1.6).  Plain lone updates, four slots
// per wave and so the fewest waves, take 12 up to 220 per CU (61 launches of 90
// to 220: 1.0% above the best at 10, 0.1 at 12; 35 of 220 to 400: 0.3 and 0.5).
// The lower preferences hold as they are (333 launches of 16 to 80: 1.5%, at 12
// 3.6).
constexpr int kAllWaves = 16;
constexpr int kShortWaves = 12;
inline int short_cap(int cap, int64_t work, bool bf16_mom, bool lone_sgd = false) {
  const int64_t per_cu = (work + kCus - 1) / kCus;
  if (per_cu <= kAllWaves) return cap > kAllWaves ? cap : kAllWaves;
  const int64_t most = cap == 10 ? (bf16_mom ? 48 : lone_sgd ? 220 : 80) : (cap == 8 ? 24 : 0);
  return per_cu <= most ? kShortWaves : cap;
}

// The wide kernel's launch (units above kMaxK members): waves per workgroup
// and workgroups per CU.
constexpr int kWideWaves = 16;  // most waves of a workgroup
constexpr int kWideC = 4;       // most members a wave holds at once
// Most waves of a wide launch that also takes a step's smaller units, most of
// whose waves have no member (a second launch costs about 2 us; a group of 16
// beside a lone update of 300,077, 9.4k waves: 11.2 us, 13.7 as two launches;
// 32 beside 8 of 80,077 with momentum, 22k waves: 18.0, 15.2 as two).
constexpr int kWideAllWaves = 10240;

struct WidePlan {
  int waves, per_cu;
};

// Waves of the wide kernel that a CU's registers hold (61, 77, 86 and 104 VGPRs).
constexpr int wide_resident(bool bf16, bool mom) { return bf16 ? (mom ? 16 : 20) : (mom ? 24 : 32); }

// Short launches, up to 16 workgroups per CU (SGD: 64): four members per wave
// as far as the waves go: eight waves, or sixteen when every workgroup has a CU
// to itself, where only the latency of a workgroup counts (256 bf16 replicas of
// 65,539: 28.8 us with sixteen, 38.4 with eight), or for more than 64 members
// with momentum.  (For 33 to 64 with it, nine to sixteen waves left one
// workgroup on a CU: 57 random launches of 1 to 16 workgroups per CU 17% above
// the best plan of each, 5% with eight.)  Sixteen waves share a CU (fp32 groups
// of 16, 10M: 325 us at 16, 342 at 12, 338 at 20-24); workgroups of three waves
// go four to a CU, as in long launches.  A cap that all workgroups fit under,
// to 32 waves, is lifted to that (24 fp32 replicas of 150,077, four workgroups
// of six waves per CU, 7.3 us, 9.7 at two); groups of 17 to 64 whose waves the
// registers do not hold that many of take fewer, down to three, so that they do
// (78 random launches: 6% less time; more members gained nothing, 9 to 16
// fit).
//
// Longer launches are bound by the streams open at once, and more waves lose
// what they gain in latency.  1752 random launches (9 to 256 members, 0.5 to
// 2900 workgroups per CU, both types), each timed with 10 to 30 plans; of those
// above 64 per CU, time above the best plan of each, four members a wave on
// eight or sixteen waves -> this plan: SGD, 13 to 24 members 3.3% -> 1.9, 25 to
// 28 2.6 -> 0.6 (31 and 32: six waves 0.7 behind eight); averaging, 21 to 24
// 11 -> 0.9; momentum, 9 to 12 2.0 -> 0.8, 13 to 24 4.0 -> 1.2, 25 to 64
// 3.2 -> 1.2, bf16 25 to 32 above 256 per CU, at four waves, 0.8 -> 0.7, at
// three 2.2 (single waves that took the members in chunks of eight, all
// workgroups capped at four per CU, 3 to 5%).  Averaging, 28 to 32 up to 256
// per CU, stays as in short launches (four waves, four workgroups: +1 to +3%).  Between 16
// and 64 per CU momentum gains (33 to 64 members 3.9%, 13 to 24 1.8%), SGD does
// not (13 to 24 +0.0%, up to 8% slower).  Replicas at a pitch of a power of two
// (64 MiB and more) stay up to 20% behind those single waves.
//
// Workgroups per CU are even (an odd count gets the residency of the even one
// below).
//
// `share`: the part of the members that update.  Up to a fifth, most streams are
// read and written only, and the averaging plan suits them (All-Reduce with a
// straggler: one of 32 fp32 replicas of 25.6M updating, with momentum: 1344 us at
// three waves, 1193 at eight).  Over 37,000 random launches above 16 workgroups
// per CU, time with the updating plan against the averaging one, a sixth updating
// or fewer: momentum, 9 to 16 members +4 to +6%, 17 to 20 +5, 25 to 32 +8 to +20,
// 33 to 64 +6; SGD, 13 to 16 +5, 25 to 28 +6 to +8; a third updating, 9 to 24 with
// momentum -2 to -4%.  (More than 64 with momentum, up to 4 per CU: +31% on
// sixteen waves, one or none in ten updating.)  Groups of 25 to 32 stay as in
// short launches up to three quarters (half of them updating with momentum, tensors
// allocated one by one, 64 to 256 per CU: 4 to 6% less time than on the updating
// plan, more 2 to 5%).  From 256 per CU on averaging groups of 28 to 64 take three
// waves (tensors one by one, against eight: 28 to 32 5% less, 33 to 64 2 to 4% less;
// rows of one buffer 0 to 2%; between 64 and 256 the two layouts differ in sign).
constexpr int64_t kLongWide = 16 * kCus;  // workgroups
inline WidePlan wide_plan(int32_t kmax, int64_t work, bool bf16, bool mom, double share) {
  WidePlan p;
  const bool updates = share > 0.2;
  if (work > (mom || !updates ? kLongWide : 4 * kLongWide) &&
      !(updates && share <= 0.75 && kmax > 24 && kmax <= 32)) {
    if (mom && updates)
      return kmax <= 12 ? WidePlan{2, 6} : kmax <= 24 ? WidePlan{2, 4}
             : kmax <= 32 && bf16 ? WidePlan{4, 2}
             : kmax <= 64 ? WidePlan{3, 2} : WidePlan{kWideWaves, 1};
    if (kmax <= 12 || (updates && kmax <= 24)) return WidePlan{3, 4};
    if (kmax <= (updates ? 28 : 27)) return updates ? WidePlan{6, 2} : WidePlan{4, 4};
    if (!updates && kmax <= 64 && work > 16 * kLongWide) return WidePlan{3, 4};
    if (updates || kmax > 32) return WidePlan{kWideWaves / 2, 2};
  }
  const int most = work <= kCus || (mom && updates && kmax > 64) ? kWideWaves : kWideWaves / 2;
  p.waves = (kmax + kWideC - 1) / kWideC;
  if (p.waves > most) p.waves = most;
  const auto even = [](int64_t n) { return n < 2 ? n : (n + 1) / 2 * 2; };
  p.per_cu = (int)(p.waves == 3 ? 4 : even(16 / p.waves));
  const int64_t all = even((work + kCus - 1) / kCus);
  const int64_t fit = wide_resident(bf16, mom) / all;
  if (kmax > 16 && kmax <= 64 && p.waves > fit && fit >= 3) p.waves = (int)fit;
  if (all > p.per_cu && all * p.waves <= 32) p.per_cu = (int)all;
  return p;
}

// Most workgroups of `waves` waves in one launch: 2^31 work-items, within the
// dispatch's 32-bit grid size.
constexpr int64_t most_blocks(int waves) { return ((int64_t)1 << 25) / (waves > 1 ? waves : 1); }

// Members per wave and round of a unit of k members on `waves` waves: the
// rounds' members split evenly.
inline int wide_share(int32_t k, int waves) {
  const int rounds = (k + kWideC * waves - 1) / (kWideC * waves);
  return (k + rounds * waves - 1) / (rounds * waves);
}

// Bytes a step moves: an updating member reads w and g and writes w (and
// reads and writes v), an averaging one reads and writes w.  `stream_bytes`:
// the bytes of one replica's parameters.
inline double step_bytes(const int32_t* k, const int32_t* act, int32_t units, bool mom,
                         int64_t stream_bytes) {
  double n = 0.0;
  for (int32_t u = 0; u < units; ++u) n += act[u] * (mom ? 5.0 : 3.0) + (k[u] - act[u]) * 2.0;
  return n * (double)stream_bytes;
}

// Whether a step is long enough to be split in two by the rule below: the
// second launch's ramp and tail cost a few microseconds, the better caps gain
// 1 to 5%.  Steps of a group of eight beside pairs, triples and lone updates,
// one launch at the mean cap against two: 12,293 elements 2.4 us against 4.3
// (fp32), 3.3 and 5.5 (momentum); 400,000 10.0 and 11.7; 12 fp32 replicas of
// 2.4M, 0.35 GB, 57.2 and 59.3; 24 with momentum of 1.2M, 0.58 GB, 103.1 and
// 104.5; 18 with momentum of 2.4M, 0.86 GB, 150.3 and 149.2; 28 with momentum
// of 2.4M, 1.3 GB, 231.6 and 225.3, of 5M 501 and 476.
constexpr double kSplitMinBytes = 1 << 30;
inline bool long_enough_to_split(double bytes) { return bytes >= kSplitMinBytes; }

// A step whose units prefer caps far apart (Global Division and Inter-Intra
// steps mix groups of two to eight, and lone updates, in one launch) runs
// as two launches, each at the cap of its own units: the units preferring
// at least kSplitCap waves per CU, then the others.  Only when the step has
// at least kSplitMinUnits units, each part carries at least kSplitMinShare
// of the step's bytes, and the parts' caps differ by at least kSplitMinGap;
// otherwise the second launch's ramp and tail cost more than the better
// caps gain (steps of one or two random groups).
constexpr int kSplitCap = 8;
constexpr int kSplitMinUnits = 3;
constexpr double kSplitMinShare = 0.15;
constexpr int kSplitMinGap = 4;
constexpr int kMaxUnits = 256;  // a launch's units are disjoint, so at most the replicas

// Decides the split of a launch's units.  Returns true and fills part[u]
// (0: the first launch, preferring >= kSplitCap waves; 1: the second) and
// the two launches' caps, or returns false (one launch at launch_waves).
inline bool split_units(const int32_t* k, const int32_t* act, int32_t units, bool mom,
                        uint8_t* part, int* waves0, int* waves1, bool segs = false) {
  if (units < kSplitMinUnits || units > kMaxUnits) return false;
  int32_t k0[kMaxUnits], a0[kMaxUnits], k1[kMaxUnits], a1[kMaxUnits];
  int32_t n0 = 0, n1 = 0;
  double b0 = 0.0, b1 = 0.0;
  for (int32_t u = 0; u < units; ++u) {
    const double bytes = act[u] * (mom ? 5.0 : 3.0) + (k[u] - act[u]) * 2.0;
    if (unit_waves(k[u], act[u], mom, segs) >= kSplitCap - 1e-9) {
      part[u] = 0;
      k0[n0] = k[u];
      a0[n0++] = act[u];
      b0 += bytes;
    } else {
      part[u] = 1;
      k1[n1] = k[u];
      a1[n1++] = act[u];
      b1 += bytes;
    }
  }
  if (n0 == 0 || n1 == 0) return false;
  if (b0 < kSplitMinShare * (b0 + b1) || b1 < kSplitMinShare * (b0 + b1)) return false;
  *waves0 = launch_waves(k0, a0, n0, mom, segs);
  *waves1 = launch_waves(k1, a1, n1, mom, segs);
  return *waves0 - *waves1 >= kSplitMinGap;
}

}  // namespace policy
}  // namespace rip
